// Host only: a launch of the grouped products has a workgroup for every tile that the groups can need, however the rows lie in them and however
// narrow the kernel makes its tiles, and no two for one.  The maps are the kernels' own (tile_of_block, fit_columns); exits with 1 on a fault.
#include <algorithm>
#include <cstdio>
#include <random>
#include <vector>

#include "gemm.h"

using namespace moe;

// Every one of `tiles` tiles is taken by the `grid` workgroups: once, or as its two halves
template <int SPLIT>
static bool all_taken(int grid, int tiles) {
    std::vector<int> whole(tiles, 0), halves(tiles, 0);
    for (int b = 0; b < grid; ++b) {
        int tile, half;
        if (!tile_of_block<SPLIT>(b, tiles, tile, half)) continue;
        if (tile < 0 || tile >= tiles || half > 1) return false;
        half < 0 ? ++whole[tile] : halves[tile] += 1 << 4 * half;
    }
    for (int t = 0; t < tiles; ++t)
        if (!(whole[t] == 1 && halves[t] == 0) && !(whole[t] == 0 && halves[t] == 0x11)) return false;
    return true;
}

int main() {
    std::mt19937 rng(7);
    auto below = [&](int n) { return (int)(rng() % (unsigned)n); };
    long long launches = 0, tight = 0, narrowed = 0, faults = 0;
    for (int it = 0; it < 20000; ++it) {
        const int E = 1 + below(it % 5 ? 16 : 64), BM = 16 << below(5), P = 1 + below(it % 3 ? 600 : 20000);
        std::vector<int> load(E, 0);
        int left = P;
        const int kind = below(4);
        if (kind == 0)  // a row more than whole tiles wherever there are rows for it: the most tiles that there can be
            for (int e = 0; e < E && left > 0; ++e) load[e] = 1, --left;
        for (int e = 0; left > 0 && kind == 0; e = (e + 1) % E) {
            const int n = std::min(left, BM);
            load[e] += n, left -= n;
        }
        for (; kind == 1 && left > 0; --left) ++load[below(E)];
        while (left > 0) {
            const int n = std::min(left, 1 + below(P)), e = below(kind == 2 ? E : std::min(E, 2));
            load[e] += n, left -= n;
        }
        int m_tiles = 0;
        for (int r : load) m_tiles += (r + BM - 1) / BM;
        const int bound = m_tiles_bound(P, E, BM);
        tight += m_tiles == bound;
        faults += m_tiles > bound;
        const int BN = 128 << below(2), N = 8 * (1 + below(it % 2 ? 128 : 768)), copies = 1 + below(4);
        const int n_tiles = (N + BN - 1) / BN;
        for (int split : {0, 32, 64})
            for (int fit : {0, 2}) {
                if (fit && split != 32) continue;
                int width = BN, n_base = n_tiles;
                if (fit) fit_columns(m_tiles * copies, N, fit, width, n_base);
                narrowed += width < BN;
                ++launches;
                const int grid = find_tile_grid(fitted_tiles(bound * n_tiles * copies, fit), split), tiles = m_tiles * n_base * copies;
                if (grid % 8 == 0 && (long long)n_base * width >= N && (split == 64 ? all_taken<64>(grid, tiles) : split == 32 ? all_taken<32>(grid, tiles) : all_taken<0>(grid, tiles))) continue;
                if (faults++ < 8) std::printf("%d rows in %d groups, tiles of %d rows, %d of %d columns, %d copies, split %d, fit %d\n", P, E, BM, N, width, copies, split, fit);
            }
    }
    std::printf("%lld launches, %lld loads at the bound, %lld with narrower tiles, %lld faults\n", launches, tight, narrowed, faults);
    return faults || tight < 1000 || narrowed < 1000;
}
