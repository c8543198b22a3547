// Host only: a launch of the grouped products has a workgroup for every tile that the groups can need, however the rows lie in them.
// The map from workgroups to tiles is the kernels' (find_tile), restated for a whole launch; exits with 1 where the grid is short.
#include <algorithm>
#include <cstdio>
#include <random>
#include <vector>

#include "gemm.h"

using namespace moe;

// workgroups per XCD that find_tile hands `tiles` tiles to
static int slots(int tiles, int split) {
    const int per_xcd = (tiles + 7) / 8;
    int most = 0;
    for (int x = 0; x < 8; ++x) {
        const int mine = std::max(0, std::min(per_xcd, tiles - x * per_xcd));
        const int whole = split ? mine / split * split : 0, rem = mine - whole;
        most = std::max(most, split && whole && rem && 2 * rem <= split ? whole + 2 * rem : mine);
    }
    return most;
}

int main() {
    std::mt19937 rng(7);
    auto below = [&](int n) { return (int)(rng() % (unsigned)n); };
    long long launches = 0, tight = 0, faults = 0;
    for (int it = 0; it < 200000; ++it) {
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
        const int n_tiles = 1 + below(it % 2 ? 8 : 60);
        for (int split : {0, 32, 64}) {
            ++launches;
            const int grid = find_tile_grid(bound * n_tiles, split);
            if (grid % 8 == 0 && slots(m_tiles * n_tiles, split) * 8 <= grid) continue;
            if (faults++ < 8) std::printf("%d rows in %d groups, tiles of %d rows, %d across, split %d\n", P, E, BM, n_tiles, split);
        }
    }
    std::printf("%lld launches, %lld loads at the bound, %lld faults\n", launches, tight, faults);
    return faults || tight < 1000;
}
