// Host only: the order in which the waves of a single token's rank experts take a pair's rows (hidden_turns, place_in_rest) takes every row once,
// and leaves neighbouring rows of no whole cache lines in one workgroup, but for the rest.  The walk is decode_hidden_kernel's; exits with 1 on a fault.
#include <algorithm>
#include <cstdio>
#include <vector>

#include "gemv.h"

using namespace moe;

int main() {
    long long faults = 0, orders[3] = {0, 0, 0};
    for (int k = 1; k <= 64; k += k < 16 ? 1 : 8)
        for (int rows = 8; rows <= 9000; rows += rows < 600 ? 8 : rows % 128 < 16 ? 24 : 104)
            for (int row_bytes : {528, 640}) {
                const long long units = (long long)k * rows;
                const int blocks = (int)std::min<long long>(kOneCus, (units + kOneWaves - 1) / kOneWaves), waves = blocks * kOneWaves / k;
                const int turns = hidden_turns(rows, waves, k, row_bytes);
                ++orders[turns < 0 ? 2 : turns > 0];
                std::vector<int> taken(units, 0), block_of(units, -1);
                for (int b = 0; b < blocks; ++b)
                    for (int w = 0; w < kOneWaves; ++w) {
                        const int at = turns < 0 ? w * blocks + b : b * kOneWaves + w, first = at / k, j = at % k;
                        if (first >= waves) continue;
                        int left = turns;
                        const int to_rest = waves + place_in_rest(b, w / k, kOneCus) - first;
                        for (int row = first; row < rows; row += --left == 0 ? to_rest : waves) {
                            ++taken[(size_t)j * rows + row];
                            block_of[(size_t)j * rows + row] = b;
                        }
                    }
                bool ok = *std::min_element(taken.begin(), taken.end()) == 1 && *std::max_element(taken.begin(), taken.end()) == 1;
                if (row_bytes % 128) {  // as many changes of workgroup as waves first has
                    const int whole = rows / waves * waves;
                    int changes = 0, most = 0;
                    for (int row = 1; row < whole; ++row) {
                        changes += block_of[row] != block_of[row - 1];
                        most += row % waves * k / kOneWaves != (row - 1) % waves * k / kOneWaves;
                    }
                    ok = ok && changes <= most;
                }
                if (!ok && faults++ < 8) std::printf("k %d, %d rows of %d bytes, %d workgroups, %d turns\n", k, rows, row_bytes, blocks, turns);
            }
    std::printf("waves first %lld, the rest alone %lld, workgroups first %lld, %lld faults\n", orders[0], orders[1], orders[2], faults);
    return faults || !orders[0] || !orders[1] || !orders[2];
}
