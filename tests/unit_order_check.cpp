// Host only: the orders in which a single token's waves take their rows (first_stage_turns, hidden_turns, place_in_rest) take every row once, and keep
// neighbouring rows in one workgroup, but for the rest, where rows are no whole cache lines, and in the first stage where they are short.  The
// walks are those of decode_first_kernel and decode_hidden_kernel; exits with 1 on a fault.
#include <algorithm>
#include <cstdio>
#include <vector>

#include "gemv.h"

using namespace moe;

static long long faults = 0;

// Every unit taken once; of the first `whole`, neighbours in one workgroup as often as on `waves` waves in their order
static void look(const char* what, const std::vector<int>& taken, const std::vector<int>& block_of, int whole, int waves, int per_block, int k, int rows, int row_bytes) {
    bool ok = *std::min_element(taken.begin(), taken.end()) == 1 && *std::max_element(taken.begin(), taken.end()) == 1;
    int changes = 0, most = 0;
    for (int i = 1; i < whole; ++i) {
        changes += block_of[i] != block_of[i - 1];
        most += i % waves * per_block / kOneWaves != (i - 1) % waves * per_block / kOneWaves;
    }
    if ((!ok || changes > most) && faults++ < 8) std::printf("%s: %d pairs of %d rows of %d bytes\n", what, k, rows, row_bytes);
}

int main() {
    long long orders[6] = {0};
    for (int k = 1; k <= 64; k += k < 16 ? 1 : 8)
        for (int rows = 8; rows <= 9000; rows += rows < 600 || rows % 256 < 16 ? 24 : 232) {
            const int units = k * rows, blocks = std::min(kOneCus, (units + kOneWaves - 1) / kOneWaves);
            std::vector<int> taken(units), block_of(units);
            for (int row_bytes : {2048, 2560, 2608, 4096}) {
                const int turns = first_stage_turns(units, blocks, row_bytes), stride = blocks * kOneWaves;
                ++orders[turns < 0 ? 2 : turns > 0];
                std::fill(taken.begin(), taken.end(), 0);
                for (int b = 0; b < blocks; ++b)
                    for (int w = 0; w < kOneWaves; ++w) {
                        const int in_order = b * kOneWaves + w;
                        int left = turns;
                        for (int i = turns < 0 ? w * blocks + b : in_order; i < units; i += --left == 0 ? stride + place_in_rest(b, w, blocks) - in_order : stride) {
                            ++taken[i];
                            block_of[i] = b;
                        }
                    }
                look("first stage", taken, block_of, row_bytes < 4096 ? units / stride * stride : 0, stride, 1, k, rows, row_bytes);
            }
            const int waves = blocks * kOneWaves / k;
            for (int row_bytes : {528, 640}) {
                const int turns = hidden_turns(rows, waves, k, row_bytes);
                ++orders[turns < 0 ? 5 : turns > 0 ? 4 : 3];
                std::fill(taken.begin(), taken.end(), 0);
                for (int b = 0; b < blocks; ++b)
                    for (int w = 0; w < kOneWaves; ++w) {
                        const int at = turns < 0 ? w * blocks + b : b * kOneWaves + w, first = at / k, j = at % k;
                        if (first >= waves) continue;
                        int left = turns;
                        const int to_rest = waves + place_in_rest(b, w / k, kOneCus) - first;
                        for (int row = first; row < rows; row += --left == 0 ? to_rest : waves) {
                            ++taken[j * rows + row];
                            block_of[j * rows + row] = b;
                        }
                    }
                look("rank rows", taken, block_of, row_bytes % 128 ? rows / waves * waves : 0, waves, k, k, rows, row_bytes);
            }
        }
    std::printf("first stage: waves first %lld, the rest alone %lld, workgroups first %lld; rank rows: %lld, %lld, %lld; %lld faults\n", orders[0], orders[1],
                orders[2], orders[3], orders[4], orders[5], faults);
    return faults || *std::min_element(orders, orders + 6) == 0;
}
