// Host only: whatever parts the plan of a call cuts a product into, a kernel that writes parts takes that product.
// Linked against the library's objects; prints the shapes where the two disagree and exits with 1.
#include <cstdio>

#include "gemm.h"

using namespace moe;

static int faults = 0, products = 0;

static void check(const moe_shape& s, const char* what, int parts, bool f32, int P, int E, int N, int K) {
    if (parts <= 1) return;
    ++products;
    GemmArgs g{};
    g.nseg = 1, g.E = E, g.P = P, g.N = N, g.row_div = 1, g.k_parts = parts, g.parts_f32 = f32;
    g.few = gemm_few_rows((long long)s.n_tokens * s.top_k, s.top_k) ? s.n_tokens : 0;
    g.seg[0].K = K;
    if (gemm_few_supported(g) || gemm_pp_supported(g)) return;
    if (faults++ < 8)
        std::printf("%s in %d parts: %d tokens, d_model %d, d_ff %d, %d of %d experts, rank %d, flags %d\n", what, parts, s.n_tokens,
                    s.d_model, s.d_ff, s.top_k, s.n_experts, s.rank, s.flags);
}

int main() {
    const int widths[] = {8, 64, 432, 1032, 2048, 5632, 8192, 16384, 65536, 262136, 262144, 524288, 1 << 20, (1 << 23) - 8, 1 << 23};
    const int ranks[] = {0, 8, 64, 1024, 1032, 8192, 262144};
    const int experts[][2] = {{1, 1}, {8, 1}, {8, 2}, {16, 4}};
    const int tokens[] = {1, 2, 3, 8, 16, 17, 32, 33, 100, 300, 2048, 20000};
    const size_t rooms[] = {1u << 16, 8u << 20, 200u << 20, (size_t)1 << 40};
    for (int d : widths)
        for (int F : widths)
            for (int r : ranks)
                for (const auto& e : experts)
                    for (int T : tokens)
                        for (size_t room : rooms)
                            for (int flags = 0; flags <= (r ? MOE_FLAG_SHARED_BASE : 0); flags += MOE_FLAG_SHARED_BASE) {
                                moe_shape s{};
                                s.n_tokens = T, s.d_model = d, s.d_ff = F, s.n_experts = e[0], s.top_k = e[1], s.rank = r;
                                s.act_dtype = MOE_BF16, s.flags = flags;
                                const SplitPlan p = split_plan(s, room, room);
                                const int P = T * s.top_k;
                                check(s, "down", p.down, p.down_f32, P, s.n_experts, d, r ? r : F);
                                check(s, "rank-down", p.rank_down, true, P, s.n_experts, r, F);
                                check(s, "base down", p.base_down, true, T, 1, d, F);
                            }
    std::printf("%d products in parts, %d without a kernel\n", products, faults);
    return faults || products < 1000;
}
