// Grouped expert GEMM on fp32 storage (gemm.h states the problem), on v_mfma_f32_16x16x4_f32.
//
// An fp32 MFMA takes 16 times as long per multiply-add as a bf16 one, so here the operands need no
// staging: a lane reads 16 bytes of one row straight from memory -- row lane % 16, k-quad lane / 16 of
// a 16-wide k-step -- and element j of that quad is its operand of the step's j-th MFMA.  (An MFMA sums
// over the k its four lane groups hold, whichever those are, as long as both operands agree.)  The
// rows a workgroup's waves share meet in L1.  The next k-step is loaded while the present one multiplies.
//
// KS > 1: the waves of a workgroup take the k-steps of one tile in turn and add up in LDS, in wave
// order: for calls with few tiles, where the chain of k-steps of a tile is what takes the time.
//
// (The 64 x 64 LDS-tiled FMA kernel that this one replaces took 32 us for either product of a
// 32-token, 128 / 256-wide layer -- 16 or fewer workgroups, a barrier pair per 16 of k.  Whole layer there
// 76 us before, 19.6 now; 512 tokens of a 512 / 1400 layer with 8 experts 516 before, 91 now.)
#include "gemm.h"

namespace moe {

template <int MI, int NI, int WAVES_M, int WAVES_N, int KS, bool SWIGLU>
__global__ __launch_bounds__(WAVES_M* WAVES_N* KS * 64) void gemm_f32_kernel(const GemmArgs g) {
    static_assert(KS == 1 || WAVES_M * WAVES_N == 1, "k-slices share one wave tile");
    constexpr int WM = 16 * MI, WN = 16 * NI, BM = WM * WAVES_M, BN = WN * WAVES_N;
    constexpr int ND = SWIGLU ? 2 : 1;
    int e, row0, row_end, nt;
    constexpr int NTHR = WAVES_M * WAVES_N * KS * 64;
    static_assert(NTHR == kF32DispatchThreads, "dispatch by whole workgroups");
    __shared__ int s_count[kKeyChunks * NTHR / kWave][kMaxExperts];
    __shared__ int s_pair[BM];
    int lo, hi;
    PairKeys<NTHR> keys;
    if (g.keys) {
        keys.load(g.keys, g.P);
        keys.bounds(g.E, s_count, lo, hi);
        if (blockIdx.x == 0 && threadIdx.x < 64) {
            if ((int)threadIdx.x < g.E) g.offsets[threadIdx.x] = lo;
            if ((int)threadIdx.x == g.E - 1) g.offsets[g.E] = hi;
        }
    } else {
        group_bounds(g.offsets, g.E, g.P, lo, hi);
    }
    if (!find_tile(lo, hi, g.E, BM, [&](int) { return g.n_tiles; }, e, row0, row_end, nt)) return;
    if (g.keys) {
        const int rows = min(row_end - row0, BM);
        keys.rows(e, row0 - MOE_READLANE(lo, e), rows, s_count, s_pair);
        if (nt == 0) {  // one column tile of each row tile writes the sorted order
            for (int r = threadIdx.x; r < rows; r += NTHR) {
                const int p = s_pair[r];
                g.row_map[row0 + r] = p;
                g.inv_perm[p] = row0 + r;
            }
        }
    }
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int ks = KS > 1 ? wave : 0;
    const int wm = KS > 1 ? 0 : wave / WAVES_N, wn = KS > 1 ? 0 : wave % WAVES_N;
    const int r = lane & 15, quad = lane >> 4;
    const int m0 = row0 + wm * WM, n0 = nt * BN + wn * WN;

    f32x4 acc[ND][MI][NI];
#pragma unroll
    for (int s = 0; s < ND; ++s)
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j) acc[s][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    struct Frags {
        f32x4 a[ND][MI], b[ND][NI];
    };
    for (int sidx = 0; sidx < g.nseg; ++sidx) {
        const GemmSeg& sg = g.seg[sidx];
        const int K = sg.K;
        const bool two_a = SWIGLU && sg.A1 != sg.A0;
        const float* pa[ND][MI];
        const float* pb[ND][NI];
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            int row = min(m0 + 16 * i + r, row_end - 1);
            if (sg.gather) row = quick_div(min(max(g.keys ? s_pair[row - row0] : g.row_map[row], 0), g.P - 1), g.row_div);
            pa[0][i] = static_cast<const float*>(sg.A0) + (size_t)row * K;
            if (SWIGLU) pa[ND - 1][i] = static_cast<const float*>(sg.A1) + (size_t)row * K;
        }
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            const size_t off = (size_t)e * sg.strideB + (size_t)min(n0 + 16 * j + r, g.N - 1) * K;
            pb[0][j] = static_cast<const float*>(sg.B0) + off;
            if (SWIGLU) pb[ND - 1][j] = static_cast<const float*>(sg.B1) + off;
        }
        // K is a multiple of 4: a lane's quad of the last step is whole or beyond K (then read from
        // the row's last quad, in bounds, and the A side cleared)
        auto load = [&](Frags& f, int step) {
            const int k = step * 16 + quad * 4;
            const int at = min(k, K - 4);
#pragma unroll
            for (int i = 0; i < MI; ++i) {
                f.a[0][i] = *reinterpret_cast<const f32x4*>(pa[0][i] + at);
                if (SWIGLU) f.a[ND - 1][i] = two_a ? *reinterpret_cast<const f32x4*>(pa[ND - 1][i] + at) : f.a[0][i];
            }
#pragma unroll
            for (int s = 0; s < ND; ++s)
#pragma unroll
                for (int j = 0; j < NI; ++j) f.b[s][j] = *reinterpret_cast<const f32x4*>(pb[s][j] + at);
            if (k >= K) {
#pragma unroll
                for (int s = 0; s < ND; ++s)
#pragma unroll
                    for (int i = 0; i < MI; ++i) f.a[s][i] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
        };
        auto multiply = [&](const Frags& f) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int s = 0; s < ND; ++s)
#pragma unroll
                    for (int i = 0; i < MI; ++i)
#pragma unroll
                        for (int j = 0; j < NI; ++j)
                            acc[s][i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(f.a[s][i][q], f.b[s][j][q],
                                                                               acc[s][i][j], 0, 0, 0);
        };
        const int steps = (K + 15) / 16;
        if (ks >= steps) continue;
        Frags f0, f1;
        load(f0, ks);
        int st = ks;
        for (; st + KS < steps; st += 2 * KS) {
            load(f1, st + KS);
            multiply(f0);
            load(f0, min(st + 2 * KS, steps - 1));  // (past the end: a step that is not used)
            multiply(f1);
        }
        if (st < steps) multiply(f0);
    }

    if constexpr (KS > 1) {
        constexpr int NF = ND * MI * NI;
        __shared__ f32x4 s_part[KS - 1][NF][kWave];
        if (ks > 0) {
#pragma unroll
            for (int q = 0; q < NF; ++q) s_part[ks - 1][q][lane] = acc[q / (MI * NI)][q / NI % MI][q % NI];
        }
        __syncthreads();
        if (ks > 0) return;
        for (int w = 0; w < KS - 1; ++w)
#pragma unroll
            for (int q = 0; q < NF; ++q) acc[q / (MI * NI)][q / NI % MI][q % NI] += s_part[w][q][lane];
    }
    // accumulator element i sits at row 4 * (lane / 16) + i, column lane % 16 of its 16 x 16 block
    float* C = static_cast<float*>(g.C);
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            const int col = n0 + 16 * j + r;
            if (col >= g.N) continue;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int row = m0 + 16 * i + 4 * quad + t;
                if (row >= row_end) break;
                const float v = acc[0][i][j][t];
                C[(size_t)row * g.N + col] = SWIGLU ? silu_f32(v) * acc[ND - 1][i][j][t] : v;
            }
        }
}

template <int MI, int NI, int WAVES_M, int WAVES_N, int KS>
static int launch_f32(GemmArgs& g, bool swiglu, hipStream_t st) {
    constexpr int BM = 16 * MI * WAVES_M, BN = 16 * NI * WAVES_N;
    g.m_tiles_max = g.P / BM + g.E;
    g.n_tiles = (g.N + BN - 1) / BN;
    const dim3 grid((g.m_tiles_max * g.n_tiles + 7) / 8 * 8), block(WAVES_M * WAVES_N * KS * 64);
    if (swiglu)
        hipLaunchKernelGGL((gemm_f32_kernel<MI, NI, WAVES_M, WAVES_N, KS, true>), grid, block, 0, st, g);
    else
        hipLaunchKernelGGL((gemm_f32_kernel<MI, NI, WAVES_M, WAVES_N, KS, false>), grid, block, 0, st, g);
    return launch_status();
}

int run_gemm_f32(GemmArgs& g, bool swiglu, hipStream_t st) {
    // Tiles of 64 x 64 once there are enough of them for 256 CUs; before that smaller tiles with the
    // k-steps shared by four waves, 32 x 32 and, for the smallest products, 16 x 16.
    auto tiles = [&](int b) { return (long long)(g.P / b + (g.E + 1) / 2) * ((g.N + b - 1) / b); };
    if (tiles(64) >= 256) return launch_f32<2, 2, 2, 2, 1>(g, swiglu, st);
    if (tiles(32) >= 256) return launch_f32<2, 2, 1, 1, 4>(g, swiglu, st);
    return launch_f32<1, 1, 1, 1, 4>(g, swiglu, st);
}

}  // namespace moe
