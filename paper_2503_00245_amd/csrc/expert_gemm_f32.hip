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
#include "router.h"

namespace moe {

template <int MI, int NI, int WAVES_M, int WAVES_N, int KS, bool SWIGLU>
__global__ __launch_bounds__(WAVES_M* WAVES_N* KS * 64) void gemm_f32_kernel(const GemmArgs g) {
    static_assert(KS == 1 || WAVES_M * WAVES_N == 1, "k-slices share one wave tile");
    constexpr int WM = 16 * MI, WN = 16 * NI, BM = WM * WAVES_M, BN = WN * WAVES_N;
    constexpr int ND = SWIGLU ? 2 : 1;
    int e, row0, row_end, nt;
    constexpr int NTHR = WAVES_M * WAVES_N * KS * 64;
    static_assert(NTHR == kF32DispatchThreads, "dispatch by whole workgroups");
    __shared__ int s_count[NTHR / kWave][kMaxExperts];
    __shared__ int s_pair[BM + kWave];
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
        keys.rows(e, row0 - MOE_READLANE(lo, e), rows, BM, s_count, s_pair);
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
    g.m_tiles_max = m_tiles_bound(g.P, g.E, BM);
    g.n_tiles = (g.N + BN - 1) / BN;
    const dim3 grid(find_tile_grid(g.m_tiles_max * g.n_tiles, 0)), block(WAVES_M * WAVES_N * KS * 64);
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

// ---- small layers of dense experts: two launches ----------------------------------------------------------------
// What bounds a small layer is launches, each a chain of memory latencies: routing, sorting inside the gate/up product,
// the down product and the combine took 16.0 us for 32 tokens of a 128 / 256 layer with 4 experts; the two launches here
// take 9.3 (64 / 136 with 8 experts 15.0 and 8.7, 256 / 640 with 2 18.9 and 11.3).  Every token
// meets every expert, so that no product waits for the routing: the tokens' rows are MFMA rows, h [E, T, F] holds them all,
// the routing runs beside the first product, and who chose whom matters only where the last one adds up.
//   token_gate_up  h[e, t] = silu(W_gate[e] x_t) * (W_up[e] x_t); the first route_blocks workgroups route
//   token_down     y_t = sum_j gate_tj W_down[e_tj] h[e_tj, t] (+ residual_t)
// Both on 16 x 16 tiles, the k-steps of one shared by waves, loads of D steps ahead of their MFMAs, tiles met in LDS.
constexpr int kTokenWaves = 16;
struct TokenLayer {
    const float *x, *w_gate, *w_up, *w_down;
    int T, d, F, E, k;
    int32_t* idx;
    float *gate, *h, *y;
    const float* residual;
    int slices;  // token_down: waves per expert
    const float *rw, *rb;
    int route_blocks;
};
// acc[m] += A row of the lane . B[m] row of the lane over the k-steps first, first + stride, ... of K.  (The next D on
// their way beside the present ones: slower, 17.3 -> 21.3 us for 32 tokens of 256 / 640, fewer waves fit.)
// The products of D steps are summed in 4 CHAINS chains apart, which meet pair by pair: one chain over all steps was up to 96 products
// long, and two tokens, whose lanes' chains on the matrix-vector path are of a few, were 1.5 times as far from 64 bits as there (120 layers of
// 2 to 8 experts, 64 to 512 wide, geometric mean; 1.00 now, 1.04 with CHAINS 1.  Three tokens and more against the stage by stage way: 0.95, 0.61 now).
// CHAINS 2 for two tokens alone: where the chip is full its registers and sums cost time (4 experts of 256 / 640, 64 tokens, 18.2 us before,
// 18.4 with 1, 20.0 with 2; two tokens of 2 experts 8.9, 9.2, 9.8; on the matrix-vector path 12 and more).
template <int D, int CHAINS, int NM>
__device__ __forceinline__ void token_tile(const float* pa, const float* const (&pb)[NM], int K, int first, int stride, f32x4 (&acc)[NM]) {
    const int quad = (threadIdx.x & (kWave - 1)) >> 4;
    int st = first, left = uniform_div((K + 15) / 16 - first + stride - 1, stride);  // the wave's steps
    // N steps at once: as many as there are, so that no load is for nothing and none stands behind a branch around a step's products,
    // where the compiler moves it (N memory latencies in a row).  Whole layer, us, with such branches / without: 32 tokens of
    // 128 / 256, 4 experts, 9.9 / 9.3, 5 tokens of 200 / 488 11.1 / 9.5, 2 experts of 448 / 1200, 3 tokens, 13.2 / 11.4; 14 shapes 1.07
    // (geometric mean, 1.00 the least).  D loads at all times: 1 of 8 experts of 64 / 160, 200 tokens, 12.9 / 13.9.
    auto batch = [&](auto n) {
        constexpr int N = decltype(n)::value;
        f32x4 a[N], b[NM][N];
#pragma unroll
        for (int q = 0; q < N; ++q) {  // (past the row's end: its last 16 bytes)
            const int k = min((st + q * stride) * 16 + quad * 4, K - 4);
            a[q] = *reinterpret_cast<const f32x4*>(pa + k);
#pragma unroll
            for (int m = 0; m < NM; ++m) b[m][q] = *reinterpret_cast<const f32x4*>(pb[m] + k);
        }
        __builtin_amdgcn_sched_barrier(0);
        f32x4 part[NM][CHAINS][4];
#pragma unroll
        for (int m = 0; m < NM; ++m)
#pragma unroll
            for (int i = 0; i < CHAINS; ++i)
#pragma unroll
                for (int c = 0; c < 4; ++c) part[m][i][c] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < N; ++q) {
            const bool in = (st + q * stride) * 16 + quad * 4 < K;  // beyond K: both operands cleared
#pragma unroll
            for (int m = 0; m < NM; ++m)
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    f32x4& p = part[m][q % CHAINS][c];
                    p = __builtin_amdgcn_mfma_f32_16x16x4f32(in ? a[q][c] : 0.f, in ? b[m][q][c] : 0.f, p, 0, 0, 0);
                }
        }
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            f32x4 sum = (part[m][0][0] + part[m][0][1]) + (part[m][0][2] + part[m][0][3]);
            if (CHAINS == 2) sum += (part[m][CHAINS - 1][0] + part[m][CHAINS - 1][1]) + (part[m][CHAINS - 1][2] + part[m][CHAINS - 1][3]);
            acc[m] += sum;
        }
        st += N * stride;
        left -= N;
    };
    while (left >= D) batch(std::integral_constant<int, D>{});
    if (left <= 0) return;
    static_for<D - 1>([&](auto n) {
        if (left == n + 1) batch(std::integral_constant<int, n + 1>{});
    });
}

template <int D, int CHAINS>
__global__ __launch_bounds__(kRouteWaves* kWave) void token_gate_up_f32_kernel(
    ptr_arg ax, ptr_arg a_gate, ptr_arg a_up, int route_blocks, int T, int d, int F, int E, const TokenLayer g) {
    const float* const x = from_arg<const float>(ax);
    if ((int)blockIdx.x < route_blocks) {
        route_tokens<float, 4, kRouteTok>(g.x, g.rw, g.rb, g.idx, g.gate, nullptr, g.T, g.d, g.E, g.k, blockIdx.x);
        return;
    }
    __shared__ float s_part[2][kRouteWaves][16][17];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int blocks = (F + 15) / 16, at = (int)blockIdx.x - route_blocks;
    const int te = uniform_div(at, blocks), f0 = (at - te * blocks) * 16, tb = uniform_div(te, E), e = te - tb * E, t0 = tb * 16;
    const int i = lane & 15, quad = lane >> 4;
    const float* pa = x + (size_t)min(t0 + i, T - 1) * d;
    const size_t row = ((size_t)e * F + min(f0 + i, F - 1)) * d;
    const float* const pb[2] = {from_arg<const float>(a_gate) + row, from_arg<const float>(a_up) + row};
    f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
    token_tile<D, CHAINS, 2>(pa, pb, d, wave, kRouteWaves, acc);
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int r = 0; r < 4; ++r) s_part[m][wave][4 * quad + r][i] = acc[m][r];
    __syncthreads();
    const int t = threadIdx.x >> 4, c = threadIdx.x & 15;
    if (t >= 16 || t0 + t >= T || f0 + c >= F) return;
    float z[2] = {0.f, 0.f};
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int w = 0; w < kRouteWaves; w += 4)
            z[m] += (s_part[m][w][t][c] + s_part[m][w + 1][t][c]) + (s_part[m][w + 2][t][c] + s_part[m][w + 3][t][c]);
    g.h[((size_t)e * T + t0 + t) * F + f0 + c] = silu_f32(z[0]) * z[1];
}

template <int D, int CHAINS>
__global__ __launch_bounds__(kTokenWaves* kWave) __attribute__((amdgpu_waves_per_eu(4, 4))) void token_down_f32_kernel(
    ptr_arg ah, ptr_arg aw, ptr_arg ai, ptr_arg ag, int T, int d, int F, int E, int slices, int k, const TokenLayer g) {
    const float *const h = from_arg<const float>(ah), *const w_down = from_arg<const float>(aw), *const gates = from_arg<const float>(ag);
    const int32_t* const idx = from_arg<const int32_t>(ai);
    __shared__ float s_part[kTokenWaves][16][17];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int n0 = blockIdx.x * 16, t0 = blockIdx.y * 16;
    const int e = uniform_div(wave, slices), ks = wave - e * slices;
    const int i = lane & 15, quad = lane >> 4;
    const int t = t0 + (int)(threadIdx.x >> 4), n = n0 + (int)(threadIdx.x & 15);  // what the thread adds up
    const bool mine = threadIdx.x < 256 && t < T && n < d;
    // The first two experts and gates, and the residual, are requested with the products' operands.  (Experts and gates without a condition: the
    // compiler would wait for them where its branch ends.  The residual stands behind one, and its pointer, of the struct, is waited for ahead of the operands.)
    const int pair = min(t, T - 1) * k;
    const int e0 = idx[pair], e1 = idx[pair + min(1, k - 1)];
    const float gate0 = gates[pair], gate1 = gates[pair + min(1, k - 1)];
    const float res = g.residual ? g.residual[(size_t)min(t, T - 1) * d + min(n, d - 1)] : 0.f;
    f32x4 acc[1] = {f32x4{0.f, 0.f, 0.f, 0.f}};
    if (e < E) {
        const float* const pb[1] = {w_down + ((size_t)e * d + min(n0 + i, d - 1)) * F};
        token_tile<D, CHAINS, 1>(h + ((size_t)e * T + min(t0 + i, T - 1)) * F, pb, F, ks, slices, acc);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) s_part[wave][4 * quad + r][i] = acc[0][r];
    __syncthreads();
    if (!mine) return;
    float total = 0.f;
    for (int j = 0; j < k; ++j) {
        const int ej = min(max(j == 0 ? e0 : j == 1 ? e1 : idx[t * k + j], 0), E - 1);
        float sum[2] = {0.f, 0.f};
        for (int sl = 0; sl < slices; sl += CHAINS)
#pragma unroll
            for (int i = 0; i < CHAINS; ++i)
                if (i == 0 || sl + i < slices) sum[i] += s_part[ej * slices + sl + i][threadIdx.x >> 4][threadIdx.x & 15];
        total = fmaf(j == 0 ? gate0 : j == 1 ? gate1 : gates[t * k + j], sum[0] + sum[1], total);
    }
    g.y[(size_t)t * d + n] = total + res;
}

// Where this is the faster way (whole layer, us, stage by stage / this): the down product's workgroups, one per 16 columns,
// read the 16 rows of all experts, so E F is bounded -- 32 tokens, 2 of 8 experts of 256 / 640 22.0 / 27.0, 4 experts 21.3 / 17.3 --
// and the products grow by E / k (32, 128, 256 tokens, 2 of 8 experts of 128 / 256 15.7 / 13.4, 17.4 / 16.6, 19.1 / 19.7; 1 of 4 of
// 256 / 640 64 tokens 20.4 / 18.2, 128 tokens 21.5 / 21.0, 256 tokens 23.2 / 28.6).  Two tokens otherwise take the
// matrix-vector path: 2 of 4 experts of 128 / 256 12.3 / 8.3.
bool token_layer_f32_shape(const moe_shape& s) {
    return s.act_dtype == MOE_F32 && s.rank == 0 && s.n_experts <= kTokenWaves && s.d_model <= 1024 &&
           (long long)s.n_experts * s.d_ff <= 3072;
}
bool token_layer_f32_supported(const moe_shape& s) {
    return token_layer_f32_shape(s) && s.n_tokens > 1 && token_layer_bytes(s) <= kTokenLayerBytes &&
           (double)s.n_tokens * s.d_model * s.d_ff * s.n_experts * s.n_experts <= 200e6 * s.top_k;
}
int launch_token_layer_f32(const moe_shape& s, const moe_weights& w, const void* x, int32_t* idx, float* gate, float* h,
                           const void* residual, void* y, hipStream_t st, StageTimer* timer) {
    int slices = kTokenWaves;
    while (slices * s.n_experts > kTokenWaves) slices /= 2;
    const int route_blocks = (s.n_tokens + kRouteTok - 1) / kRouteTok;
    const TokenLayer g{static_cast<const float*>(x), static_cast<const float*>(w.w_gate), static_cast<const float*>(w.w_up),
                       static_cast<const float*>(w.w_down), s.n_tokens, s.d_model, s.d_ff, s.n_experts, s.top_k, idx, gate, h,
                       static_cast<float*>(y), static_cast<const float*>(residual), slices, w.router_w, w.router_b, route_blocks};
    const int tb = (s.n_tokens + 15) / 16;
    const dim3 grid(route_blocks + tb * s.n_experts * ((s.d_ff + 15) / 16));
    const bool two = s.n_tokens == 2;
    // (3 and not 4 steps at once of the longest rows: 94 registers would be two workgroups a CU for three, 48 tokens of 320 / 760 18.7 / 17.6)
    const auto first = s.d_model <= 16 * kRouteWaves       ? token_gate_up_f32_kernel<1, 1>
                       : s.d_model <= 2 * 16 * kRouteWaves ? (two ? token_gate_up_f32_kernel<2, 2> : token_gate_up_f32_kernel<2, 1>)
                                                           : (two ? token_gate_up_f32_kernel<3, 2> : token_gate_up_f32_kernel<3, 1>);
    hipLaunchKernelGGL(first, grid, dim3(kRouteWaves * kWave), 0, st, as_arg(x), as_arg(w.w_gate), as_arg(w.w_up), route_blocks, s.n_tokens, s.d_model,
                       s.d_ff, s.n_experts, g);
    int rc = launch_status();
    if (rc != MOE_OK) return rc;
    stage_mark(timer, "route_gate_up_swiglu");
    hipLaunchKernelGGL((two ? token_down_f32_kernel<4, 2> : token_down_f32_kernel<4, 1>), dim3((s.d_model + 15) / 16, tb), dim3(kTokenWaves * kWave), 0, st,
                       as_arg(h), as_arg(w.w_down), as_arg(idx), as_arg(gate), s.n_tokens, s.d_model, s.d_ff, s.n_experts, slices, s.top_k, g);
    rc = launch_status();
    stage_mark(timer, "gemm_down_combine");
    return rc;
}

}  // namespace moe
