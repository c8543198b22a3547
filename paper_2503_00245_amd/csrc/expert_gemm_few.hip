// Grouped bf16 GEMM for few rows per group (gemm.h states the problem).
//
// What bounds it: the experts' weights, read once from HBM.  The direct-fill kernels read them behind barriers, a k-step of
// 128 bytes per row at a time, and pay for two rounds of tiles: 8 tokens of 2048 / 5632, 290 MB of gate and up weights, took
// 60 us there (4.8 TB/s) and take 49 here (5.9; a plain read of that size 47.5).  So here
//   - one workgroup per CU walks an equal share of all (group, part of K, 16 output columns) units;
//   - its eight waves split a unit's K, so that a wave's share of the activations stays in registers while the group's
//     columns go by, and a unit ends in one sum over the waves through LDS, made by one wave in turn;
//   - a wave has one to two chunks of eight 1 KB loads in flight, past the caches, in the longest runs its share of a
//     row gives (load, below); the way into MFMA layout is through a region of LDS of the wave's own, with no barrier;
//   - the one barrier per unit waits for no load.
#include "gemm.h"

namespace moe {

namespace {

constexpr int kStepK = 32;      // k of one MFMA
constexpr int kWaves = 8;       // per workgroup: two per SIMD, so a wave may hold 256 registers
constexpr int kMaxSteps = 8;    // MFMA k-steps of a wave
constexpr int kKeyWords = 4;    // pairs' keys per lane
constexpr int kGrid = 256;      // one workgroup per CU

__device__ __forceinline__ void lds_barrier() {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#endif
}

// LDS written by one lane of a wave and read by another: the hardware keeps the order, the compiler has to
__device__ __forceinline__ void wave_lds_order() {
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_wave_barrier();
    asm volatile("" ::: "memory");
#endif
}
// The lane index, counted anew: what is derived from it is computed where it is used, not kept in registers
__device__ __forceinline__ int lane_again() {
#if defined(__HIP_DEVICE_COMPILE__)
    int v = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    asm volatile("" : "+v"(v));
    return v;
#else
    return 0;
#endif
}
__device__ __forceinline__ void wait_loads() {
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
#endif
}

// A unit's weights are requested in chunks of up to eight loads: both matrices at once, or one after the other.
constexpr int chunks(int s, bool pair) { return pair && s > 4 ? 2 : 1; }
template <int MT, int S, bool PAIR>
constexpr int region_bytes() {
    constexpr int nm = PAIR ? 2 : 1, stage = nm / chunks(S, PAIR) * 16 * (S * 64 + 16), part = nm * MT * kWave * 16;
    return stage > part ? stage : part;
}

// Wave w of the workgroup's NW owns the w-th share of every row's k-steps (of the part's, where K is cut into parts).
// MT: 16-row blocks of activations held.  S: k-steps of a wave, at most.
// PAIR: two matrices (gate and up, or C and C1); SWIGLU: one output of both; DUAL: the second has activations of its own.
// F32: k-parts in fp32.
template <int MT, int S, bool PAIR, bool SWIGLU, bool DUAL, bool F32>
__global__ __launch_bounds__(kWaves* kWave) __attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_few_kernel(
    ptr_arg a_keys, ptr_arg a_offsets, int g_P, int g_E, const GemmArgs g) {
    const int32_t *const g_keys = from_arg<const int32_t>(a_keys), *const g_offsets = from_arg<const int32_t>(a_offsets);
    static_assert(!SWIGLU || PAIR, "the activation takes two products");
    static_assert(!DUAL || PAIR, "two activation operands with two matrices");
    constexpr int NW = kWaves, NM = PAIR ? 2 : 1, NX = DUAL ? 2 : 1, ROWS = 16 * MT;
    constexpr int CHUNKS = chunks(S, PAIR), CM = NM / CHUNKS;  // chunks of a unit, matrices of a chunk
    // LDS, per wave: two regions by turns, each first the weights on their way into MFMA layout, then the wave's
    // partial sums [NM][MT][64]; and the group's pairs
    constexpr int PITCH = S * 64 + 16, REGION = region_bytes<MT, S, PAIR>();
    extern __shared__ __align__(16) char smem[];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    int* const s_rows = reinterpret_cast<int*>(smem + 2 * NW * REGION) + wave * ROWS;
    char* const my_region = smem + wave * REGION;

    const GemmSeg& sg = g.seg[0];
    const int K = sg.K, N = g.N, E = g_E;
    const int parts = F32 ? g.k_parts : 1;
    const int steps = (K + kStepK - 1) / kStepK, blocks = (N + 15) / 16;

    // ---- groups: in lane e, group e's bounds
    int lo, hi, key[kKeyWords];
    if (g_keys) {
#pragma unroll
        for (int c = 0; c < kKeyWords; ++c) key[c] = c * kWave + lane < g_P ? g_keys[c * kWave + lane] : -1;
        int at = 0;
        lo = hi = 0;
        int slot[kKeyWords];
#pragma unroll
        for (int c = 0; c < kKeyWords; ++c) slot[c] = -1;
        for (int e = 0; e < E; ++e) {
            if (lane == e) lo = at;
#pragma unroll
            for (int c = 0; c < kKeyWords; ++c) {
                const unsigned long long same = __ballot(key[c] == e);
                if (key[c] == e) slot[c] = at + lanes_below(same);
                at += __popcll(same);
            }
            if (lane == e) hi = at;
        }
        if (blockIdx.x == 0 && wave == 0) {  // the sorted order, for later stages
            if (lane < E) g.offsets[lane] = lo;
            if (lane == E - 1) g.offsets[E] = hi;
#pragma unroll
            for (int c = 0; c < kKeyWords; ++c)
                if (slot[c] >= 0) {
                    g.row_map[slot[c]] = c * kWave + lane;
                    g.inv_perm[c * kWave + lane] = slot[c];
                }
        }
    } else {
        group_bounds(g_offsets, E, g_P, lo, hi);
    }

    // ---- this workgroup's share of the units (group, part, 16 output columns), in that order
    const int cnt = (hi - lo + ROWS - 1) / ROWS;  // a group of more than ROWS rows counts several times
    int total = 0, before = 0;
    for (int e = 0; e < E; ++e) {
        before = lane == e ? total : before;
        total += MOE_READLANE(cnt, e);
    }
    const int per_group = parts * blocks;
    const long long units = (long long)total * per_group;
    const int u_begin = (int)(units * blockIdx.x / kGrid), u_end = (int)(units * (blockIdx.x + 1) / kGrid);
    if (u_begin >= u_end) return;

    struct Unit {
        int vg, e, row0, n;  // group counted with its repetitions; first sorted row and number of rows
        int part, nb;
        int s0, ns;  // the wave's k-steps
    };
    auto find_group = [&](Unit& u) {
        const unsigned long long at = __ballot(lane < E && cnt > 0 && before <= u.vg);
        u.e = 63 - __clzll((long long)at);
        const int first = (u.vg - MOE_READLANE(before, u.e)) * ROWS;
        u.row0 = MOE_READLANE(lo, u.e) + first;
        u.n = min(ROWS, MOE_READLANE(hi, u.e) - u.row0);
    };
    auto find_steps = [&](Unit& u) {
        const int p0 = uniform_div(steps * u.part, parts), p1 = uniform_div(steps * (u.part + 1), parts);
        u.s0 = p0 + (p1 - p0) * wave / NW;
        u.ns = p0 + (p1 - p0) * (wave + 1) / NW - u.s0;
    };
    auto next = [&](Unit u) {  // (asked for only if there is one)
        if (++u.nb == blocks) {
            u.nb = 0;
            if (++u.part == parts) {
                u.part = 0;
                ++u.vg;
                find_group(u);
            }
            if (F32) find_steps(u);
        }
        return u;
    };

    // ---- the wave's k-steps: step s covers bytes [64 (s0 + s), + 64) of every row.  What lies past the wave's share or the
    // row's end is loaded from the last valid place and counts as zero in both operands; that can be part of the
    // last two steps only.
    struct Rows {
        bf16x8 w[CM][S];
    };
    auto pieces = [&](const Unit& u) { return min(u.ns * 4, K / 8 - u.s0 * 4); };  // valid 16-byte pieces of a row
    // Load i of a chunk: 64 pieces of the 16 rows, row after row (runs of 64 bytes, as MFMA operands lie, are read at
    // 5.0 TB/s, of 128 and more at 6.3; where rows are no multiples of a line, longer runs share fewer lines with other
    // waves': 8 tokens of 2040 / 5624 116.7 us in runs of 256 bytes, 95.3 of 512; the direct-fill kernels' 128: 149.6).
    auto piece = [&](int i, int ln, int& row, int& k) {
        const int at = i * kWave + ln;
        row = at / (4 * S);
        k = at - row * (4 * S);
    };
    auto load = [&](auto chunk, Rows& r, const Unit& u) {
        constexpr int M0 = decltype(chunk)::value * CM;
        const int first = u.nb * 16, rows = min(N - first, 16), last = max(pieces(u) - 1, 0);
        const size_t base = ((size_t)u.e * sg.strideB + (size_t)first * K) * 2 + (size_t)min(u.s0, steps - 1) * 64;
        const int ln = lane_again();
#pragma unroll
        for (int i = 0; i < S; ++i) {
            int row, k;
            piece(i, ln, row, k);
            const unsigned off = (unsigned)min(row, rows - 1) * (unsigned)(K * 2) + (unsigned)min(k, last) * 16;
#pragma unroll
            for (int m = 0; m < CM; ++m)
                r.w[m][i] = __builtin_nontemporal_load(
                    reinterpret_cast<const bf16x8*>(static_cast<const char*>(M0 + m == 0 ? sg.B0 : sg.B1) + base + off));
        }
        __builtin_amdgcn_sched_barrier(0);  // the requests stay ahead of the sums
    };
    bf16x8 x[NX][MT][S];
    auto load_x = [&](const Unit& u) {
        if (g_keys && sg.gather) {  // the group's pairs, in order
            int rank = -u.row0 + MOE_READLANE(lo, u.e);
#pragma unroll
            for (int c = 0; c < kKeyWords; ++c) {
                const unsigned long long same = __ballot(key[c] == u.e);
                const int at = rank + lanes_below(same);
                if (key[c] == u.e && (unsigned)at < (unsigned)ROWS) s_rows[at] = c * kWave + lane;
                rank += __popcll(same);
            }
        }
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const int m = min(mt * 16 + (lane & 15), u.n - 1);
            int row = u.row0 + m;
            if (sg.gather) {
                row = g_keys ? s_rows[m] : g.row_map[row];
                row = quick_div(min(max(row, 0), g.P - 1), g.row_div);
            }
#pragma unroll
            for (int i = 0; i < NX; ++i) {
                const char* a = static_cast<const char*>(i == 0 ? sg.A0 : sg.A1) + (size_t)row * (K * 2);
#pragma unroll
                for (int s = 0; s < S; ++s) {
                    const int k = s * 4 + (lane >> 4), n = pieces(u);
                    x[i][mt][s] = *reinterpret_cast<const bf16x8*>(a + min(u.s0, steps - 1) * 64 + min(k, max(n - 1, 0)) * 16);
                    if (s + 2 >= S && k >= n) x[i][mt][s] = bf16x8{};
                }
            }
        }
    };
    int turn = 0;
    f32x4 acc[NM][MT];
    auto multiply = [&](auto chunk, const Rows& r, const Unit& u) {
        constexpr int M0 = decltype(chunk)::value * CM;
        char* const stage = my_region + (turn & 1) * (NW * REGION);
        const int n = pieces(u), ln = lane_again();
        auto put = [&](auto whole) {
#pragma unroll
            for (int i = 0; i < S; ++i) {
                int row, k;
                piece(i, ln, row, k);
#pragma unroll
                for (int m = 0; m < CM; ++m)
                    *reinterpret_cast<bf16x8*>(stage + (m * 16 + row) * PITCH + k * 16) = decltype(whole)::value || k < n ? r.w[m][i] : bf16x8{};
            }
        };
        if (n >= 4 * S) put(std::true_type{});
        else put(std::false_type{});
        wave_lds_order();
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int m = 0; m < CM; ++m) {
                const bf16x8 w = *reinterpret_cast<const bf16x8*>(stage + (m * 16 + (lane & 15)) * PITCH + s * 64 + (lane >> 4) * 16);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    acc[M0 + m][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, x[DUAL ? M0 + m : 0][mt][s],
                                                                              s == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[M0 + m][mt], 0, 0, 0);
            }
        wave_lds_order();
    };
    auto finish = [&](const Unit& u) {
        char* const buf = smem + (turn & 1) * (NW * REGION);
#pragma unroll
        for (int m = 0; m < NM; ++m)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) *reinterpret_cast<f32x4*>(buf + wave * REGION + ((m * MT + mt) * kWave + lane) * 16) = acc[m][mt];
        __builtin_amdgcn_sched_barrier(0);
        lds_barrier();  // (the other buffer's readers arrive here only when they have read it)
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            if (wave != (turn * MT + mt) % NW) continue;
            f32x4 sum[NM];
#pragma unroll
            for (int m = 0; m < NM; ++m) sum[m] = f32x4{0.f, 0.f, 0.f, 0.f};
            const char* at_w = buf + (mt * kWave + lane) * 16;
#pragma unroll 1  // (all of them at once do not fit the registers beside the weights in flight)
            for (int w0 = 0; w0 < NW; w0 += 4, at_w += 4 * REGION) {
                f32x4 t[NM][4];
#pragma unroll
                for (int m = 0; m < NM; ++m)
#pragma unroll
                    for (int w = 0; w < 4; ++w) t[m][w] = *reinterpret_cast<const f32x4*>(at_w + w * REGION + m * (MT * kWave * 16));
#pragma unroll
                for (int m = 0; m < NM; ++m)
#pragma unroll
                    for (int w = 0; w < 4; ++w) sum[m] += t[m][w];
            }
            const int row = mt * 16 + (lane & 15), col = u.nb * 16 + (lane >> 4) * 4;
            if (row < u.n && col < N) {
                const size_t at = (size_t)(u.row0 + row) * N + col;
                if constexpr (F32) {
                    *reinterpret_cast<f32x4*>(static_cast<float*>(g.parts) + (size_t)u.part * ((size_t)g.P * N) + at) = sum[0];
                } else {
                    bf16x4 o, o1;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        o[j] = (bf16_t)(SWIGLU ? silu_f32(sum[0][j]) * sum[NM - 1][j] : sum[0][j]);
                        o1[j] = (bf16_t)sum[NM - 1][j];
                    }
                    *reinterpret_cast<bf16x4*>(static_cast<bf16_t*>(g.C) + at) = o;
                    if constexpr (PAIR && !SWIGLU) *reinterpret_cast<bf16x4*>(static_cast<bf16_t*>(g.C1) + at) = o1;
                }
            }
        }
        ++turn;
    };

    // (no load is conditional inside the loop, and a change of activations waits for them on the spot: what
    // the compiler cannot count it waits for as a whole)
    Rows r0, r1;
    Unit u0, u1;
    u0.vg = uniform_div(u_begin, per_group);
    u0.part = uniform_div(u_begin - u0.vg * per_group, blocks);
    u0.nb = u_begin - u0.vg * per_group - u0.part * blocks;
    find_group(u0);
    find_steps(u0);
    const std::integral_constant<int, 0> c0{};
    const std::integral_constant<int, 1> c1{};
    load(c0, r0, u0);
    load_x(u0);
    auto change_x = [&](const Unit& from, const Unit& to) {
        if (to.vg == from.vg && to.part == from.part) return;
        load_x(to);
        wait_loads();
    };
    if constexpr (CHUNKS == 1) {
        for (int left = u_end - u_begin;;) {
            if (--left == 0) {
                multiply(c0, r0, u0);
                finish(u0);
                break;
            }
            u1 = next(u0);
            load(c0, r1, u1);
            multiply(c0, r0, u0);
            finish(u0);
            change_x(u0, u1);
            if (--left == 0) {
                multiply(c0, r1, u1);
                finish(u1);
                break;
            }
            u0 = next(u1);
            load(c0, r0, u0);
            multiply(c0, r1, u1);
            finish(u1);
            change_x(u1, u0);
        }
    } else {
        for (int left = u_end - u_begin;;) {
            load(c1, r1, u0);
            multiply(c0, r0, u0);
            if (--left == 0) break;
            u1 = next(u0);
            load(c0, r0, u1);
            multiply(c1, r1, u0);
            finish(u0);
            change_x(u0, u1);
            u0 = u1;
        }
        multiply(c1, r1, u0);
        finish(u0);
    }
}

// two activation operands: their registers beside the weights in flight
constexpr bool dual_fits(int mt, int s) { return mt == 1 || s <= 6; }

template <int MT, int S, bool PAIR, bool SWIGLU, bool DUAL, bool F32>
int launch_few(const GemmArgs& g, hipStream_t st) {
    constexpr size_t lds = 2 * kWaves * region_bytes<MT, S, PAIR>() + kWaves * 16 * MT * 4;
    static_assert(lds <= 160 * 1024, "LDS of a CU");
    static std::atomic<uint64_t> lds_allowed;
    const auto kern = gemm_few_kernel<MT, S, PAIR, SWIGLU, DUAL, F32>;
    if (lds > 64 * 1024 && allow_dynamic_lds(reinterpret_cast<const void*>(kern), lds, lds_allowed) != MOE_OK) return MOE_ERR_LAUNCH;
    hipLaunchKernelGGL(kern, dim3(kGrid), dim3(kWaves * kWave), lds, st, as_arg(g.keys), as_arg(g.offsets), g.P, g.E, g);
    return launch_status();
}
template <int MT, int S>
int launch_few(const GemmArgs& g, bool swiglu, hipStream_t st) {
    if (swiglu && g.seg[0].A0 != g.seg[0].A1) {
        if constexpr (dual_fits(MT, S)) return launch_few<MT, S, true, true, true, false>(g, st);
        else return MOE_ERR_UNSUPPORTED;
    }
    if (swiglu) return launch_few<MT, S, true, true, false, false>(g, st);
    if (g.C1) return launch_few<MT, S, true, false, false, false>(g, st);
    return g.k_parts > 1 ? launch_few<MT, S, false, false, false, true>(g, st) : launch_few<MT, S, false, false, false, false>(g, st);
}
template <int MT, int S>
int launch_few(const GemmArgs& g, int s, bool swiglu, hipStream_t st) {
    if constexpr (S > kMaxSteps) {
        return MOE_ERR_UNSUPPORTED;
    } else {
        return s == S ? launch_few<MT, S>(g, swiglu, st) : launch_few<MT, S + 1>(g, s, swiglu, st);
    }
}

int few_steps(int K, int parts) {
    const int steps = (K + kStepK - 1) / kStepK;
    return ((steps + parts - 1) / parts + kWaves - 1) / kWaves;
}

}  // namespace

// Where these kernels are taken: up to 32 rows in a group, two MFMA row blocks (a token meets an expert once, so 32
// tokens).  Whole layer, us, weights cold, direct-fill kernels / these.  Up to 16 tokens these are the faster at every size
// measured: 2048 / 5632 3 tokens 89 / 73, 16 tokens 120 / 102; 1024 / 2816 3, 8 and 16 tokens 31.2 / 27.8, 36.0 / 33.9, 37.5 / 35.5;
// 432 / 1152 16 tokens 25.3 / 21.1.  From 17 on they are so for narrow layers, few experts, cut lines, rank factors and a shared base (32
// tokens: 432 / 1152 24.7 / 21.7, 768 / 2048 30.4 / 28.0, 4 experts of 1024 / 2816 30.5 / 27.5, 2040 / 5624 107.9 / 103.3, rank 1024 on 2048 / 5632
// 93.9 / 86.8, shared base with rank 64 95.6 / 79.6) and about even for 8 experts of whole lines: 1024 / 2816 38.2 / 38.8 (4 chosen 40.5 /
// 41.7, the worst found), 1280 / 3456 48.6 / 49.0, 1792 / 4864 81.4 / 82.0; 2048 / 5632 takes 99-122 there by where its matrices lie, here
// 102-105.  With four row blocks the activations do not fit the registers: 64 tokens 111 / 247.
bool gemm_few_rows(long long P, int top_k) { return P <= kKeyWords * kWave && P <= 32ll * top_k; }

// What the kernels demand of a product's sizes, its K in `parts` parts: the plan of a call and the choice of a kernel ask the same
static bool few_sizes_supported(long long P, int N, int K, int parts) {
    return P <= kKeyWords * kWave && few_steps(K, parts) <= kMaxSteps && K >= 8 && K % 8 == 0 && K < (1 << 23) &&
           (long long)N * K * 2 < (1ll << 32);
}

int gemm_few_split(long long P, int N, int K, int parts_min, int parts_max) {
    int q = parts_min;
    while (q <= parts_max && !few_sizes_supported(P, N, K, q)) ++q;
    return q <= parts_max ? q : 0;
}

bool gemm_few_supported(const GemmArgs& g) {
    const GemmSeg& sg = g.seg[0];
    const int parts = g.k_parts > 1 ? g.k_parts : 1;
    const bool dual = sg.A0 != sg.A1;
    return g.nseg == 1 && !g.add0 && g.few > 0 && few_sizes_supported(g.P, g.N, sg.K, parts) && (parts == 1 || g.parts_f32) &&
           !(dual && (g.C1 || !dual_fits(g.few <= 16 ? 1 : 2, few_steps(sg.K, parts))));
}

int run_gemm_few(const GemmArgs& g, bool swiglu, hipStream_t st) {
    const int s = few_steps(g.seg[0].K, g.k_parts > 1 ? g.k_parts : 1);
    return g.few <= 16 ? launch_few<1, 1>(g, s, swiglu, st) : launch_few<2, 1>(g, s, swiglu, st);
}

}  // namespace moe
