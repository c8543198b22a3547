// Grouped bf16 GEMM for products with enough rows per expert to be bound by the matrix cores (gemm.h
// states the problem): 256-row tiles on eight waves, operands fetched from memory straight into LDS.
//
// What bounds it.  A 256 x 256 x 64 k-step is 2048 clocks of MFMA per SIMD; beside them go 64 KB of fills
// (L1 takes about 64 B per clock: 1024 clocks) and 192 KB of fragment reads (128 B per clock: 1536).  All
// three have to overlap.  A wave issues in order, so whatever it issues before an MFMA and has to queue
// for holds the MFMA back: with a k-step's eight fill instructions per wave issued together, fills and
// MFMAs added up (3600 clocks per step, MFMAs alone 2260, fills alone 2020-3360).  Here
//   - the eight waves form two groups, one wave of each per SIMD, half a step apart: in every phase one
//     group multiplies out of registers while the other reads the fragments of its whole next step;
//   - fills go only between MFMAs, one per four 16-clock MFMAs or more, B by group 0 and A by group 1, and
//     nothing in the loop branches (a scalar branch around each fill: 3600 clocks again);
//   - B, the weights, has three k-steps in LDS and A two (160 KB): weights come from HBM.
// 2320-2760 clocks per step, and then the board's power limit sets the clock (1.6-1.9 GHz from 2.2), so
// what counts next is energy: 16 x 16 x 32 MFMAs move half the accumulator bytes of 32 x 32 x 16 ones and
// run 5 % faster at the same schedule.
// Measured on the 2048 / 5632 layer, Zipf loads (us; the register-staged kernel before / this one):
// gate/up 222 / 189 and down 115 / 99 at 2048 tokens; 1410 / 1180 and 720 / 601 at 16384 tokens
// (1.28 PFLOP/s).
#include "gemm.h"

namespace moe {

namespace {

#define INLINE __attribute__((always_inline))

constexpr int BM = 256, BK = 64;
constexpr int kThreads = 512;

typedef __attribute__((address_space(3))) char lds_char;

// 64 lanes x 16 bytes from memory straight to 1 KB of LDS at byte address lds (wave-uniform).  The compiler
// does not see these loads: they are waited for by hand (wait_vm), and what it inserts for loads of
// its own can only wait longer.
__device__ __forceinline__ void dma16(unsigned lds, const char* base, unsigned off) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(off), "s"(base)
                 : "memory");
#endif
}
// at most N of the wave's memory loads are still in flight afterwards (they complete in order)
template <int N>
__device__ __forceinline__ void wait_vm() {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
#endif
}
// The lane index, counted anew: what is derived from it is computed where it is used and not kept in
// registers through the main loop.
__device__ __forceinline__ int lane_again() {
#if defined(__HIP_DEVICE_COMPILE__)
    int v = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    asm volatile("" : "+v"(v));
    return v;
#else
    return 0;
#endif
}
__device__ __forceinline__ void phase_end() {
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
#endif
}

// BN: rows of the B tile.  SWIGLU: its first half are gate rows, the second half the matching up rows.
// DUAL (SwiGLU with two activation operands, the rank products of a weight-decomposed expert): the tile
// is BN gate rows for the first K / 64 steps, over A0, and the matching BN up rows for as many more, over A1,
// into two sets of accumulators.
template <int BN, int WAVES_M, bool SWIGLU, bool DUAL>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_pp_kernel(const GemmArgs g) {
    static_assert(!DUAL || SWIGLU, "two activation operands only with the activation");
    constexpr int WAVES_N = 8 / WAVES_M;
    constexpr int MB = BM / 32 / WAVES_M;         // 32-row blocks of a wave
    constexpr int WN = BN / WAVES_N, NI = WN / 16;  // columns, 16-column blocks of a wave
    constexpr int NP = DUAL ? 2 : 1;
    constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2;
    constexpr int SA = 2, SB = 3;                 // k-steps of A and of B in LDS
    constexpr int PA = BM / 32, PB = BN / 32;     // fill instructions per k-step of a wave of group 1 / 0
    constexpr bool SPLIT_B = SWIGLU && !DUAL;     // the B tile is half gate rows, half up rows
    constexpr int BN_OUT = SPLIT_B ? BN / 2 : BN;
    extern __shared__ __align__(16) char smem[];

    int e, row0, row_end, nt;
    if (!find_tile(g.offsets, g.E, g.P, BM, g.n_tiles, e, row0, row_end, nt, g.n_inner, g.split_slots)) return;
    // two plain products in one launch: the upper half of the n-tiles belongs to (A1, B1, C1)
    const bool second = !SWIGLU && g.C1 != nullptr && nt >= g.n_tiles / 2;
    if (second) nt -= g.n_tiles / 2;
    // k-parts ride on the n-tile index: n-tiles [q * n_base, (q + 1) * n_base) are part q
    int part = 0;
    if (!SWIGLU && g.k_parts > 1) {
        const int n_base = g.n_tiles / g.k_parts;
        part = nt / n_base;
        nt -= part * n_base;
    }
    const int n0 = nt * BN_OUT;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int grp = wave >> 2;                    // waves i and i + 4 share a SIMD
    const int wm = wave / WAVES_N, wn = wave % WAVES_N;

    const GemmSeg& sg = g.seg[0];
    const int K = sg.K;
    const char* A0 = static_cast<const char*>(second ? sg.A1 : sg.A0);
    const char* A1 = DUAL ? static_cast<const char*>(sg.A1) : A0;
    const char* B0 = static_cast<const char*>(second ? sg.B1 : sg.B0) + (size_t)e * sg.strideB * 2;
    const char* B1 = SWIGLU ? static_cast<const char*>(sg.B1) + (size_t)e * sg.strideB * 2 : B0;
    int nk = (K + BK - 1) / BK, k_begin = 0;
    if (!SWIGLU && g.k_parts > 1) {
        const int s0 = nk * part / g.k_parts, s1 = nk * (part + 1) / g.k_parts;
        k_begin = s0;
        nk = s1 - s0;
    }
    const int nv = NP * nk;                       // k-steps over all passes
    // A partial last k-step is fetched as the operands' last 64 columns, in bounds; the chunks that it
    // shares with the step before are cleared in the A fragments.
    const int tail_back = max(0, (k_begin + nk) * BK - K) * 2;

    // ---- fills: instruction p of wave w fetches rows (4 p + w % 4) * 8 .. + 8 of its operand's tile; lane l the
    // 16-byte slot l % 8 of row l / 8, which holds chunk slot ^ ((row / 2) % 8) (free of bank conflicts
    // for the fragment reads).  Byte offsets from wave-uniform bases; rows past the group's or the
    // matrix's end are the last one again, so that no fill is conditional.
    const int fw = wave & 3;
    const int f_row = fw * 8 + (lane >> 3);
    const int f_chunk = (lane & 7) ^ (((wave & 1) << 2) | (lane >> 4));
    const int rows_here = row_end - row0;
    unsigned off[PA > PB ? PA : PB];
    if (grp == 1) {
        int arow[PA];
#pragma unroll
        for (int p = 0; p < PA; ++p) arow[p] = min(row0 + f_row + 32 * p, row_end - 1);
        if (sg.gather) {
#pragma unroll
            for (int p = 0; p < PA; ++p) arow[p] = g.row_map[arow[p]];
#pragma unroll
            for (int p = 0; p < PA; ++p) arow[p] = min(max(arow[p], 0), g.P - 1) / g.row_div;
        }
#pragma unroll
        for (int p = 0; p < PA; ++p) off[p] = __umul24(arow[p], K * 2) + f_chunk * 16;
    } else {
#pragma unroll
        for (int p = 0; p < PB; ++p) {
            const int j = f_row + 32 * p;
            off[p] = __umul24(min(SPLIT_B ? n0 + j % (BN / 2) : n0 + j, g.N - 1), K * 2) + f_chunk * 16;
        }
    }
    // what this wave fetches: instructions below PH from src_lo, the others from src_hi; in the second
    // pass (DUAL) all from src_2
    constexpr int PH = SPLIT_B ? PB / 2 : PB;
    const size_t k_off = (size_t)k_begin * (BK * 2);
    const char* const src_lo = (grp == 1 ? A0 : B0) + k_off;
    const char* const src_hi = (grp == 1 ? A0 : SPLIT_B ? B1 : B0) + k_off;
    const char* const src_2 = grp == 1 ? A1 : B1;
    const unsigned lds0 = (unsigned)(uintptr_t)(lds_char*)smem + fw * 1024;
    auto fill = [&](int v, int p) INLINE {
        const unsigned slot = grp == 1 ? v % SA * A_BYTES : SA * A_BYTES + v % SB * B_BYTES;
        const int t = DUAL && v >= nk ? v - nk : v;
        const char* src = DUAL && v >= nk ? src_2 : p < PH ? src_lo : src_hi;
        src += t * (BK * 2) - (t == nk - 1 ? tail_back : 0);
        dma16(lds0 + slot + p * 4096, src, off[p]);
    };
    auto fill_all = [&](int v) INLINE {
#pragma unroll
        for (int p = 0; p < (PA > PB ? PA : PB); ++p)
            if (p < (grp == 1 ? PA : PB)) fill(v, p);
    };

    f32x4 acc[NP][2 * MB][NI];
#pragma unroll
    for (int s = 0; s < NP; ++s)
#pragma unroll
        for (int mi = 0; mi < 2 * MB; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) acc[s][mi][ni] = f32x4{0.f, 0.f, 0.f, 0.f};

    // A wave's 32-row blocks are wm, wm + WAVES_M, ... of the tile's eight: those that hold rows of the group
    // are spread over the waves.
    const int live = min(MB, max(0, ((rows_here + 31) / 32 + WAVES_M - 1 - wm) / WAVES_M));
    // fragment reads: row lane % 16 of a 16-row block, chunk 4 ks + lane / 16
    const unsigned c16 = ((lane >> 4) ^ ((lane & 15) >> 1)) << 4;
    const unsigned ra = wm * 4096 + (lane & 15) * 128 + c16;
    const unsigned rb = SA * A_BYTES + wn * (SPLIT_B ? WN / 2 : WN) * 128 + (lane & 15) * 128 + c16;

    // Phases: group 0 reads step v's fragments in phase 2 v and multiplies in phase 2 v + 1, group 1 a phase
    // later.  The LDS slots of step v are free from the end of phase 2 v + 1 on.  A of step v + 2 is fetched in
    // phase 2 v + 2 by group 1, B of step v + 2 in phase 2 v + 1 by group 0; both have to have landed when
    // phase 2 v + 4 begins.
    fill_all(0);
    if (nv > 1 && grp == 0) {
        fill_all(1);
        wait_vm<PB>();
    } else {
        wait_vm<0>();
    }
    phase_end();
    if (grp == 1) {
        if (nv > 1) fill_all(1);
        phase_end();
    }
    // gc: the group, known at compile time where the groups' fills differ in number (a fill must not be
    // conditional inside the loop)
    auto k_loop = [&](auto ma, auto pass, auto gc) INLINE {
        constexpr int MA = decltype(ma)::value;  // the wave's row blocks that hold rows of the group
        constexpr int S = decltype(pass)::value, MR = MA > 0 ? MA : 1;
        bf16x8 fa[2][2 * MR], fb[2][NI];
        auto read = [&](int v) INLINE {
            const char* pa = smem + v % SA * A_BYTES;
            const char* pb = smem + v % SB * B_BYTES;
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                const char* a = pa + (ra ^ (ks << 6));
                const char* b = pb + (rb ^ (ks << 6));
#pragma unroll
                for (int ni = 0; ni < NI; ++ni)  // SPLIT_B: NI / 2 gate blocks, then as many up blocks
                    fb[ks][ni] = *reinterpret_cast<const bf16x8*>(
                        b + (SPLIT_B ? ni / (NI / 2) * (B_BYTES / 2) + ni % (NI / 2) * 2048 : ni * 2048));
#pragma unroll
                for (int mi = 0; mi < 2 * MA; ++mi)
                    fa[ks][mi] = *reinterpret_cast<const bf16x8*>(a + (mi >> 1) * (WAVES_M * 4096) + (mi & 1) * 2048);
            }
        };
        auto clear_shared = [&]() INLINE {
            const int ln = lane_again();
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
                if ((ks * 4 + (ln >> 4)) * 16 < tail_back) {
#pragma unroll
                    for (int mi = 0; mi < 2 * MA; ++mi) fa[ks][mi] = bf16x8{};
                }
        };
        // the MFMAs of a step (the weights are the first operand: a lane's four results are neighbouring
        // columns of one row) with the fills of another between them
        auto multiply = [&](auto filling, int vf) INLINE {
            constexpr int NF = decltype(gc)::value == 1 ? PA : PB;
            constexpr int NM = MA * 4 * NI, GAP = NM / NF > 0 ? NM / NF : 1;
            int p = 0;
#pragma unroll
            for (int i = 0; i < NM; ++i) {
                const int ni = i % NI, mi = i / NI % (2 * MR), ks = i / (NI * 2 * MR);
                acc[S][mi][ni] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[ks][ni], fa[ks][mi], acc[S][mi][ni], 0, 0, 0);
                if (decltype(filling)::value && i % GAP == GAP - 1 && p < NF) {
                    __builtin_amdgcn_sched_barrier(0);
                    fill(vf, p);
                    ++p;
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            if (decltype(filling)::value) {
#pragma unroll
                for (; p < NF; ++p) fill(vf, p);
            }
        };
        int v = S * nk;
        const int v_end = v + nk;
        for (; v < v_end && v + 2 < nv; ++v) {
            if (MA > 0) read(v);
            if (DUAL && S == 0 && v == v_end - 1 && tail_back > 0) clear_shared();
            if (grp == 1) wait_vm<0>();  // A of step v + 1
            phase_end();
            multiply(std::true_type{}, v + 2);
            if (grp == 0) wait_vm<PB>();  // B of step v + 1
            phase_end();
        }
        for (; v < v_end; ++v) {
            if (MA > 0) read(v);
            if (v == v_end - 1 && tail_back > 0) clear_shared();
            if (grp == 1) wait_vm<0>();
            phase_end();
            multiply(std::false_type{}, 0);
            if (grp == 0) wait_vm<0>();
            phase_end();
        }
    };
    auto loops = [&](auto ma) INLINE {
        typedef std::integral_constant<int, 0> c0;
        typedef std::integral_constant<int, 1> c1;
        auto passes = [&](auto gc) INLINE {
            k_loop(ma, c0{}, gc);
            if constexpr (DUAL) k_loop(ma, c1{}, gc);
        };
        if (PA == PB || grp == 0) passes(c0{});
        else passes(c1{});
    };
    if (live == MB) loops(std::integral_constant<int, MB>{});
    else if (live == 0) loops(std::integral_constant<int, 0>{});
    else if (live == 1) loops(std::integral_constant<int, 1>{});
    else if (live == 2) loops(std::integral_constant<int, (MB > 2 ? 2 : 1)>{});
    else loops(std::integral_constant<int, (MB > 3 ? 3 : 1)>{});
    if (grp == 0) phase_end();

    // ---- epilogue: accumulator element i of a block is output column 4 (lane / 16) + i of row lane % 16.
    // Staged through LDS, 32 rows at a time in a region per wave, so that the tile leaves in 16-byte
    // stores.
    bf16_t* const Ct = static_cast<bf16_t*>(second ? g.C1 : g.C) + (size_t)part * g.part_stride +
                       (size_t)row0 * g.N + n0;
    const unsigned ldc = (unsigned)g.N;
    constexpr int OC = BN_OUT / WAVES_N;             // output columns of a wave
    constexpr int PITCH = OC * 2 + 16;
    constexpr int LPR = OC / 8, RPI = 64 / LPR;      // lanes per staged row, rows per read instruction
    const int ln = lane_again();
    char* const region = smem + wave * (32 * PITCH);
    char* const wr = region + (ln & 15) * PITCH + (ln >> 4) * 8;
    const int rd_row = ln / LPR, rd_chunk = ln % LPR;
    const int c0 = wn * OC + rd_chunk * 8;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
        if (mb >= live) continue;
        const int rbk = (WAVES_M * mb + wm) * 32;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int nb = 0; nb < OC / 16; ++nb) {
                bf16x4 o;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    float v = acc[0][2 * mb + h][nb][j];
                    if (SWIGLU) v = silu_f32(v) * (DUAL ? acc[NP - 1][2 * mb + h][nb][j] : acc[0][2 * mb + h][(nb + NI / 2) % NI][j]);
                    o[j] = (bf16_t)v;
                }
                *reinterpret_cast<bf16x4*>(wr + h * 16 * PITCH + nb * 32) = o;
            }
#pragma unroll
        for (int it = 0; it < 32 / RPI; ++it) {
            const int r = it * RPI + rd_row;
            const uint4 v = *reinterpret_cast<const uint4*>(region + r * PITCH + rd_chunk * 16);
            if (rbk + r < rows_here && n0 + c0 < g.N)
                *reinterpret_cast<uint4*>(Ct + (unsigned)(rbk + r) * ldc + (unsigned)c0) = v;
        }
    }
}

template <int BN, int WAVES_M, bool SWIGLU, bool DUAL>
int launch_pp(GemmArgs& g, hipStream_t st) {
    constexpr int BN_OUT = SWIGLU && !DUAL ? BN / 2 : BN;
    g.m_tiles_max = g.P / BM + g.E;
    g.n_tiles = (g.N + BN_OUT - 1) / BN_OUT * ((!SWIGLU && g.C1) ? 2 : 1) * (g.k_parts > 1 ? g.k_parts : 1);
    constexpr size_t lds = (2 * BM + 3 * BN) * BK * 2;
    g.split_slots = 32;  // one workgroup per CU
    const int grid = ((g.m_tiles_max * g.n_tiles + 7) / 8 + g.split_slots / 2) * 8;
    static std::atomic<uint64_t> lds_allowed;
    const auto kern = gemm_pp_kernel<BN, WAVES_M, SWIGLU, DUAL>;
    if (allow_dynamic_lds(reinterpret_cast<const void*>(kern), lds, lds_allowed) != MOE_OK) return MOE_ERR_LAUNCH;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(kThreads), lds, st, g);
    return launch_status();
}

}  // namespace

// One segment, no addends, operands whose rows are reached by 32-bit byte offsets (rows below 2^24 and
// row lengths below 2^23 by the 24-bit multiply), at least one whole k-step.
bool gemm_pp_supported(const GemmArgs& g) {
    const GemmSeg& sg = g.seg[0];
    if (g.nseg != 1 || g.add0 || sg.K < BK || sg.K >= (1 << 23) || g.N >= (1 << 24)) return false;
    const long long a_rows = sg.gather ? (g.P - 1) / (g.row_div > 0 ? g.row_div : 1) + 1 : g.P;
    return a_rows * sg.K * 2 < (1ll << 32) && (long long)g.N * sg.K * 2 < (1ll << 32);
}

int run_gemm_pp(GemmArgs& g, bool swiglu, hipStream_t st) {
    if (!swiglu) return launch_pp<256, 2, false, false>(g, st);
    if (g.seg[0].A0 != g.seg[0].A1) return launch_pp<128, 4, true, true>(g, st);
    // blocks of four n-tiles with the expert's m-tiles inside: the 32 tiles in flight on an XCD then share
    // eight A and four B tiles in its L2 instead of all m-tiles of one or two n-tiles (gate/up at 16384
    // tokens 1180 us from 1210; no difference at 2048, where an expert has up to seven m-tiles)
    g.n_inner = 4;
    return launch_pp<256, 2, true, false>(g, st);
}

}  // namespace moe
