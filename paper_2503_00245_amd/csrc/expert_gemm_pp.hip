// Grouped bf16 GEMM of one K-segment without addends (gemm.h states the problem): 256-, 128- or 64-row tiles on
// eight waves, operands fetched from memory straight into LDS.
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
// 2490 clocks per step (what 16 more steps per tile add at 16384 tokens; 16 K clocks per round of tiles beside
// it), and then the board's power limit sets the clock (1.8 GHz there, from 2.2), so what counts next is
// energy: 16 x 16 x 32 MFMAs move half the accumulator bytes of 32 x 32 x 16 ones and run 5 % faster at the
// same schedule.
// Measured on the 2048 / 5632 layer, Zipf loads (us; the register-staged kernel before / this one):
// gate/up 222 / 189 and down 115 / 99 at 2048 tokens; 1410 / 1180 and 720 / 601 at 16384 tokens
// (1.28 PFLOP/s).
#include "gemm.h"

#include <array>
#include <cmath>

namespace moe {

namespace {

#define INLINE __attribute__((always_inline))

constexpr int BK = 64;
constexpr int kThreads = kPpThreads;
constexpr int kSplitSlots = 32;  // one workgroup per CU

typedef __attribute__((address_space(3))) char lds_char;

// 64 lanes x 16 bytes from memory straight to 1 KB of LDS at byte address lds (wave-uniform).  The compiler
// does not see these loads: they are waited for by hand (wait_vm), and what it inserts for loads of
// its own can only wait longer.  NT: the data is used once, here; it need not stay in the caches.  (m0 is
// reserved to the compiler, which sets it right before an instruction of its own that reads it and accepts no
// clobber of it; these kernels have no such instruction: every m0 in their assembly is one of these moves.)
template <bool NT>
__device__ __forceinline__ void dma16(unsigned lds, const char* base, unsigned off) {
#if defined(__HIP_DEVICE_COMPILE__)
    if (NT)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(lds), "v"(off), "s"(base)
                     : "memory");
    else
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
// The wave's LDS reads have landed, and all waves have come here.  (The wait is the compiler's own instruction: one that it does not see it
// makes again, fragment by fragment between a phase's MFMAs, eight for 64: 16384 tokens of 2048 / 5632 1809 us with these, 1786 without, 2048 tokens
// 305.8 and 302.7, of rank 1024 263.0 and 261.6.)
__device__ __forceinline__ void phase_end() {
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0) alone
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
#endif
}

// The arguments beyond those that arrive in registers, all of them at this place: their loads, from memory that no cache holds yet, are
// then one latency, under that of the keys or bounds, where the compiler left one before every stage of a tile's way to its first fill.
__device__ __forceinline__ void arguments_here(const GemmArgs& g) {
#if defined(__HIP_DEVICE_COMPILE__)
    const GemmSeg& s = g.seg[0];
    asm volatile("" ::"s"(s.A0), "s"(s.A1), "s"(s.B0), "s"(s.B1), "s"(s.strideB), "s"(s.K), "s"(s.gather), "s"(g.C), "s"(g.C1), "s"(g.N), "s"(g.offsets),
                 "s"(g.row_map), "s"(g.row_div), "s"(g.hidden_a), "s"(g.k_parts), "s"(g.parts), "s"(g.fit_width), "s"(g.inv_perm));
#endif
}

// BN: rows of the B tile.  SWIGLU: its first half are gate rows, the second half the matching up rows.
// DUAL (SwiGLU with two activation operands, the rank products of a weight-decomposed expert): the tile
// is BN gate rows for the first K / 64 steps, over A0, and the matching BN up rows for as many more, over A1,
// into two sets of accumulators.
// SA, SB: k-steps of A and of B in LDS.
// F32: k-parts stored in fp32.
// NT_B: weights past the caches (run_gemm_pp has the rule).
// LINES: rows of B that are no multiples of a cache line are fetched in whole lines all the same.  Line t of a row, counted
// from the line that the row begins in, goes to slot t % SB; row r begins shift(r) 16-byte chunks into its line 0, so
// step t is read from lines t and t + 1, and a line more than there are k-steps is fetched.
template <int BM, int BN, int WAVES_M, int SA, int SB, bool SWIGLU, bool DUAL, bool F32, bool NT_B, bool LINES>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_pp_kernel(
    ptr_arg a_keys, ptr_arg a_offsets, int g_P, int g_E, const GemmArgs g) {
    const int32_t *const g_keys = from_arg<const int32_t>(a_keys), *const g_offsets = from_arg<const int32_t>(a_offsets);
    static_assert(!DUAL || SWIGLU, "two activation operands only with the activation");
    constexpr int WAVES_N = 8 / WAVES_M;
    constexpr int MB = BM / 32 / WAVES_M;         // 32-row blocks of a wave
    static_assert(!LINES || (!DUAL && SB >= 4), "a step lies in two lines");
    static_assert(MB >= 1 && SA >= 2 && SB >= 3, "a group reads one step while the other's is being fetched");
    constexpr int WN = BN / WAVES_N, NI = WN / 16;  // columns, 16-column blocks of a wave
    static_assert(NI % 2 == 0 || !SWIGLU || DUAL, "whole blocks of gate and of up columns");
    constexpr int NP = DUAL ? 2 : 1;
    constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2;
    constexpr int PA = BM / 32, PB = BN / 32;     // fill instructions per k-step of a wave of group 1 / 0
    constexpr bool SPLIT_B = SWIGLU && !DUAL;     // the B tile is half gate rows, half up rows
    constexpr int BN_OUT = SPLIT_B ? BN / 2 : BN;
    extern __shared__ __align__(16) char smem[];

    int e, row0, row_end, nt;
    // Output columns of a tile and tiles across N.  fit_width: the m-tiles are known only here; where the
    // launch is a few rounds of 256 workgroups, tiles are made narrower until the last round is full.
    int width = BN_OUT, n_base = (g.N + BN_OUT - 1) / BN_OUT;
    const int copies = SWIGLU ? 1 : g.C1 ? 2 : max(g.k_parts, 1);  // products, or k-parts, of the launch
    auto n_tiles_of = [&](int m_tiles) INLINE {
        if (m_tiles > 0) fit_columns(m_tiles * copies, g.N, g.fit_width, width, n_base);
        return n_base * copies;
    };
    // (in the last slot of B, which is first filled after the first phase)
    int (*const s_count)[kMaxExperts] = reinterpret_cast<int (*)[kMaxExperts]>(smem + SA * A_BYTES + (SB - 1) * B_BYTES);
    int* const s_pair = &s_count[kThreads / kWave][0];
    static_assert((kThreads / kWave * kMaxExperts + BM + kWave) * 4 <= B_BYTES, "dispatch scratch");
    int lo, hi;
    PairKeys<kThreads> keys;
    if (g_keys) {
        keys.load(g_keys, g_P);
        arguments_here(g);
        keys.bounds(g_E, s_count, lo, hi);
        const int lane_ = threadIdx.x & 63;
        if (blockIdx.x == 0 && threadIdx.x < 64) {
            if (lane_ < g.E) g.offsets[lane_] = lo;
            if (lane_ == g.E - 1) g.offsets[g.E] = hi;
        }
    } else {
        group_bounds(g_offsets, g_E, g_P, lo, hi);
        arguments_here(g);
    }
    // SwiGLU products of 256-row tiles: blocks of four n-tiles with the expert's m-tiles inside, so that the 32
    // tiles in flight on an XCD share eight A and four B tiles in its L2 instead of all m-tiles of one
    // or two n-tiles (gate/up at 16384 tokens 1180 us from 1210; no difference at 2048, where an expert
    // has up to seven m-tiles)
    constexpr int INNER = SWIGLU && !DUAL && BM == 256 ? 4 : 1;
    if (!(g.hidden_a ? find_tile<kHiddenOperandBlock, kSplitSlots>(lo, hi, g.E, BM, n_tiles_of, e, row0, row_end, nt)
                     : find_tile<INNER, kSplitSlots>(lo, hi, g.E, BM, n_tiles_of, e, row0, row_end, nt)))
        return;
    // the copies ride on the n-tile index: n-tiles [q n_base, (q + 1) n_base) are part q, or of two plain
    // products in one launch (A0, B0, C) and (A1, B1, C1)
    const int copy = !SWIGLU && copies > 1 ? uniform_div(nt, n_base) : 0;
    nt -= copy * n_base;
    const bool second = !SWIGLU && g.C1 != nullptr && copy == 1;
    const int part = second ? 0 : copy;
    const int n0 = nt * width;
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
        const int s0 = uniform_div(nk * part, g.k_parts), s1 = uniform_div(nk * (part + 1), g.k_parts);
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
    // LINES: slot (m + row / 2 - shift) % 8 holds chunk m of the line, so that a fragment read finds chunk c of a step in
    // slot (c + row / 2) % 8 of either line.  Tiles begin at multiples of 8 rows, of which all bytes are whole lines: the
    // shift is a row's within the tile.
    const int shift_f = f_row * (K >> 3) & 7;
    const int rows_here = row_end - row0;
    unsigned off[PA > PB ? PA : PB];
    if (grp == 0) {
#pragma unroll
        for (int p = 0; p < PB; ++p) {
            const int j = f_row + 32 * p;
            if constexpr (LINES) {  // (a row past the end is one of the last eight, of the same shift; + 128: fill takes it back)
                const int r = SPLIT_B ? j % (BN / 2) : j, end = min(width, g.N - n0);
                off[p] = (__umul24(n0 + (r < end ? r : end - 8 + (r & 7)), K * 2) & ~127u) + 128 + ((lane - (f_row >> 1) + shift_f) & 7) * 16;
            } else {
                off[p] = __umul24(min(n0 + min(SPLIT_B ? j % (BN / 2) : j, width - 1), g.N - 1), K * 2) + f_chunk * 16;
            }
        }
    }
    // what this wave fetches: instructions below PH from src_lo, the others from src_hi; in the second
    // pass (DUAL) all from src_2
    constexpr int PH = SPLIT_B ? PB / 2 : PB;
    const size_t k_off = (size_t)k_begin * (BK * 2);
    const size_t b_off = LINES ? k_off - 128 : k_off;  // (the offsets are unsigned, and one may be a line less)
    const char* const src_lo = grp == 1 ? A0 + k_off : B0 + b_off;
    const char* const src_hi = grp == 1 ? A0 + k_off : (SPLIT_B ? B1 : B0) + b_off;
    const char* const src_2 = grp == 1 ? A1 : B1;
    const unsigned lds0 = (unsigned)(uintptr_t)(lds_char*)smem + fw * 1024;
    auto fill = [&](auto gc, int v, int p) INLINE {
        constexpr int GRP = decltype(gc)::value;
        const unsigned slot = GRP == 1 ? v % SA * A_BYTES : SA * A_BYTES + v % SB * B_BYTES;
        const int t = DUAL && v >= nk ? v - nk : v;
        const char* src = DUAL && v >= nk ? src_2 : p < PH ? src_lo : src_hi;
        if constexpr (LINES && GRP == 0) {
            // (the last line, where the row ends before it: the one before again)
            const unsigned back = t == nk && shift_f * 16 <= tail_back ? 128 : 0;
            dma16<NT_B>(lds0 + slot + p * 4096, src + t * (BK * 2), off[p] - back);
            return;
        }
        src += t * (BK * 2) - (t == nk - 1 ? tail_back : 0);
        dma16<GRP == 0 && NT_B>(lds0 + slot + p * 4096, src, off[p]);
    };
    if (grp == 0) {  // the first steps of B, before the rows of A are known
#pragma unroll
        for (int q = 0; q < SB - 1; ++q)
            if (q < nv + LINES) {
#pragma unroll
                for (int p = 0; p < PB; ++p) fill(std::integral_constant<int, 0>{}, q, p);
            }
    }
    if (g_keys) {
        const int rows = min(rows_here, BM);
        keys.rows(e, row0 - MOE_READLANE(lo, e), rows, BM, s_count, s_pair);
        if (nt == 0 && copy == 0) {  // one column tile of each row tile writes the sorted order
            for (int r = threadIdx.x; r < rows; r += kThreads) {
                const int p = s_pair[r];
                g.row_map[row0 + r] = p;
                g.inv_perm[p] = row0 + r;
            }
        }
    }
    if (grp == 1) {
        int arow[PA];
#pragma unroll
        for (int p = 0; p < PA; ++p) arow[p] = min(row0 + f_row + 32 * p, row_end - 1);
        if (sg.gather) {
#pragma unroll
            for (int p = 0; p < PA; ++p) arow[p] = g_keys ? s_pair[arow[p] - row0] : g.row_map[arow[p]];
#pragma unroll
            for (int p = 0; p < PA; ++p) arow[p] = quick_div(min(max(arow[p], 0), g.P - 1), g.row_div);
        }
#pragma unroll
        for (int p = 0; p < PA; ++p) off[p] = __umul24(arow[p], K * 2) + f_chunk * 16;
    }
    f32x4 acc[NP][2 * MB][NI];
#pragma unroll
    for (int s = 0; s < NP; ++s)
#pragma unroll
        for (int mi = 0; mi < 2 * MB; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) acc[s][mi][ni] = f32x4{0.f, 0.f, 0.f, 0.f};

    // A wave's 32-row blocks are wm, wm + WAVES_M, ... of the tile's eight: those that hold rows of the group
    // are spread over the waves.
    const int live = wn * (BN_OUT / WAVES_N) >= width ? -1 : min(MB, max(0, ((rows_here + 31) / 32 + WAVES_M - 1 - wm) / WAVES_M));
    // fragment reads: row lane % 16 of a 16-row block, chunk 4 ks + lane / 16
    const unsigned c16 = ((lane >> 4) ^ ((lane & 15) >> 1)) << 4;
    const unsigned ra = wm * 4096 + (lane & 15) * 128 + c16;
    const unsigned c16_b = LINES ? (((lane >> 4) + ((lane & 15) >> 1)) & 7) << 4 : c16;
    const unsigned rb0 = SA * A_BYTES + wn * (SPLIT_B ? WN / 2 : WN) * 128 + (lane & 15) * 128, rb = rb0 + c16_b;

    // Phases: group 0 reads step v's fragments in phase 2 v and multiplies in phase 2 v + 1, group 1 a phase
    // later.  The LDS slots of step v are free from the end of phase 2 v + 1 on: group 1, multiplying step v
    // in phase 2 v + 2, fetches A of step v + SA; group 0, multiplying step v in phase 2 v + 1, fetches B of
    // step v + SB - 1.  Step v + 1 has to have landed when phase 2 v + 2 begins.
    // gc: the group, known at compile time: the groups' fills differ in number, and a fill must not be
    // conditional inside the loop.
    auto k_loop = [&](auto ma, auto pass, auto gc) INLINE {
        // the wave's row blocks that hold rows of the group; -1: none of its columns are the tile's
        constexpr int MA = decltype(ma)::value > 0 ? decltype(ma)::value : 0;
        constexpr bool NO_COLS = decltype(ma)::value < 0;
        constexpr int S = decltype(pass)::value, GRP = decltype(gc)::value, MR = MA > 0 ? MA : 1;
        // Fill instructions: all of B; of A those that can hold rows of the group (32 rows each: a wave of
        // group 1 with MA live blocks belongs to a tile with at most this many).
        constexpr int NF = GRP == 0 ? PB : NO_COLS || MA == MB ? PA : WAVES_M * (MA + 1) - 1 < PA ? WAVES_M * (MA + 1) - 1 : PA;
        bf16x8 fa[2][2 * MR], fb[2][NI];
        // LINES: the lane's first chunk of a step within its row's line
        const int chunk0 = (lane >> 4) + ((lane & 15) * (K >> 3) & 7);
        // (tail: the step may be a partial one, whose 64 columns begin tail_back bytes earlier)
        auto read = [&](int v, auto tail) INLINE {
            const char* pa = smem + v % SA * A_BYTES;
            const char* pb = smem + v % SB * B_BYTES;
            const char* pb1 = smem + (v + 1) % SB * B_BYTES;
            const char* pb0 = smem + (v + SB - 1) % SB * B_BYTES;
            const int tb = decltype(tail)::value && v == S * nk + nk - 1 ? tail_back : 0;
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                const char* a = pa + (ra ^ (ks << 6));
                const int at = ks * 4 + chunk0 - tb / 16;  // the lane's chunk, from the start of line v
                const char* b = (LINES && at >= 8 ? pb1 : LINES && at < 0 ? pb0 : pb) +
                                (LINES && decltype(tail)::value ? rb0 + ((rb - rb0 + (ks << 6) - tb) & 127) : rb ^ (ks << 6));
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
            constexpr int NM = MA * 4 * NI, GAP = NM / NF > 0 ? NM / NF : 1;
            int p = 0;
#pragma unroll
            for (int i = 0; i < NM; ++i) {
                const int ni = i % NI, mi = i / NI % (2 * MR), ks = i / (NI * 2 * MR);
                acc[S][mi][ni] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[ks][ni], fa[ks][mi], acc[S][mi][ni], 0, 0, 0);
                if (decltype(filling)::value && i % GAP == GAP - 1 && p < NF) {
                    __builtin_amdgcn_sched_barrier(0);
                    fill(gc, vf, p);
                    ++p;
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            if (decltype(filling)::value) {
#pragma unroll
                for (; p < NF; ++p) fill(gc, vf, p);
            }
        };
        constexpr int AHEAD = GRP == 0 ? SB - 1 : SA;                     // the step fetched while v is multiplied
        constexpr bool MORE = LINES && GRP == 0;                          // a step takes its line and the next one
        constexpr int FLY = (GRP == 0 ? SB - 2 - MORE : SA - 2) * NF;     // fills behind those of step v + 1
        const int n_fill = nv + MORE;
        int v = S * nk;
        const int v_end = v + nk;
        if (S == 0) {  // the first steps (of B: above)
#pragma unroll
            for (int q = 0; q < (GRP == 1 ? AHEAD : 0); ++q)
                if (q < nv) {
#pragma unroll
                    for (int p = 0; p < NF; ++p) fill(gc, q, p);
                }
            if (n_fill >= AHEAD) wait_vm<(AHEAD - 1 - MORE) * NF>();  // step 0 has landed
            else wait_vm<0>();
            phase_end();
            if (GRP == 1) phase_end();
        }
        for (; v < v_end && v + AHEAD < n_fill; ++v) {
            if (MA > 0) read(v, std::false_type{});
            if (DUAL && S == 0 && v == v_end - 1 && tail_back > 0) clear_shared();
            if (GRP == 1) wait_vm<FLY>();  // A of step v + 1
            phase_end();
            multiply(std::true_type{}, v + AHEAD);
            if (GRP == 0) wait_vm<FLY>();  // B of step v + 1
            phase_end();
        }
        for (; v < v_end; ++v) {
            if (MA > 0) read(v, std::true_type{});
            if (v == v_end - 1 && tail_back > 0) clear_shared();
            if (GRP == 1) wait_vm<0>();
            phase_end();
            multiply(std::false_type{}, 0);
            if (GRP == 0) wait_vm<0>();
            phase_end();
        }
    };
    auto loops = [&](auto ma) INLINE {
        typedef std::integral_constant<int, 0> c0;
        typedef std::integral_constant<int, 1> c1;
        if (grp == 0) {
            k_loop(ma, c0{}, c0{});
            if constexpr (DUAL) k_loop(ma, c1{}, c0{});
        } else {
            k_loop(ma, c0{}, c1{});
            if constexpr (DUAL) k_loop(ma, c1{}, c1{});
        }
    };
    if (live == MB) loops(std::integral_constant<int, MB>{});
    else if (live == 0) loops(std::integral_constant<int, 0>{});
    else if (live < 0) loops(std::integral_constant<int, -1>{});
    else if (live == 1) loops(std::integral_constant<int, 1>{});
    else if (live == 2) loops(std::integral_constant<int, (MB > 2 ? 2 : 1)>{});
    else loops(std::integral_constant<int, (MB > 3 ? 3 : 1)>{});
    if (grp == 0) phase_end();

    // ---- epilogue: accumulator element i of a block is output column 4 (lane / 16) + i of row lane % 16.
    // Staged through LDS, 32 rows at a time in a region per wave, so that the tile leaves in 16-byte
    // stores.
    const size_t at0 = (size_t)part * ((size_t)g.P * g.N) + (size_t)row0 * g.N + n0;
    const unsigned ldc = (unsigned)g.N;
    if constexpr (F32) {  // 16-byte stores straight from the accumulators
        const int ln = lane_again();
        float* const Ft = static_cast<float*>(g.parts) + at0;
#pragma unroll
        for (int mi = 0; mi < 2 * MB; ++mi) {
            if (mi / 2 >= live) continue;
            const int row = (WAVES_M * (mi / 2) + wm) * 32 + mi % 2 * 16 + (ln & 15);
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
                const int col = wn * WN + ni * 16 + (ln >> 4) * 4;
                if (row < rows_here && col < width && n0 + col < g.N)
                    *reinterpret_cast<f32x4*>(Ft + (unsigned)row * ldc + (unsigned)col) = acc[0][mi][ni];
            }
        }
        return;
    }
    bf16_t* const Ct = static_cast<bf16_t*>(second ? g.C1 : g.k_parts > 1 ? g.parts : g.C) + at0;
    constexpr int OC = BN_OUT / WAVES_N;             // output columns of a wave
    constexpr int PITCH = OC * 2 + 16;
    constexpr int LPR = OC / 8, RPI = 64 / LPR;      // lanes per staged row, rows per read instruction
    const int ln = lane_again();
    char* const region = smem + wave * (32 * PITCH);
    char* const wr = region + (ln & 15) * PITCH + (ln >> 4) * 8;
    const int rd_row = ln / LPR, rd_chunk = ln % LPR;  // (lanes left over: rows past the last)
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
        for (int it = 0; it < (32 + RPI - 1) / RPI; ++it) {
            const int r = it * RPI + rd_row;
            if ((64 % LPR || 32 % RPI) && (rd_row >= RPI || r >= 32)) continue;
            const uint4 v = *reinterpret_cast<const uint4*>(region + r * PITCH + rd_chunk * 16);
            if (rbk + r < rows_here && c0 < width && n0 + c0 < g.N)
                *reinterpret_cast<uint4*>(Ct + (unsigned)(rbk + r) * ldc + (unsigned)c0) = v;
        }
    }
}

template <int BM, int BN, int WAVES_M, int SA, int SB, bool SWIGLU, bool DUAL, bool F32, bool NT_B, bool LINES>
int launch_pp(GemmArgs& g, hipStream_t st) {
    constexpr int BN_OUT = SWIGLU && !DUAL ? BN / 2 : BN;
    g.m_tiles_max = m_tiles_bound(g.P, g.E, BM);
    g.n_tiles = (g.N + BN_OUT - 1) / BN_OUT * ((!SWIGLU && g.C1) ? 2 : 1) * (g.k_parts > 1 ? g.k_parts : 1);
    constexpr size_t lds = (SA * BM + SB * BN) * BK * 2;
    static_assert(lds <= 160 * 1024, "LDS of a CU");
    const int grid = find_tile_grid(fitted_tiles(g.m_tiles_max * g.n_tiles, g.fit_width), kSplitSlots);
    static std::atomic<uint64_t> lds_allowed;
    const auto kern = gemm_pp_kernel<BM, BN, WAVES_M, SA, SB, SWIGLU, DUAL, F32, NT_B, LINES>;
    if (allow_dynamic_lds(reinterpret_cast<const void*>(kern), lds, lds_allowed) != MOE_OK) return MOE_ERR_LAUNCH;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(kThreads), lds, st, as_arg(g.keys), as_arg(g.offsets), g.P, g.E, g);
    return launch_status();
}
template <int BM, int BN, int WAVES_M, int SA, int SB, bool SWIGLU, bool DUAL, bool F32 = false>
int launch_pp(GemmArgs& g, bool nt, hipStream_t st) {
    return nt ? launch_pp<BM, BN, WAVES_M, SA, SB, SWIGLU, DUAL, F32, true, false>(g, st)
              : launch_pp<BM, BN, WAVES_M, SA, SB, SWIGLU, DUAL, F32, false, false>(g, st);
}
// weights in rows that are no multiples of a line, past the caches
template <int BM, int BN, int WAVES_M, int SA, int SB>
int launch_pp_lines(GemmArgs& g, bool swiglu, hipStream_t st) {
    if (swiglu) return launch_pp<BM, BN, WAVES_M, SA, SB, true, false, false, true, true>(g, st);
    return g.k_parts > 1 && g.parts_f32 ? launch_pp<BM, BN, WAVES_M, SA, SB, false, false, true, true, true>(g, st)
                                        : launch_pp<BM, BN, WAVES_M, SA, SB, false, false, false, true, true>(g, st);
}

}  // namespace

// Operands whose rows are reached by 32-bit byte offsets (a 24-bit multiply), at least one whole k-step
static bool rows_supported(long long a_rows, long long N, long long K) {
    return K >= BK && K < (1 << 23) && N < (1 << 24) && a_rows * K * 2 < (1ll << 32) && N * K * 2 < (1ll << 32);
}

// One segment, no addends
bool gemm_pp_supported(const GemmArgs& g) {
    const GemmSeg& sg = g.seg[0];
    const long long a_rows = sg.gather ? (g.P - 1) / (g.row_div > 0 ? g.row_div : 1) + 1 : g.P;
    return g.nseg == 1 && !g.add0 && rows_supported(a_rows, g.N, sg.K);
}

// ---- rows per tile and parts of K, by a model of the launch in us ------------------------------------------
// Rounds of 256 workgroups (one per CU), each with 6 us of fixed cost and its k-steps at what bounds them:
// fills at 46 GB/s per CU, the matrix cores, or the latency from a fill of A to its use, which is shorter the
// more k-steps of A LDS holds (two of 256 rows, four of 128 or 64).  Few rows per group and narrow outputs
// want small tiles, large groups tall ones; cutting K pays where the tiles are too few for the CUs (the
// 2048-wide down projection of 4096 rows has 160 of 256 x 256) or the chain of k-steps of a tile is long.
// Parts are written and read at 6 TB/s, in place of the 4 bytes of one bf16 output; a launch of its own that adds
// them, and leaves that output all the same, costs 5 us.
// Checked against (us): gate/up of the 2048 / 5632 layer at 4 to 32 rows per expert 80 / 79 with 128 / 64 rows
// against 82 with 256, at 64 rows 88 with 128 against 96; of the 1024 / 2816 layer at 128 rows 28 with
// 256 against 38 with 128; down projection at 2048 tokens 107 in three bf16 parts, 115 in three fp32 ones, 124 in one.
// fp32 parts forced to 1 to 4 at 36 sizes from 128 to 6000 tokens on four layers (432 to 2048 wide): the count taken
// here is within 2 % of the fastest, 3 % once (whole layer, 1 / 2 / 3 / 4 parts: 2048 / 5632 at 128 tokens 127 / 115 /
// 115 / 115; 1024 / 2816 at 128 tokens 49.9 / 43.5 / 41.4 / 40.6, at 512 tokens 59.8 / 56.2 / 53.8 / 53.8).
struct PpChoice {
    int bm, parts;
};
static PpChoice choose(long long P, int E, int N, int K, int copies, bool swiglu, bool dual, int parts_max, bool f32,
                       bool sum_launch) {
    const double groups = P < E ? (double)P : (double)E, n = P / groups;
    const int bn = swiglu && !dual ? 2 : 1;  // B rows per output column of a tile
    const int cols = dual || bn == 2 ? 128 : 256, nb = (N + cols - 1) / cols;
    const int steps = (K + BK - 1) / BK * (dual ? 2 : 1);
    PpChoice best{256, 1};
    double best_cost = 0;
    for (int bm = 256; bm >= 64; bm /= 2) {
        const double rows = n < bm ? n : bm, mt = groups * (n / bm + 0.5 > 1.0 ? n / bm + 0.5 : 1.0) * 1.05;
        const double latency = bm == 256 ? 0.75 : bm == 128 ? 0.55 : 0.45;
        for (int q = 1; q <= parts_max && (q == 1 || steps / q >= 4); ++q) {
            const double m_all = mt * q * copies, rounds = (double)(long long)((m_all * nb + 255) / 256);
            const double fit = (double)(long long)(256 * rounds / m_all), width = rounds > 2 || fit < nb ? (nb > 1 ? cols : N) : N / fit;
            double step = (rows + width * bn) * (BK * 2) / 46e3;
            const double mfma = rows * width * bn * (1.05 / 65536);
            if (step < mfma) step = mfma;
            if (step < latency) step = latency;
            double cost = rounds * (steps * step / q + 6);
            if (q > 1) cost += (double)(!f32 ? (q - 1) * 4 : sum_launch ? q * 8 : q * 8 - 4) * P * N / 6e6 + (sum_launch ? 5 : 0);
            if ((bm == 256 && q == 1) || cost < best_cost) {
                best_cost = cost;
                best = PpChoice{bm, q};
            }
        }
    }
    return best;
}

int gemm_pp_split(long long P, int E, int N, int K, int parts_max, bool parts_f32, bool sum_launch) {
    if (P <= 0 || !rows_supported(P, N, K)) return 1;
    return choose(P, E, N, K, 1, false, false, parts_max, parts_f32, sum_launch).parts;
}

// ---- weights whose rows are no multiples of a cache line ---------------------------------------------------------
// Fetched 128 bytes of every row at a time from where the rows begin, each line is read by two k-steps and each request touches
// two lines: 2040 / 5624 took 17-23 % more than 2048 / 5632 from 128 to 4000 tokens.  Fetched in whole lines a step lies in
// two, so LDS holds a step more: 128-row tiles with two steps of A, or 256-row tiles 192 columns wide.  Whole layer, us, before /
// with gate and up fetched so: 2040 / 5624 48 tokens 124.6 / 113.5, 128 tokens 134.5 / 121.9, 300 tokens 153.9 / 136.7; 1208 /
// 3224 128 tokens 60.3 / 50.4, 300 tokens 76.9 / 62.8; 1032 / 2760 48 tokens 47.0 / 42.1; the down product too: 2040 / 5624 48
// tokens 124 / 117 (alone), 300 tokens 154 / 147, 900 tokens 212 / 204.  Taken where
//   - no round of tiles is added, with Zipf loads nor with even ones, a quarter more than the average to be on the safe
//     side (one more: 700 tokens of 1400 / 3736 98.3 / 106.8, 512 tokens of 1440 / 3840, 128 rows per expert, 82.1 / 97.8).  Loads more
//     skewed than that may still add one (984 / 2624, 570 tokens, 47 % of them with one expert, 65.2 / 78.4): with a quarter more of
//     the Zipf loads too, that case and two more of 170 drawn ones are spared 7-20 %, and 13 lose 3-10 % (mean gain 6.0 %, 6.1 without);
//   - a plain product has tiles for half the CUs, and not fewer than it had (300 tokens of 1032 / 2760, one part, 62.6 / 71.4);
//   - the weights are large, a matrix of all experts 30 MB for gate and up, 50 each for two plain products, 40 for a single one.  Below, a launch is short, and the step more that its
//     tiles start with costs what the lines save.  Weights cold (as many copies of the layer in turn as are past the memory-side
//     cache, the state of any model of several layers), whole layer, without / with gate and up fetched so: 664 / 1800 (2 x 18 MB) 48
//     tokens 31.2 / 31.4, 500 tokens 43.7 / 43.2; 712 / 1944 (21 MB) 32.7 / 32.6, 46.7 / 45.6; 4 experts of 1096 / 2968 (25 MB), 150
//     tokens, 42.6 / 44.0, of 1200 / 3200 (29 MB), 142 tokens, Zipf loads, 43.5 / 44.6; 856 / 2320 (30 MB) 53 tokens 38.7 / 36.2; 880 / 2416 (32 MB)
//     178 tokens 42.6 / 38.8; 904 / 2440 (34 MB) 48 tokens 41.0 / 37.4, 500 tokens 59.9 / 57.5; 1400 / 3736 (80 MB) 66.0 / 56.5 at 48.  The
//     down product alone: 952 / 2568 (37 MB) 48 tokens 42.7 / 43.3, 128 tokens 44.8 / 45.9; 4 experts of 1400 / 3736 (40 MB), 64 tokens,
//     46.8 / 48.9; 1032 / 2760 (43 MB) 47.1 / 46.4 and, 128 tokens with Zipf loads, 53.9 / 56.3; 4 experts of 1448 / 3928 (43 MB), 509
//     tokens, 85.8 / 82.8; 1400 / 3736 (80 MB) 66.0 / 64.1, 78.2 / 79.0.  The two rank
//     products, 16 experts: rank 640 on 1272 / 3408 (25 MB) 253 tokens 86.9 / 92.1, 768 on 1528 / 4120 (36 MB) 164 tokens 111.3 / 117.8, 832 on
//     1672 / 4520 (43 MB) 38 tokens 109.2 / 113.8, 912 on 1824 / 4904 (51 MB) 602 tokens 193.3 / 190.2, 1024 on 2040 / 5584 (64 MB) 1579 tokens
//     275.5 / 266.9.  Where one layer runs alone and its weights stay in that cache,
//     cut lines cost little: 760 / 2056 48 tokens 29.4 / 32.5, 1304 / 3560 50.3 / 52.3;
//   - groups are one tall tile on average: beyond, the narrow tiles' LDS reads cost what the fills save (2500 tokens of
//     2040 / 5624 406 / 404, 4000 tokens 653 / 664).
// The rows have to lie in whole lines together: none is then read that is not the weights'.
static int m_tiles(double P, int E, int bm, bool zipf) {
    static const std::array<double, kMaxExperts> shares = [] {
        std::array<double, kMaxExperts> w;
        for (int e = 0; e < kMaxExperts; ++e) w[e] = pow(e + 1, -1.1);
        return w;
    }();
    double sum = 0;
    for (int e = 0; e < E; ++e) sum += shares[e];
    int tiles = 0;
    for (int e = 0; e < E; ++e) tiles += (int)ceil(P * (zipf ? shares[e] / sum : 1.0 / E) / bm);
    return tiles;
}

// Rows per tile of that form, 0: not taken.  bm: rows per tile of the other form
static int line_rows(const GemmArgs& g, bool swiglu, int bm) {
    const GemmSeg& sg = g.seg[0];
    const int K = sg.K, parts = g.k_parts > 1 ? g.k_parts : 1;
    auto whole = [](const void* p) { return reinterpret_cast<uintptr_t>(p) % 128 == 0; };
    if (K % 64 == 0 || K % 8 != 0 || g.N % 8 != 0 || sg.strideB % 64 != 0 || !whole(sg.B0) || !whole(sg.B1) ||
        (K + BK - 1) / BK < 2 * parts || (swiglu && sg.A0 != sg.A1))
        return 0;
    if (g.P > 256ll * g.E || (sg.strideB != 0 ? g.E : 1) * 2ll * g.N * K < ((swiglu ? 30 : g.C1 ? 50 : 40) << 20)) return 0;
    const int copies = parts * (!swiglu && g.C1 ? 2 : 1), per_row = swiglu ? 2 : 1;
    for (int rows = 256; rows >= 128; rows /= 2) {
        bool ok = true;
        for (int zipf = 0; zipf < 2; ++zipf) {
            const int cols = (rows == 256 ? 192 : 256) / per_row, before = 256 / per_row;
            const int tiles = m_tiles(zipf ? g.P : 1.25 * g.P, g.E, rows, zipf) * copies * ((g.N + cols - 1) / cols);
            const int other = m_tiles(g.P, g.E, bm, zipf) * copies * ((g.N + before - 1) / before);
            ok = ok && (tiles + 255) / 256 <= (other + 255) / 256 && (swiglu || (tiles >= 128 && tiles >= other));
        }
        if (ok) return rows;
    }
    return 0;
}

int run_gemm_pp(GemmArgs& g, bool swiglu, hipStream_t st) {
    const bool dual = swiglu && g.seg[0].A0 != g.seg[0].A1;
    const int parts = g.k_parts > 1 ? g.k_parts : 1;  // decided by the caller
    const int bm = choose(g.P, g.E, g.N, g.seg[0].K / parts, parts * (!swiglu && g.C1 ? 2 : 1), swiglu, dual, 1, false, false).bm;
    g.fit_width = 2;
    // Weights past the caches where an expert has one or two m-tiles: a plain read of 335 MB in this pattern
    // runs at 6.0 TB/s without the hint and at 6.7 with it.  (2048 / 5632 layer at 8 tokens 95 -> 86 us, 64
    // tokens 124 -> 114, 256 tokens 129 -> 120; where the m-tiles of an expert share its weights in L2 it
    // hurts: 2048 tokens 313 -> 326.)  Drawn at an average of 256 rows per expert, one tile of the tallest kind:
    // 512 tokens 1024 / 2816 55.9 -> 51.9.
    // The smaller tiles follow the same line (whole layer, us, hint at every size / by this rule: 1100 tokens 432 / 1152
    // 37.9 / 33.2, 1024 / 2816 80.1 / 78.4, 400 / 1064 of rank 200 51.6 / 45.3; 2048 tokens on a shared base 282.8 / 280.4; two
    // of 32 sizes were faster with it, 512 tokens on the shared base of 2048 / 5632 142.7 without and 138.3 with).
    // Rows that are no multiples of a line: a k-step ends inside a line, the next one reads that line again, and with the hint
    // it comes from HBM again.  Whole layer, us, with / without: 2040 / 5624 40 tokens 161.7 / 125.6, 256 tokens 171.6 / 149.4,
    // 1024 tokens 305.5 / 259.0; 1032 / 2760 54.2 / 47.4, 128 tokens 58.1 / 50.2, 1024 tokens 104.7 / 97.1; 520 / 1400, 4 experts,
    // 150 tokens 24.7 / 21.5.  The same where rows are whole half-lines and only every other one is cut (a chain of layers past the
    // memory-side cache on one workspace): 480 / 1312 400 tokens 30.4 / 29.1, 864 / 2336 256 tokens 44.2 / 42.3, 1440 / 3840 600 tokens
    // 87.0 / 85.5, 777 tokens 92.6 / 91.4, 1000 tokens 127.8 / 122.6, 1952 / 5216 1000 tokens 201.6 / 182.9; none of nine widths at eleven
    // sizes was 1 % faster with it.  Where calls take turns on several workspaces, whose lines the weights
    // then drive out of that cache, part of it is lost again: 8 experts of 1056 to 1440 wide, 120 to 194 rows per expert, 1-2 % slower without
    // (1440 / 3840 777 tokens 90.4 / 92.5; on one workspace 90.4 / 87.8), wider ones and 16 experts 1-8 % faster all the same.
    const bool nt = g.seg[0].K % 64 == 0 && g.P <= 256 * g.E;
    if (const int rows = line_rows(g, swiglu, bm))
        return rows == 128 ? launch_pp_lines<128, 256, 2, 2, 4>(g, swiglu, st) : launch_pp_lines<256, 192, 4, 2, 4>(g, swiglu, st);
    if (!swiglu) {
        const bool f32 = g.k_parts > 1 && g.parts_f32;
        // One part and few row tiles: to fill the chip the kernel makes the tiles narrower (fit_width); where that leaves half a
        // tile or less, the other half of its rows of B would be the last one over and over, and half of its waves idle.
        // Whole layer, us, 256 / 128 columns: 300 tokens 1024 / 2816 53.2 / 49.7, 512 tokens 640 / 1728 40.6 / 37.9, 777 tokens 432 /
        // 1152 32.8 / 31.0, 2048 tokens 43.9 / 40.3.  In parts, or with tall tiles, there was no gain (512 tokens 1024 / 2816
        // 53.1 / 53.9, 432 / 1152 28.4 / 29.1), and none where the tiles are a few k-steps long (a low-rank term of rank 128, 300
        // tokens, 128.5 / 130.8).
        // Tiles for one round by the model above; past that the wide ones are the better fit (1024 tokens of rank 1024 on 2048 /
        // 5632 204 / 209).
        const double groups = g.P < g.E ? g.P : g.E, m_all = groups * 1.05 * fmax(g.P / groups / bm + 0.5, 1.0);
        if (bm <= 128 && parts == 1 && !g.C1 && g.seg[0].K >= 512 && m_all * ((g.N + 127) / 128) <= 256)
            return bm == 64 ? launch_pp<64, 128, 2, 8, 6, false, false>(g, nt, st) : launch_pp<128, 128, 4, 5, 5, false, false>(g, nt, st);
        if (bm == 64)
            return f32 ? launch_pp<64, 256, 2, 4, 4, false, false, true>(g, nt, st) : launch_pp<64, 256, 2, 4, 4, false, false>(g, nt, st);
        if (bm == 128)
            return f32 ? launch_pp<128, 256, 2, 4, 3, false, false, true>(g, nt, st) : launch_pp<128, 256, 2, 4, 3, false, false>(g, nt, st);
        return f32 ? launch_pp<256, 256, 2, 2, 3, false, false, true>(g, nt, st) : launch_pp<256, 256, 2, 2, 3, false, false>(g, nt, st);
    }
    if (dual) {
        if (bm == 64) return launch_pp<64, 128, 2, 8, 6, true, true>(g, nt, st);
        if (bm == 128) return launch_pp<128, 128, 4, 4, 5, true, true>(g, nt, st);
        return launch_pp<256, 128, 4, 2, 3, true, true>(g, nt, st);
    }
    if (bm == 64) return launch_pp<64, 256, 2, 4, 4, true, false>(g, nt, st);
    if (bm == 128) return launch_pp<128, 256, 2, 4, 3, true, false>(g, nt, st);
    return launch_pp<256, 256, 2, 2, 3, true, false>(g, nt, st);
}

// out = sum of the parts, in part order, rounded once; n a multiple of 8
__global__ __launch_bounds__(256) void sum_parts_kernel(const f32x4* __restrict__ parts, int q, long long n8,
                                                        bf16x8* __restrict__ out) {
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n8; i += (long long)gridDim.x * 256) {
        f32x4 lo = parts[2 * i], hi = parts[2 * i + 1];
        for (int p = 1; p < q; ++p) {
            lo += parts[(p * n8 + i) * 2];
            hi += parts[(p * n8 + i) * 2 + 1];
        }
        bf16x8 o;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            o[j] = (bf16_t)lo[j];
            o[4 + j] = (bf16_t)hi[j];
        }
        out[i] = o;
    }
}

int launch_sum_parts(const float* parts, int q, long long n, void* out, hipStream_t st) {
    const long long n8 = n / 8;
    const int grid = (int)((n8 + 255) / 256 < 2048 ? (n8 + 255) / 256 : 2048);
    hipLaunchKernelGGL(sum_parts_kernel, dim3(grid), dim3(256), 0, st, reinterpret_cast<const f32x4*>(parts), q, n8,
                       static_cast<bf16x8*>(out));
    return launch_status();
}

}  // namespace moe
