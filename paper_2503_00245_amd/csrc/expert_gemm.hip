// Grouped expert GEMMs for prefill: every expert multiplies its own contiguous group of
// sorted rows by its own matrices (Sec. 2.1), with the SwiGLU activation fused into the
// gate/up product's epilogue and weight-decomposed experts (Sec. 2.2, Eq. 1) expressed
// as extra K-segments accumulated into the same output tile.
//
// The problem and the tile enumeration are in gemm.h; both operands are K-contiguous, which is
// exactly what an MFMA lane wants: 8 consecutive k of one row per 16-byte read.
//
// bf16 kernels: block tile BM x BN x BK on (BM / WM) * (BN / WN) waves, wave tile WM x WN built
// from v_mfma_f32_32x32x16_bf16, fp32 accumulators in registers.  Global -> registers -> LDS
// with two LDS stages and two register sets, so that three tiles are in flight; a K that is
// not a multiple of BK (any multiple of 8) ends in a partly zero-filled step.  LDS rows are BK bf16 wide with the 16-byte chunk index XOR-ed by a
// function of the row, which spreads both the row-wise fills and the column-of-rows MFMA
// operand reads over all banks.  Tiles are enumerated expert-major, then n-tile, then the
// expert's m-tiles, and the workgroup id is remapped so that each XCD walks a contiguous
// eighth of that order (consecutive tiles share a weight tile and hit in that XCD's L2).
// run_gemm picks the tile shape from the pair count and the output width.  bf16 products of one K-segment of 64
// or more without per-token addends run in expert_gemm_pp.hip; what is left for the kernel here are the
// shared base's low-rank SwiGLU product (addends), its staged form (two segments) and small or huge K and N.
// fp32 problems: expert_gemm_f32.hip.
#include "gemm.h"

namespace moe {

// ============================================================================= bf16 MFMA
// LDS tile rows hold BK bf16 (BK/8 chunks of 16 bytes).  The chunk index is XOR-ed with a
// function of the row chosen so that 16 consecutive rows read at one chunk index (an MFMA
// operand read) touch 16 distinct 16-byte bank groups, as do the row-wise fills.
template <int BK>
__device__ __forceinline__ int lds_off(int row, int chunk) {
    constexpr int CPR = BK / 8;  // chunks per row
    return row * (BK * 2) + ((chunk ^ ((row / (16 / CPR)) % CPR)) << 4);
}

// LDS of a workgroup of the kernel below
template <int BM, int BN, int BK, bool DUAL_A, int KG>
constexpr size_t lds_bytes() {
    return KG * 2 * ((size_t)BM * BK * 2 * (DUAL_A ? 2 : 1) + (size_t)BN * BK * 2);
}
// Workgroups of a kernel that one XCD (32 CUs) holds at a time, for the tail split: bounded by LDS and, for
// these tiles (64 or more accumulator registers per lane), by two waves per SIMD; halves of BM / 2
// rows only make sense when each wave's rows fall in one half.
// (For kernels that run one or two workgroups per CU.  It needs a full round before the thin
// one: with less than one round of tiles in all, halves -- which each still stream the whole
// weight tile -- measured slower, down product at 512 tokens 94 us instead of 73.  Cutting the
// halves once more along the columns, one wave of four left with work, was slower too:
// down product at 2048 tokens 152 us against 144.)
template <int BM, int BN, int BK, int WM, int WN, bool DUAL_A, int KG>
constexpr int split_slots() {
    constexpr int NTHR = (BM / WM) * (BN / WN) * 64 * KG;
    constexpr int kWavesPerSimd = (WM * WN / 64 >= 64) ? 2 : 3;  // by accumulator registers per lane
    constexpr int kByLds = (int)((160 * 1024) / lds_bytes<BM, BN, BK, DUAL_A, KG>()), kByWaves = kWavesPerSimd * 256 / NTHR;
    constexpr int kPerCU = kByLds < kByWaves ? kByLds : kByWaves;
    return (BM / 2) % WM == 0 && KG == 1 && kPerCU <= 2 ? 32 * kPerCU : 0;
}

// ============================================================================= bf16 MFMA, deep pipeline
// K a multiple of 8 (rows are read in 16-byte chunks).  Two register sets and two LDS stages, so
// three tiles are in flight: tile kt is multiplied out of LDS while tile kt+1 waits in registers to be
// written to the other LDS stage at the end of the step and tile kt+2 is being fetched.
// That puts two full steps of MFMA work between issuing a global load and first needing
// its data.  Loads are unconditional (rows past the end of a group / matrix are clamped to
// its last row and only feed outputs the epilogue never stores), so the loop has no
// divergent control flow.  (Direct global->LDS loads gained nothing in this
// schedule, where a step's loads are issued together and hold back the MFMAs behind them;
// expert_gemm_pp.hip spreads them between the MFMAs.)
//
// KG > 1: the workgroup holds KG groups of (BM / WM) * (BN / WN) waves.  Every group runs
// the whole pipeline on its own 1/KG of the k-steps, with its own LDS stages, and the
// groups' accumulators meet in LDS at the end, added in group order.  This is for products
// with fewer tiles than CUs and a long K, where the serial chain of k-steps of a single
// tile, not the chip's throughput, sets the time.  Needs K % (KG * BK) == 0.
// TAIL: K need not be a multiple of BK (a separate instantiation, so that the loop of the common
// case carries none of the tail's bookkeeping: with it the down product of a 2048 x 5632 layer
// measured 3.5 % slower).
template <int BM, int BN, int BK, int WM, int WN, bool SWIGLU, bool DUAL_A, int NS, int KG, bool ADD = false,
          bool TAIL = false>
__global__ __launch_bounds__((BM / WM) * (BN / WN) * 64 * KG) void gemm_bf16_deep_kernel(const GemmArgs g) {
    static_assert(!ADD || SWIGLU, "per-token addends belong to the SwiGLU epilogue");
    static_assert(!TAIL || KG == 1, "a K tail only without k-groups");
    constexpr int WAVES_N = BN / WN;
    constexpr int NTHR = (BM / WM) * WAVES_N * 64;  // threads of one k-group
    constexpr int MT = WM / 32, NT = WN / 32;
    static_assert(!SWIGLU || NT % 2 == 0, "gate and up fragments pair up");
    constexpr int CPR = BK / 8;
    constexpr int RPP = NTHR / CPR;
    static_assert(BM % RPP == 0 && BN % RPP == 0 && (BN / 2) % RPP == 0, "fill passes");
    constexpr int AI = BM / RPP, BI = BN / RPP;
    constexpr int NA = DUAL_A ? 2 : 1;
    constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2;
    constexpr int STAGE = A_BYTES * NA + B_BYTES;
    extern __shared__ __align__(16) char smem[];

    int e, row0, row_end, nt;
    constexpr int SPLIT = split_slots<BM, BN, BK, WM, WN, DUAL_A, KG>();
    auto n_tiles_of = [&](int) { return g.n_tiles; };
    int lo, hi;
    group_bounds(g.offsets, g.E, g.P, lo, hi);
    if (!(g.hidden_a ? find_tile<kHiddenOperandBlock, SPLIT>(lo, hi, g.E, BM, n_tiles_of, e, row0, row_end, nt)
                    : find_tile<1, SPLIT>(lo, hi, g.E, BM, n_tiles_of, e, row0, row_end, nt))) return;
    constexpr int BN_OUT = SWIGLU ? BN / 2 : BN;
    // two plain products in one launch: the upper half of the n-tiles belongs to (A1, B1, C1)
    const bool second = !SWIGLU && g.C1 != nullptr && nt >= g.n_tiles / 2;
    if (second) nt -= g.n_tiles / 2;
    const int n0 = nt * BN_OUT;

    const int kg = threadIdx.x / NTHR;   // k-group of this wave
    const int tid = threadIdx.x % NTHR;  // thread within the group
    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WAVES_N, wn = wave % WAVES_N;
    const int ld_row = tid / CPR, ld_chunk = tid % CPR;
    char* const gmem = smem + kg * (2 * STAGE);  // this group's two stages

    f32x16 acc[MT][NT];
    if constexpr (ADD) {
        // Per-token addends: the accumulators start from the token's rows of add0 / add1 instead
        // of zero.  The gathers are issued here, ahead of the first tile loads and with every
        // register still free, so their latency hides behind the pipeline's own start-up.
        static_assert(KG == 1, "addends are added once");
        const bf16_t* add0 = static_cast<const bf16_t*>(g.add0);
        const bf16_t* add1 = static_cast<const bf16_t*>(g.add1);
#pragma unroll
        for (int mi = 0; mi < MT; ++mi) {
            int tok[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int row = min(row0 + wm * WM + mi * 32 + (i >> 2) * 8 + (lane >> 5) * 4 + (i & 3), row_end - 1);
                tok[i] = quick_div(min(max(g.row_map[row], 0), g.P - 1), g.row_div);
            }
#pragma unroll
            for (int ni = 0; ni < NT / 2; ++ni) {
                const int col = min(n0 + wn * (WN / 2) + ni * 32 + (lane & 31), g.N - 1);
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const size_t at = (size_t)tok[i] * g.N + col;
                    acc[mi][ni][i] = (float)add0[at];
                    acc[mi][ni + NT / 2][i] = (float)add1[at];
                }
            }
        }
    } else {
#pragma unroll
        for (int mi = 0; mi < MT; ++mi)
#pragma unroll
            for (int ni = 0; ni < NT; ++ni)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[mi][ni][i] = 0.f;
    }

    struct Regs {  // a tile's share of one thread: AI and BI fill passes of RPP rows
        bf16x8 a[AI], a1[DUAL_A ? AI : 1], b[BI];
    };

    for (int sidx = 0; sidx < g.nseg; ++sidx) {
        const GemmSeg& sg = g.seg[sidx];
        const int K = sg.K;
        const bool dual = DUAL_A && sg.A1 != sg.A0;
        const bf16_t* B0 = static_cast<const bf16_t*>(second ? sg.B1 : sg.B0) + (size_t)e * sg.strideB;
        const bf16_t* B1 = SWIGLU ? static_cast<const bf16_t*>(sg.B1) + (size_t)e * sg.strideB : B0;
        const int nk = (K + BK * KG - 1) / (BK * KG);  // k-steps of this group (the same for every group)
        const int k_begin = kg * nk * BK;
        const int k_last = (nk - 1) * BK;    // relative to k_begin
        // K tail (TAIL: K % BK != 0, a multiple of 8): in the last k-step a thread whose 16-byte
        // chunk lies at or beyond K reads an earlier chunk of its row instead (in bounds) and zeroes
        // its registers before they go to LDS.  Which threads those are never changes (a thread
        // always loads the same chunk of a tile), so the loop pays one vector min per step.
        const int tail_kt = (TAIL && K % BK != 0) ? nk - 1 : -1;               // wave-uniform
        const bool tail_dead = TAIL && k_begin + k_last + ld_chunk * 8 >= K;    // per thread
        const int k_last_t = tail_dead ? max(k_last - BK, -(ld_chunk * 8)) : k_last;

        const bf16_t* pa[AI];
        const bf16_t* pa1[DUAL_A ? AI : 1];
        const bf16_t* pb[BI];
        // (the row-map lookups of all of a thread's rows are issued together: one latency, not AI)
        int arow[AI];
#pragma unroll
        for (int i = 0; i < AI; ++i) arow[i] = min(row0 + ld_row + RPP * i, row_end - 1);
        if (sg.gather) {
#pragma unroll
            for (int i = 0; i < AI; ++i) arow[i] = g.row_map[arow[i]];
#pragma unroll
            for (int i = 0; i < AI; ++i) arow[i] = quick_div(min(max(arow[i], 0), g.P - 1), g.row_div);
        }
#pragma unroll
        for (int i = 0; i < AI; ++i) {
            const size_t off = (size_t)arow[i] * K + k_begin + ld_chunk * 8;
            pa[i] = static_cast<const bf16_t*>(second ? sg.A1 : sg.A0) + off;
            if (DUAL_A) pa1[i] = static_cast<const bf16_t*>(sg.A1) + off;
        }
#pragma unroll
        for (int i = 0; i < BI; ++i) {
            const int j = ld_row + RPP * i;
            const int n = min(SWIGLU ? n0 + (j % (BN / 2)) : n0 + j, g.N - 1);
            const size_t off = (size_t)n * K + k_begin + ld_chunk * 8;
            pb[i] = ((SWIGLU && i >= BI / 2) ? B1 : B0) + off;
        }
        auto gload = [&](Regs& r, int k0) {
#pragma unroll
            for (int i = 0; i < AI; ++i) {
                r.a[i] = *reinterpret_cast<const bf16x8*>(pa[i] + k0);
                if (DUAL_A && dual) r.a1[i] = *reinterpret_cast<const bf16x8*>(pa1[i] + k0);
            }
#pragma unroll
            for (int i = 0; i < BI; ++i) r.b[i] = *reinterpret_cast<const bf16x8*>(pb[i] + k0);
        };
        auto zero_dead = [&](Regs& r) {
            if (tail_dead) {
#pragma unroll
                for (int i = 0; i < AI; ++i) {
                    r.a[i] = bf16x8{};
                    if (DUAL_A) r.a1[i] = bf16x8{};
                }
#pragma unroll
                for (int i = 0; i < BI; ++i) r.b[i] = bf16x8{};
            }
        };
        auto lstore = [&](int stage, const Regs& r) {
            char* base = gmem + stage * STAGE;
#pragma unroll
            for (int i = 0; i < AI; ++i) {
                const int row = ld_row + RPP * i;
                *reinterpret_cast<bf16x8*>(base + lds_off<BK>(row, ld_chunk)) = r.a[i];
                if (DUAL_A && dual)
                    *reinterpret_cast<bf16x8*>(base + A_BYTES + lds_off<BK>(row, ld_chunk)) = r.a1[i];
            }
            char* bb = base + A_BYTES * NA;
#pragma unroll
            for (int i = 0; i < BI; ++i)
                *reinterpret_cast<bf16x8*>(bb + lds_off<BK>(ld_row + RPP * i, ld_chunk)) = r.b[i];
        };
        // MA = how many of the wave's MT 32-row blocks hold rows of the group (the rest are skipped)
        auto compute = [&](int stage, auto ma) {
            constexpr int MA = decltype(ma)::value;
            const char* base = gmem + stage * STAGE;
            const char* a0b = base;
            const char* a1b = (DUAL_A && dual) ? base + A_BYTES : base;
            const char* bb = base + A_BYTES * NA;
#pragma unroll
            for (int ks = 0; ks < BK / 16; ++ks) {
                const int chunk = ks * 2 + (lane >> 5);
                bf16x8 fa[MA], fa1[DUAL_A ? MA : 1], fb[NT];
#pragma unroll
                for (int mi = 0; mi < MA; ++mi) {
                    const int r = wm * WM + mi * 32 + (lane & 31);
                    fa[mi] = *reinterpret_cast<const bf16x8*>(a0b + lds_off<BK>(r, chunk));
                    if (DUAL_A) fa1[mi] = *reinterpret_cast<const bf16x8*>(a1b + lds_off<BK>(r, chunk));
                }
#pragma unroll
                for (int ni = 0; ni < NT; ++ni) {
                    int r;
                    if constexpr (SWIGLU)
                        r = (ni < NT / 2 ? 0 : BN / 2) + wn * (WN / 2) + (ni % (NT / 2)) * 32 + (lane & 31);
                    else
                        r = wn * WN + ni * 32 + (lane & 31);
                    fb[ni] = *reinterpret_cast<const bf16x8*>(bb + lds_off<BK>(r, chunk));
                }
#pragma unroll
                for (int mi = 0; mi < MA; ++mi)
#pragma unroll
                    for (int ni = 0; ni < NT; ++ni) {
                        const bf16x8 av = (DUAL_A && SWIGLU && ni >= NT / 2) ? fa1[mi] : fa[mi];
                        acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, fb[ni], acc[mi][ni], 0, 0, 0);
                    }
            }
        };

        // NS register sets: tile kt is multiplied out of LDS while tile kt+1 waits in registers to
        // be written to the other LDS stage at the end of the step and tiles kt+2 .. kt+NS are in
        // flight from memory.  Every load and LDS write below is unconditional (k offsets are
        // clamped to the last tile, whose re-fetch near the end is harmless): the
        // outstanding-load count at each wait is then a compile-time constant and a wait for
        // tile kt+1 never also waits for the younger loads behind it.
        constexpr int UNR = (NS % 2 == 0) ? NS : 2 * NS;  // steps until (set, stage) repeat
        Regs r[NS];
#pragma unroll
        for (int q = 0; q < NS; ++q) gload(r[q], min(q * BK, k_last_t));
        if constexpr (TAIL) {
            if (tail_kt == 0) zero_dead(r[0]);
        }
        __syncthreads();  // the previous segment's readers are done with both stages
        lstore(0, r[0]);
        __syncthreads();
        // Issue order inside a step: the step's global loads and LDS writes are spread through
        // the MFMA sequence (one memory instruction in the shadow of each MFMA) instead of
        // running as separate phases, so a wave's MFMA stream has no load/store-only gaps.
        auto interleave = [&](auto ma) {
#if defined(__HIP_DEVICE_COMPILE__)
            constexpr int MA = decltype(ma)::value;
            constexpr int NM = MA * NT * (BK / 16);           // MFMAs per step
            constexpr int NR = (MA * NA + NT) * (BK / 16);    // LDS fragment reads per step
            constexpr int NL = AI * NA + BI;                  // global loads = LDS writes per step
            constexpr int RPM = (NR + NM - 1) / NM;
            constexpr int LPM = (2 * NL + NM - 1) / NM;
            __builtin_amdgcn_sched_group_barrier(0x100, MA * NA + NT, 0);  // first fragments
#pragma unroll
            for (int i = 0; i < NM; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);    // one MFMA
                __builtin_amdgcn_sched_group_barrier(0x100, RPM, 0);  // next fragments
                if (i < NM / 2)
                    __builtin_amdgcn_sched_group_barrier(0x020, LPM, 0);  // global loads, tile kt+2
                else
                    __builtin_amdgcn_sched_group_barrier(0x200, LPM, 0);  // LDS writes, tile kt+1
            }
#endif
        };
        // The wave multiplies only those of its 32-row blocks that hold rows of the group.  A wave
        // with none keeps filling LDS and meeting the barriers but issues no fragment reads or
        // MFMAs, which leaves its SIMD and the LDS read port to the waves that do have rows.
        auto k_loop = [&](auto ma) {
            constexpr int MA = decltype(ma)::value;
            // step S of the unrolled body: multiply tile kt (stage S & 1), refill set S % NS (its
            // tile went to LDS at the end of the previous step) with tile kt + NS, write tile
            // kt + 1 (set (S + 1) % NS) to the other stage
            auto step = [&](auto sc, int kt) {
                constexpr int S = decltype(sc)::value;
                if constexpr (TAIL) {
                    if (kt + 1 == tail_kt) zero_dead(r[(S + 1) % NS]);  // the tile this step writes to LDS
                }
                gload(r[S % NS], min((kt + NS) * BK, k_last_t));
                if constexpr (MA > 0) compute(S & 1, ma);
                lstore((S & 1) ^ 1, r[(S + 1) % NS]);
                if constexpr (MA > 0) interleave(ma);
                __syncthreads();
            };
            for (int kt = 0; kt < nk; kt += UNR) {
                bool more = true;
                static_for<UNR>([&](auto sc) {
                    constexpr int S = decltype(sc)::value;
                    if (more) {
                        step(sc, kt + S);
                        more = kt + S + 1 < nk;
                    }
                });
                if (!more) break;
            }
        };
        const int live = min(MT, max(0, (row_end - row0 - wm * WM + 31) / 32));  // wave-uniform
        static_assert(MT <= 4, "one k_loop instance per count of live 32-row blocks");
        if (live == MT) k_loop(std::integral_constant<int, MT>{});
        else if (live == 0) k_loop(std::integral_constant<int, 0>{});
        else if (live == 1) k_loop(std::integral_constant<int, 1>{});
        else if (live == 2) k_loop(std::integral_constant<int, (MT > 2 ? 2 : 1)>{});
        else k_loop(std::integral_constant<int, (MT > 3 ? 3 : 1)>{});
    }

    // ---- k-groups 1 .. KG-1 hand their sums to group 0 through LDS (every stage is idle now) ------
    if constexpr (KG > 1) {
        constexpr int NACC = MT * NT * 16;
        static_assert(NACC * NTHR * 4 <= 2 * STAGE, "a group's accumulators fit in its own stages");
        float* mine = reinterpret_cast<float*>(gmem) + tid;
        if (kg > 0) {
#pragma unroll
            for (int mi = 0; mi < MT; ++mi)
#pragma unroll
                for (int ni = 0; ni < NT; ++ni)
#pragma unroll
                    for (int i = 0; i < 16; ++i) mine[((mi * NT + ni) * 16 + i) * NTHR] = acc[mi][ni][i];
        }
        __syncthreads();
        if (kg > 0) return;
        for (int q = 1; q < KG; ++q) {
            const float* src = reinterpret_cast<const float*>(smem + q * (2 * STAGE)) + tid;
#pragma unroll
            for (int mi = 0; mi < MT; ++mi)
#pragma unroll
                for (int ni = 0; ni < NT; ++ni)
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[mi][ni][i] += src[((mi * NT + ni) * 16 + i) * NTHR];
        }
    }

    // ---- epilogue: accumulator element i of a 32x32 block sits at row (i/4)*8 + (lane/32)*4 + i%4,
    //      column lane%32 -------------------------------------------------------------------------
    // A block with no rows of the group is skipped.
    bf16_t* const Ct = static_cast<bf16_t*>(second ? g.C1 : g.C) + (size_t)row0 * g.N + n0;  // wave-uniform
    const unsigned ldc = (unsigned)g.N;
    if constexpr (KG == 1) {
        // Through LDS, so that the tile leaves in 16-byte stores (8 per wave and 32 x 64 block)
        // instead of one bf16 per lane and instruction (64 of them).  Each wave stages 32 rows x up
        // to 64 columns at a time in a region of its own (every wave is past the k-loop's last
        // barrier, so the tile stages are free; a wave's LDS operations complete in order, so no
        // further barrier is needed): neighbouring lanes first swap half of their values so that
        // a lane holds two adjacent columns of two rows, written as 32-bit words; then the rows
        // are read back 16 bytes per lane.  Worth 0.5-1 % of a prefill step on the shapes measured.
        constexpr int OC = SWIGLU ? WN / 2 : WN;   // output columns of a wave
        constexpr int PW = OC < 64 ? OC : 64;      // columns staged per pass
        constexpr int NB = PW / 32;
        constexpr int PITCH = PW * 2 + 32;         // bytes per staged row (keeps the four lane groups of a write on distinct banks)
        constexpr int REGION = 32 * PITCH;
        static_assert(REGION * (NTHR / 64) <= 2 * STAGE, "the staging regions fit in the tile stages");
        constexpr int LPR = PW / 8, RPI = 64 / LPR;  // lanes per staged row, rows per read instruction
        char* const region = smem + wave * REGION;
        const bool odd = lane & 1;
        const int wr_row = (lane >> 5) * 4 + (odd ? 2 : 0);
        const int wr_col = (lane & 30) * 2;        // byte offset of the column pair in a 32-column block
        const int rd_row = lane / LPR, rd_chunk = lane % LPR;
#pragma unroll
        for (int mi = 0; mi < MT; ++mi) {
            const int rb = wm * WM + mi * 32;           // the block's first row within the tile
            const int rows_here = row_end - row0 - rb;  // rows of the group from there on (wave-uniform)
            if (rows_here <= 0) continue;
#pragma unroll
            for (int cg = 0; cg < OC / PW; ++cg) {
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    const int ni = cg * NB + nb;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        float o[4];
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            o[j] = acc[mi][ni][q * 4 + j];
                            if (SWIGLU) o[j] = silu_f32(o[j]) * acc[mi][ni + NT / 2][q * 4 + j];
                        }
                        const bf16x2 t01 = {(bf16_t)o[0], (bf16_t)o[1]}, t23 = {(bf16_t)o[2], (bf16_t)o[3]};
                        const unsigned p01 = __builtin_bit_cast(unsigned, t01);  // rows +0, +1 of my column
                        const unsigned p23 = __builtin_bit_cast(unsigned, t23);  // rows +2, +3
                        // even lanes keep rows +0, +1 and get them of the next column; odd lanes keep
                        // rows +2, +3 and get them of the previous column
                        const unsigned keep = odd ? p23 : p01;
                        const unsigned recv = (unsigned)dpp_i32<kDppSwap1>((int)(odd ? p01 : p23));
                        const unsigned lo = odd ? recv : keep, hi = odd ? keep : recv;  // even / odd column
                        char* at = region + (q * 8 + wr_row) * PITCH + nb * 64 + wr_col;
                        *reinterpret_cast<unsigned*>(at) = (lo & 0xffffu) | (hi << 16);
                        *reinterpret_cast<unsigned*>(at + PITCH) = (lo >> 16) | (hi & 0xffff0000u);
                    }
                }
                const int c0 = wn * OC + cg * PW + rd_chunk * 8;  // first of this lane's 8 columns within the tile
#pragma unroll
                for (int it = 0; it < 32 / RPI; ++it) {
                    const int r = it * RPI + rd_row;
                    const uint4 v = *reinterpret_cast<const uint4*>(region + r * PITCH + rd_chunk * 16);
                    if (r < rows_here && n0 + c0 < g.N)
                        *reinterpret_cast<uint4*>(Ct + (unsigned)(rb + r) * ldc + (unsigned)c0) = v;
                }
            }
        }
        return;
    }
    // Kernels with k-groups (small products) store straight from the accumulator layout.  Offsets
    // are 32-bit, relative to the tile's first output (a 64-bit multiply per element costs as much
    // as the SiLU), and a 32-row block that lies wholly inside the group and the matrix stores
    // without per-element predicates.
    const unsigned lane_off = (unsigned)((lane >> 5) * 4) * ldc + (unsigned)(lane & 31);
    const bool cols_inside = n0 + BN_OUT <= g.N;
#pragma unroll
    for (int mi = 0; mi < MT; ++mi) {
        const int rb = wm * WM + mi * 32;             // the block's first row within the tile
        const int rows_here = row_end - row0 - rb;    // rows of the group from there on (wave-uniform)
        if (rows_here <= 0) continue;
#pragma unroll
        for (int ni = 0; ni < (SWIGLU ? NT / 2 : NT); ++ni) {
            const int cb = wn * (SWIGLU ? WN / 2 : WN) + ni * 32;
            const unsigned base = lane_off + (unsigned)rb * ldc + (unsigned)cb;
            if (rows_here >= 32 && cols_inside) {
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    float v = acc[mi][ni][i];
                    if (SWIGLU) v = silu_f32(v) * acc[mi][ni + NT / 2][i];
                    Ct[base + (unsigned)((i >> 2) * 8 + (i & 3)) * ldc] = (bf16_t)v;
                }
            } else {
                const bool col_ok = n0 + cb + (lane & 31) < g.N;
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int rr = (i >> 2) * 8 + (lane >> 5) * 4 + (i & 3);
                    if (rr < rows_here && col_ok) {
                        float v = acc[mi][ni][i];
                        if (SWIGLU) v = silu_f32(v) * acc[mi][ni + NT / 2][i];
                        Ct[base + (unsigned)((i >> 2) * 8 + (i & 3)) * ldc] = (bf16_t)v;
                    }
                }
            }
        }
    }
}

// ============================================================================= host side
template <int BM, int BN, int BK, int WM, int WN, bool SWIGLU, bool DUAL_A, int NS = 2, int KG = 1, bool ADD = false>
static int launch_bf16_deep(GemmArgs& g, hipStream_t st) {
    if ((g.add0 != nullptr) != ADD) return MOE_ERR_INVALID;
    constexpr int BN_OUT = SWIGLU ? BN / 2 : BN;
    constexpr int NTHR = (BM / WM) * (BN / WN) * 64 * KG;
    static_assert(NTHR <= 1024, "workgroup size");
    g.m_tiles_max = m_tiles_bound(g.P, g.E, BM);
    g.n_tiles = (g.N + BN_OUT - 1) / BN_OUT * ((!SWIGLU && g.C1) ? 2 : 1);
    const int total = g.m_tiles_max * g.n_tiles;
    constexpr size_t lds = lds_bytes<BM, BN, BK, DUAL_A, KG>();
    static_assert(lds <= 160 * 1024, "LDS stages exceed the CU's 160 KB");
    const int grid = find_tile_grid(total, split_slots<BM, BN, BK, WM, WN, DUAL_A, KG>());
    bool tail = false;
    for (int i = 0; i < g.nseg; ++i) {
        const int K = g.seg[i].K;  // rows are read in 16-byte chunks; a K tail only without k-groups
        if (K < 8 || K % 8 != 0 || (KG > 1 && K % (BK * KG) != 0)) return MOE_ERR_UNSUPPORTED;
        tail |= K % BK != 0;
    }
    static std::atomic<uint64_t> lds_allowed[2];
    auto launch = [&](auto kern, int which) {
        if (lds > 32 * 1024 &&
            allow_dynamic_lds(reinterpret_cast<const void*>(kern), lds, lds_allowed[which]) != MOE_OK)
            return (int)MOE_ERR_LAUNCH;
        hipLaunchKernelGGL(kern, dim3(grid), dim3(NTHR), lds, st, g);
        return launch_status();
    };
    if constexpr (KG == 1) {
        if (tail) return launch(gemm_bf16_deep_kernel<BM, BN, BK, WM, WN, SWIGLU, DUAL_A, NS, KG, ADD, true>, 1);
    }
    return launch(gemm_bf16_deep_kernel<BM, BN, BK, WM, WN, SWIGLU, DUAL_A, NS, KG, ADD, false>, 0);
}

static int run_gemm(const moe_shape& s, GemmArgs& g, bool swiglu, hipStream_t st) {
    if (g.P == 0) return MOE_OK;
    if (g.add0 && (!g.add1 || !g.row_map || !swiglu || s.act_dtype != MOE_BF16)) return MOE_ERR_INVALID;
    for (int i = 0; g.add0 && i < g.nseg; ++i)
        if (g.seg[i].K % 8 != 0) return MOE_ERR_UNSUPPORTED;  // addends exist only in the deep kernels
    const int n_eff = g.N * (g.C1 ? 2 : 1);  // output columns of the launch
    bool fast = s.act_dtype != MOE_F32;
    for (int i = 0; i < g.nseg; ++i) fast &= g.seg[i].K >= 8 && g.seg[i].K % 8 == 0;  // rows are read in 16-byte chunks
    const bool few = fast && gemm_few_supported(g);
    if (g.k_parts > 1 && !few && !(fast && gemm_pp_supported(g))) return MOE_ERR_UNSUPPORTED;  // (the consumer expects the parts)
    if (g.C1 && !fast) {  // only the bf16 kernels take two products per launch: run them one by one
        GemmArgs second = g;
        second.C = g.C1;
        second.C1 = nullptr;
        for (int i = 0; i < g.nseg; ++i) {
            second.seg[i].A0 = g.seg[i].A1;
            second.seg[i].B0 = g.seg[i].B1;
        }
        g.C1 = nullptr;
        const int rc = run_gemm(s, g, swiglu, st);
        return rc != MOE_OK ? rc : run_gemm(s, second, swiglu, st);
    }
    if (s.act_dtype == MOE_F32) return run_gemm_f32(g, swiglu, st);
    if (few) return run_gemm_few(g, swiglu, st);
    if (fast && gemm_pp_supported(g)) return run_gemm_pp(g, swiglu, st);
    if (fast) {
        // What is left: products with per-token addends, with two segments, with K below 64 or operands of
        // 4 GB and more.  256 x 256 tiles where they fill 256 CUs, else 128 x 128 (two workgroups per CU), 64-row
        // tiles once the groups hold about 128 rows or fewer, and for a plain product with few tiles
        // and a long K two k-groups per workgroup (on 64 x 64 tiles while the groups average 64 rows or
        // less).
        const int n256 = (n_eff + (swiglu ? 127 : 255)) / (swiglu ? 128 : 256);
        const long long big_tiles = (long long)(g.P / 256 + (g.E + 1) / 2) * n256;
        if (g.P >= 384 * g.E && big_tiles >= 400) {
            if (swiglu && g.add0) return launch_bf16_deep<256, 256, 32, 64, 128, true, true, 2, 1, true>(g, st);
            if (swiglu) return launch_bf16_deep<256, 256, 32, 64, 128, true, true>(g, st);
            return launch_bf16_deep<256, 256, 32, 64, 128, false, false>(g, st);
        }
        const bool small_groups = g.P <= 128 * g.E;
        if (swiglu && g.add0)
            return small_groups ? launch_bf16_deep<64, 128, 64, 32, 64, true, true, 2, 1, true>(g, st)
                                : launch_bf16_deep<128, 128, 64, 64, 64, true, true, 2, 1, true>(g, st);
        if (swiglu)
            return small_groups ? launch_bf16_deep<64, 128, 64, 32, 64, true, true>(g, st)
                                : launch_bf16_deep<128, 128, 64, 64, 64, true, true>(g, st);
        const long long tiles128 = (long long)(g.P / 128 + (g.E + 1) / 2) * ((n_eff + 127) / 128);
        bool k_pairs = true;
        for (int i = 0; i < g.nseg; ++i) k_pairs &= g.seg[i].K % 128 == 0;
        if (tiles128 < 160 && k_pairs) {
            if (g.P <= 64 * g.E) return launch_bf16_deep<64, 64, 64, 32, 32, false, false, 2, 2>(g, st);
            return launch_bf16_deep<64, 128, 64, 32, 64, false, false, 2, 2>(g, st);
        }
        return launch_bf16_deep<128, 128, 64, 64, 64, false, false>(g, st);
    }
    return MOE_ERR_UNSUPPORTED;  // bf16 rows that are not whole 16-byte chunks (the entry points reject them)
}

// Parts of the final down projection are sums like any other and kept in fp32, except for tall groups with
// enough 256-row tiles (four parts of each, one per expert at least, make some 220 workgroups) and a long K: there
// they may be rounded to bf16, each like y_perm itself, because twice the traffic costs what the cut saves (fp32
// against bf16 parts, whole layer: 2048 tokens 2048 / 5632 323 us against 311, 777 tokens 1440 / 3840 96.8 against 92.4,
// 2048 tokens 1024 / 2816 107 against 101; below, fp32 parts cost nothing: 8 tokens 2048 / 5632 99.4 against 100.2, up to
// 128 tokens within 1 %).  Rounding errors do not grow with it on independent data (2.3e-3 of the result either
// way), but parts that cancel lose bits that one sum keeps, so the number of bf16 parts is also bounded by the
// one that alone counts full rounds of 256 workgroups (steps of 32 and 12 of fixed cost each).  1: none.
static int bf16_parts_max(long long P, int E, int N, int K) {
    const int n256 = (N + 255) / 256, steps = K / 32;
    const long long tiles = (P / 256 + (E + 1) / 2) * n256;
    if (P <= 24 * E || tiles >= 400 || K % 32 != 0 || K < 2048 || (P / 256 + E) * n256 * 4 < 224) return 1;
    int best = 1;
    long long best_cost = 0;
    for (int q = 2; q <= kMaxParts; ++q) {
        const long long cost = (tiles * q + 255) / 256 * (steps / q + 12);
        if (best == 1 || cost < best_cost) best_cost = cost, best = q;
    }
    return best;
}

// Whether the final down projection may be cut: only where a tile's chain of k-steps is long (and not the
// low-rank term of a shared base, or a product of two segments)
bool down_cut_supported(const moe_shape& s) {
    return s.act_dtype == MOE_BF16 && !(s.flags & MOE_FLAG_SHARED_BASE) && (s.rank > 0 ? s.rank : s.d_ff) > 1024;
}

// Rows that a group can have, for the kernels of few rows: a token meets an expert once
static int few_rows(const moe_shape& s) {
    return s.act_dtype == MOE_BF16 && gemm_few_rows((long long)s.n_tokens * s.top_k, s.top_k) ? s.n_tokens : 0;
}

// Two tokens of dense experts on those kernels (else on the matrix-vector path): where that path would not have
// kept the hidden vectors in fp32 -- from there on it is the slower one, too, unless each token has one expert (us,
// matrix-vector path / this: 2048 / 5632 60.5 / 52.0, 1024 / 2816 26.3 / 24.5, 4 of 16 experts 44.0 / 36.5, 4 of 4 42.6 / 25.2; 1
// of 8 17.3 / 19.7)
bool few_two_tokens(const moe_shape& s) {
    return s.n_tokens == 2 && few_rows(s) && s.rank == 0 && s.top_k > 1 && 2ll * s.top_k * s.d_ff * 4 > 32 * 1024 &&
           s.d_model <= 2048 && down_cut_supported(s) && gemm_few_split(2ll * s.top_k, s.d_model, s.d_ff, 2, kMaxParts);
}

SplitPlan split_plan(const moe_shape& s, size_t down_bytes, size_t rank_bytes) {
    SplitPlan p{1, 1, 1, true};
    if (s.act_dtype != MOE_BF16 || s.n_tokens == 0) return p;
    const long long P = (long long)s.n_tokens * s.top_k;
    const bool base = s.flags & MOE_FLAG_SHARED_BASE, token_base = token_base_supported(s);
    const bool few = few_rows(s) > 0;
    auto at_most = [](int parts, size_t room, long long out_bytes) {
        return (long long)room < parts * out_bytes ? (int)((long long)room / out_bytes) : parts;
    };
    if (down_cut_supported(s)) {
        const int K = s.rank > 0 ? s.rank : s.d_ff;
        const int bf16_max = bf16_parts_max(P, s.n_experts, s.d_model, K);
        p.down_f32 = bf16_max == 1;
        p.down = few ? gemm_few_split(P, s.d_model, K, 2, at_most(kMaxParts, down_bytes, P * s.d_model * 4)) : 0;  // (in fp32: cut)
        if (p.down) p.down_f32 = true;
        else p.down = gemm_pp_split(P, s.n_experts, s.d_model, K,
                                    at_most(p.down_f32 ? kMaxParts : bf16_max, down_bytes, P * s.d_model * (p.down_f32 ? 4 : 2)),
                                    p.down_f32, false);
    }
    if (s.rank > 0 && (!base || token_base)) {
        const int room = at_most(kMaxParts, rank_bytes, P * s.rank * 4);
        p.rank_down = few ? gemm_few_split(P, s.rank, s.d_ff, 1, room) : 0;
        if (!p.rank_down) p.rank_down = gemm_pp_split(P, s.n_experts, s.rank, s.d_ff, room, true, true);
    }
    if (token_base) {
        const FfnLayout l = ffn_layout(s);  // its parts lie in what h .. bu held
        const int room = at_most(kMaxParts, l.end - l.h, (long long)s.n_tokens * s.d_model * 4);
        p.base_down = few ? gemm_few_split(s.n_tokens, s.d_model, s.d_ff, 2, room) : 0;
        if (!p.base_down) p.base_down = gemm_pp_split(s.n_tokens, 1, s.d_model, s.d_ff, room, true, false);
    }
    return p;
}

// The per-token treatment of a shared base needs the deep bf16 kernels (every K a multiple of 8,
// which the shape check of the entry points already demands) and pays only when a token has more
// than one expert.
bool token_base_supported(const moe_shape& s) {
    return (s.flags & MOE_FLAG_SHARED_BASE) && s.rank > 0 && s.top_k > 1 && s.act_dtype == MOE_BF16 &&
           s.d_model % 8 == 0 && s.d_ff % 8 == 0 && s.rank % 8 == 0;
}

FfnLayout ffn_layout(const moe_shape& s) {
    const size_t P = (size_t)s.n_tokens * s.top_k, es = elt_size(s.act_dtype);
    const size_t rank = round_up(P * s.rank * es, 256), hidden = round_up(P * s.d_ff * es, 256);
    const size_t base = token_base_supported(s) ? round_up((size_t)s.n_tokens * s.d_ff * es, 256) : 0;
    FfnLayout l;
    l.td = 0;
    l.z = l.td + rank;
    l.h = l.z + base;
    l.tg = l.h + hidden;
    l.tu = l.tg + rank;
    l.bg = l.tu + rank;
    l.bu = l.bg + base;
    l.end = l.bu + base;
    return l;
}

// Whether the layer's first product can sort the pairs by expert itself (GemmArgs::keys)
bool ffn_takes_keys(const moe_shape& s, const int32_t* keys) {
    const int P = s.n_tokens * s.top_k, E = s.n_experts;
    if (!aligned16(keys)) return false;
    if (s.act_dtype == MOE_F32) return dispatch_in_product(P, kF32DispatchThreads);
    GemmArgs g{};
    g.P = P; g.E = E; g.row_div = s.top_k; g.N = s.rank > 0 ? s.rank : s.d_ff; g.nseg = 1;
    g.seg[0].K = s.d_model; g.seg[0].gather = 1;
    return dispatch_in_product(P, kPpThreads) && gemm_pp_supported(g);
}

// td = h R_d^T, a product with few tiles and a long K: in parts that a kernel of its own adds, if the plan says so
static int run_rank_down(const moe_shape& s, GemmArgs& g, const SplitPlan* plan, float* parts, hipStream_t st) {
    if (plan && plan->rank_down > 1) {
        g.k_parts = plan->rank_down;
        g.parts_f32 = 1;
        g.parts = parts;
    }
    const int rc = run_gemm(s, g, false, st);
    if (rc != MOE_OK || g.k_parts <= 1) return rc;
    return launch_sum_parts(parts, g.k_parts, (long long)g.P * g.N, g.C, st);
}

int launch_expert_ffn(const moe_shape& s, const moe_weights& w, const void* x,
                      int32_t* a_row_map, int a_row_div, int32_t* offsets,
                      void* y_perm, void* scratch, hipStream_t st, StageTimer* timer, const SplitPlan* plan,
                      const int32_t* keys, int32_t* inv_perm) {
    const int d = s.d_model, F = s.d_ff, r = s.rank, E = s.n_experts;
    const int P = s.n_tokens * s.top_k;
    if (P == 0) return MOE_OK;
    const FfnScratch f = ffn_scratch(s, scratch);
    void *h = f.h, *tg = f.tg, *tu = f.tu, *td = f.td;
    const bool base = (r == 0) || (s.flags & MOE_FLAG_SHARED_BASE);
    const int gather = a_row_map ? 1 : 0;
    int rc;
    auto fresh = [&]() {
        GemmArgs g{};
        g.offsets = offsets; g.row_map = a_row_map; g.row_div = a_row_div > 0 ? a_row_div : 1;
        g.E = E; g.P = P;
        g.few = few_rows(s);
        return g;
    };
    if (r > 0) {  // tg = x R_g^T, tu = x R_u^T   [P, r], both in one launch
        GemmArgs g = fresh();
        g.nseg = 1; g.N = r; g.C = tg; g.C1 = tu;
        g.seg[0] = GemmSeg{x, x, w.rg, w.ru, (long long)r * d, d, gather};
        g.keys = keys; g.inv_perm = inv_perm;
        if ((rc = run_gemm(s, g, false, st)) != MOE_OK) return rc;
        stage_mark(timer, "gemm_rank_gate_up");
    }
    {  // h = silu(M_gate x) * (M_up x)   [P, F]
        GemmArgs g = fresh();
        int ns = 0;
        if (base) g.seg[ns++] = GemmSeg{x, x, w.w_gate, w.w_up, r == 0 ? (long long)F * d : 0, d, gather};
        if (r > 0) g.seg[ns++] = GemmSeg{tg, tu, w.lg, w.lu, (long long)F * r, r, 0};
        g.nseg = ns; g.N = F; g.C = h;
        if (r == 0) g.keys = keys, g.inv_perm = inv_perm;
        if ((rc = run_gemm(s, g, true, st)) != MOE_OK) return rc;
        stage_mark(timer, "gemm_gate_up_swiglu");
    }
    if (r > 0) {  // td = h R_d^T   [P, r]
        GemmArgs g = fresh();
        g.nseg = 1; g.N = r; g.C = td; g.hidden_a = 1;
        g.seg[0] = GemmSeg{h, h, w.rd, w.rd, (long long)r * F, F, 0};
        if ((rc = run_rank_down(s, g, plan, f.rank_parts, st)) != MOE_OK) return rc;
        stage_mark(timer, "gemm_rank_down");
    }
    {  // y_perm = M_down h   [P, d]
        GemmArgs g = fresh();
        int ns = 0;
        if (base) g.seg[ns++] = GemmSeg{h, h, w.w_down, w.w_down, r == 0 ? (long long)d * F : 0, F, 0};
        if (r > 0) g.seg[ns++] = GemmSeg{td, td, w.ld, w.ld, (long long)d * r, r, 0};
        g.nseg = ns; g.N = d; g.C = y_perm; g.hidden_a = 1;
        if (plan) {
            g.k_parts = plan->down;
            g.parts_f32 = plan->down_f32;
            g.parts = y_perm;
        }
        if ((rc = run_gemm(s, g, false, st)) != MOE_OK) return rc;
        stage_mark(timer, "gemm_down");
    }
    return MOE_OK;
}

// M_e = M0 + L_e R_e with M0 shared by all experts.  Per token t with experts e_j and gates g_j:
//   gate/up:  M0 x_t is the same for every j, so it is computed once per token (a plain product
//             over T rows) and added, per pair, to the low-rank term in the SwiGLU epilogue;
//   down:     sum_j g_j M0 h_tj = M0 (sum_j g_j h_tj): the shared matrix meets the gate-mixed
//             hidden vector once per token; the low-rank terms stay per pair and are mixed by
//             the combine, which also adds the shared part.
// This halves the base work at k = 2 (6 T d F flops instead of 6 P d F).
int launch_expert_ffn_token_base(const moe_shape& s, const moe_weights& w, const void* x,
                                 int32_t* perm, int32_t* inv_perm, const float* topk_gate,
                                 int32_t* offsets, void* y_perm, void* y_base, void* scratch,
                                 hipStream_t st, StageTimer* timer, const SplitPlan& plan, const int32_t* keys) {
    const int d = s.d_model, F = s.d_ff, r = s.rank, E = s.n_experts, T = s.n_tokens;
    const int P = T * s.top_k;
    if (P == 0) return MOE_OK;
    const FfnScratch f = ffn_scratch(s, scratch);
    void *h = f.h, *tg = f.tg, *tu = f.tu, *td = f.td, *bg = f.bg, *bu = f.bu, *z = f.z;
    int rc;
    auto grouped = [&]() {  // rows = pairs in expert order
        GemmArgs g{};
        g.offsets = offsets; g.row_map = perm; g.row_div = s.top_k; g.E = E; g.P = P;
        g.few = few_rows(s);
        return g;
    };
    auto per_token = [&]() {  // rows = tokens, one group, one matrix
        GemmArgs g{};
        g.offsets = nullptr; g.row_map = nullptr; g.row_div = 1; g.E = 1; g.P = T;
        g.few = few_rows(s);
        return g;
    };
    {  // tg = x R_g^T, tu = x R_u^T   [P, r]
        GemmArgs g = grouped();
        g.nseg = 1; g.N = r; g.C = tg; g.C1 = tu;
        g.seg[0] = GemmSeg{x, x, w.rg, w.ru, (long long)r * d, d, 1};
        g.keys = keys; g.inv_perm = inv_perm;
        if ((rc = run_gemm(s, g, false, st)) != MOE_OK) return rc;
        stage_mark(timer, "gemm_rank_gate_up");
    }
    {  // bg = x M0_gate^T, bu = x M0_up^T   [T, F]
        GemmArgs g = per_token();
        g.nseg = 1; g.N = F; g.C = bg; g.C1 = bu;
        g.seg[0] = GemmSeg{x, x, w.w_gate, w.w_up, 0, d, 0};
        if ((rc = run_gemm(s, g, false, st)) != MOE_OK) return rc;
        stage_mark(timer, "gemm_base_gate_up");
    }
    {  // h = silu(bg[t] + tg L_g^T) * (bu[t] + tu L_u^T)   [P, F]
        GemmArgs g = grouped();
        g.nseg = 1; g.N = F; g.C = h; g.add0 = bg; g.add1 = bu;
        g.seg[0] = GemmSeg{tg, tu, w.lg, w.lu, (long long)F * r, r, 0};
        if ((rc = run_gemm(s, g, true, st)) != MOE_OK) return rc;
        stage_mark(timer, "gemm_gate_up_swiglu");
    }
    {  // td = h R_d^T   [P, r]
        GemmArgs g = grouped();
        g.nseg = 1; g.N = r; g.C = td; g.hidden_a = 1;
        g.seg[0] = GemmSeg{h, h, w.rd, w.rd, (long long)r * F, F, 0};
        if ((rc = run_rank_down(s, g, &plan, f.rank_parts, st)) != MOE_OK) return rc;
        stage_mark(timer, "gemm_rank_down");
    }
    {  // z[t] = sum_j g_tj h[slot(t, j)]   [T, F]
        moe_shape sm = s;
        sm.d_model = F;
        if ((rc = launch_combine(sm, h, inv_perm, topk_gate, nullptr, z, st)) != MOE_OK) return rc;
        stage_mark(timer, "mix_hidden");
    }
    {  // y_base = z M0_down^T   [T, d]
        GemmArgs g = per_token();
        g.nseg = 1; g.N = d; g.C = y_base; g.hidden_a = 1;
        g.seg[0] = GemmSeg{z, z, w.w_down, w.w_down, 0, F, 0};
        if (plan.base_down > 1) {  // parts for the combine to add
            g.k_parts = plan.base_down;
            g.parts_f32 = 1;
            g.parts = f.base_parts;
        }
        if ((rc = run_gemm(s, g, false, st)) != MOE_OK) return rc;
        stage_mark(timer, "gemm_base_down");
    }
    {  // y_perm = td L_d^T   [P, d]
        GemmArgs g = grouped();
        g.nseg = 1; g.N = d; g.C = y_perm;
        g.seg[0] = GemmSeg{td, td, w.ld, w.ld, (long long)d * r, r, 0};
        if ((rc = run_gemm(s, g, false, st)) != MOE_OK) return rc;
        stage_mark(timer, "gemm_down");
    }
    return MOE_OK;
}

}  // namespace moe
