// What the grouped GEMM kernels share: the problem description, and the mapping of workgroups to tiles.
//
// One generic problem:   C[s, n] = epi( sum_seg  A_seg[row(s), :] . B_seg[e(s)][n, :] )
//   PLAIN   one accumulator, C = acc
//   SWIGLU  two accumulators over (A0,B0) and (A1,B1); C = silu(acc0) * acc1
// A and B are both K-contiguous ("NT" GEMM), the natural layout of activations [rows, in]
// and linear-layer weights [out, in].
#pragma once

#include <type_traits>
#include <utility>

#include "common.h"

namespace moe {

template <int... I, typename F>
__device__ __forceinline__ void static_for_impl(std::integer_sequence<int, I...>, F&& f) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
    static_for_impl(std::make_integer_sequence<int, N>{}, static_cast<F&&>(f));
}

struct GemmSeg {
    const void* A0;     // [*, K]
    const void* A1;     // A of the second accumulator (SWIGLU); may equal A0
    const void* B0;     // [Eb, N, K]
    const void* B1;
    long long strideB;  // elements between experts; 0 = shared by all experts
    int K;
    int gather;         // 1: the A row of sorted slot s is row_map[s] / row_div
};

struct GemmArgs {
    GemmSeg seg[2];
    int nseg;
    void* C;            // [P, N]
    void* C1;           // PLAIN only, bf16 kernels: second product (A1 . B1) of the same shape, or NULL
    int N;
    int32_t* offsets;        // [E+1]
    int32_t* row_map;        // [P] or NULL
    int row_div;
    int E;
    int P;
    int m_tiles_max;
    int n_tiles;        // n-tiles of the launch (twice those of one product when C1 is set)
    // SWIGLU, gemm_bf16_deep_kernel: per-token rows added to the two accumulators before the activation
    // (the token of sorted slot s is row_map[s] / row_div), [*, N] in the activation type, or NULL
    const void* add0;
    const void* add1;
    int hidden_a;       // the activation operand is the F-wide hidden tensor (tile order: kHiddenOperandBlock)
    // PLAIN, one segment, expert_gemm_pp.hip: the k-steps of every tile are cut into k_parts consecutive
    // ranges, each computed by a workgroup of its own and stored to its own output [P, N] (part q at
    // parts + q * P * N elements, fp32 if parts_f32, else the activation type), to be added by the
    // consumer.  0 or 1: one output, in C.
    int k_parts;
    int parts_f32;
    void* parts;
    // expert_gemm_pp.hip: where the launch is at most this many rounds of 256 workgroups, the tiles are made
    // narrower until they fill the last round (decided on the device, where the m-tiles are known)
    int fit_width;
    // Dispatch in the first product of a layer (expert_gemm_pp.hip, expert_gemm_f32.hip): keys [P] are the pairs'
    // experts; offsets, row_map and inv_perm [P] are then outputs of the launch, as moe_permute states
    // them, and its own rows are found from the keys.  NULL: offsets and row_map are inputs.
    const int32_t* keys;
    int32_t* inv_perm;
    // expert_gemm_few.hip: no group holds more rows than this (a speed matter only).  0: not known
    int few;
};

// Products whose activation operand is the F-wide hidden tensor (down, rank-down): that operand is
// as large as an expert's weights, so tiles are ordered in blocks of this many n-tiles with the
// expert's m-tiles inside a block -- the workgroups in flight on an XCD then share a few A tiles
// and a few B tiles instead of one B tile and every A tile (measured on the phone shape with
// Zipf loads: down product 145 us with blocks of 8 or 16, 148 with 4, 153-157 with n-tile outer).
constexpr int kHiddenOperandBlock = 8;

// Group e's row range; offsets == NULL means one group holding all P rows (a plain product).
__device__ __forceinline__ int group_begin(const int32_t* __restrict__ offsets, int e) {
    return offsets ? offsets[e] : 0;
}
__device__ __forceinline__ int group_end(const int32_t* __restrict__ offsets, int e, int P) {
    return offsets ? offsets[e + 1] : P;
}

// Workgroup -> output tile.  Tiles are ordered expert-major, then n-tile, then the expert's
// own m-tiles, so neighbouring tiles share the expert's activation rows (and, for equal
// n-tile, its weight tile).  Workgroups are handed to the 8 XCDs round-robin by id; XCD x
// takes the x-th contiguous eighth of that order, which keeps each XCD's L2 working set to
// about one expert's rows plus the weight tiles it is streaming.  The grid is an upper
// bound (group sizes live on the device); surplus workgroups return false.
//
// Tail split: an XCD runs split_slots workgroups at a time, so its tiles take
// ceil(tiles / split_slots) rounds and the last round may be nearly empty.  When there is at
// least one full round and the last one holds at most split_slots / 2 tiles, each of those is
// cut into an upper and a lower half (BM / 2 rows) handled by two workgroups: the halves still
// fit in one round and each is shorter than a whole tile (it fills half the activation rows
// and multiplies half the blocks).
//
// n_tiles_of(m): the launch's n-tiles when all groups together have m m-tiles.
// lo, hi: in lane e of every wave, group e's bounds (group_bounds; 0, 0 in lanes from E on).  The sums over groups
// are a scan over the lanes.  (A loop of dependent scalar loads over the offsets cost
// 2.6-3.3 us per tile here, a twentieth of a 256 x 256 tile's duration.)
__device__ __forceinline__ void group_bounds(const int32_t* __restrict__ offsets, int E, int P, int& lo, int& hi) {
    const int lane = threadIdx.x & (kWave - 1);
    lo = hi = 0;
    if (lane < E) {
        lo = group_begin(offsets, lane);
        hi = group_end(offsets, lane, P);
    }
}
// The tile, of `total`, that workgroup `block` takes, and the half of it (-1: all of it); none: false
template <int SPLIT_SLOTS>
__host__ __device__ __forceinline__ bool tile_of_block(unsigned block, int total, int& tile, int& half) {
    const int per_xcd = (total + 7) / 8;
    const int slot = block >> 3;
    const int first = (block & 7) * per_xcd;                    // this XCD's first tile
    const int mine = max(0, min(per_xcd, total - first));       // and how many it has
    int local_tile = slot;
    half = -1;
    if (SPLIT_SLOTS > 0) {
        constexpr int SLOTS = SPLIT_SLOTS > 0 ? SPLIT_SLOTS : 1;
        const int whole = (mine / SLOTS) * SLOTS;               // tiles in full rounds
        const int rem = mine - whole;
        if (whole > 0 && rem > 0 && 2 * rem <= SLOTS && slot >= whole) {
            const int idx = slot - whole;
            local_tile = whole + idx / 2;
            half = idx & 1;
        }
    }
    if (local_tile >= mine) return false;
    tile = first + local_tile;
    return true;
}
// GemmArgs::fit_width: where m_all row tiles (of all products or k-parts) by n_base column tiles are at most that many rounds of
// 256 workgroups, the columns of a tile and the tiles across N become those that fill the last of them
__host__ __device__ __forceinline__ void fit_columns(int m_all, int N, int fit_width, int& width, int& n_base) {
    const int rounds = (int)((unsigned)(m_all * n_base + 255) / 256u);
    if (rounds > fit_width) return;
    const int n = uniform_div(256 * rounds, m_all);  // tiles across N that fit
    width = max(8, (uniform_div(N + n - 1, n) + 7) / 8 * 8);
    n_base = uniform_div(N + width - 1, width);
}
// Tiles that a launch of up to `tiles` of them can come to have by that
inline int fitted_tiles(int tiles, int fit_width) { return tiles < 256 * fit_width ? (tiles + 255) / 256 * 256 : tiles; }
// N_INNER (a power of two): tile order inside an expert in blocks of this many n-tiles, block outer, the
// expert's m-tiles in the middle, the block's n-tiles inner (1: n-tile outer, m-tiles inner).
template <int N_INNER = 1, int SPLIT_SLOTS = 0, typename NTiles>
__device__ __forceinline__ bool find_tile(int lo, int hi, int E, int BM, NTiles n_tiles_of, int& e_out,
                                          int& row0, int& row_end, int& nt_out) {
    const int lane = threadIdx.x & (kWave - 1);
    const int cnt = (hi - lo + BM - 1) / BM;  // m-tiles of group `lane` (0 beyond E)
    const int upto = wave_scan(cnt), before = upto - cnt;  // m-tiles of the groups up to and below `lane`
    int total = MOE_READLANE(upto, kWave - 1);
    const int n_tiles = n_tiles_of(total);
    total *= n_tiles;
    int L, half;
    if (!tile_of_block<SPLIT_SLOTS>(blockIdx.x, total, L, half)) return false;
    // the group whose tiles hold L: the last one with tiles at or before it
    const unsigned long long at = __ballot(lane < E && cnt > 0 && before * n_tiles <= L);
    const int e = 63 - __clzll((long long)at);
    const int mtiles = MOE_READLANE(cnt, e), prev = MOE_READLANE(lo, e), next = MOE_READLANE(hi, e);
    const int local = L - MOE_READLANE(before, e) * n_tiles;
    const int full = (n_tiles / N_INNER) * N_INNER * mtiles;  // tiles in whole blocks
    int mt, nt;
    if (local < full) {
        const int block = uniform_div(local, mtiles * N_INNER);
        const int rem = local - block * (mtiles * N_INNER);
        mt = rem / N_INNER;
        nt = block * N_INNER + rem % N_INNER;
        if (N_INNER == 1) mt = rem, nt = block;
    } else {
        const int nb_tail = n_tiles % N_INNER;
        const int rem = local - full;
        mt = uniform_div(rem, nb_tail);
        nt = (n_tiles / N_INNER) * N_INNER + rem - mt * nb_tail;
    }
    e_out = e;
    nt_out = nt;
    row0 = prev + mt * BM;
    row_end = next;
    if (half >= 0) {
        row0 += half * (BM / 2);
        row_end = min(next, row0 + BM / 2);
        if (row0 >= row_end) return false;  // the tile had no rows in its lower half
    }
    return true;
}

// Tiles of BM rows that P rows in E groups can need at most: a group of r rows takes 1 + (r - 1) / BM, an empty one none
inline int m_tiles_bound(int P, int E, int BM) {
    const int groups = P < E ? P : E;
    return groups + (P - groups) / BM;
}
// Workgroups for up to `tiles` tiles on find_tile<., split_slots>.  A last round cut into halves fills a round at most, so a launch
// needs no more than whole rounds, and none beside the tiles where they are one.  A surplus workgroup is not free: it finds the
// bounds before it leaves, and with all of a CU's LDS to its name it starts only when a tile has ended: 256 of them are 1.1 us at a
// launch's end.  Whole layer, us, with P / BM + E row tiles and half a round beside them / by this rule: 64 tokens of 1024 / 2816
// 36.7 / 35.5, 300 tokens 47.0 / 46.1, 512 tokens 51.4 / 48.8, 777 tokens of 1440 / 3840 90.3 / 88.9.
inline int find_tile_grid(int tiles, int split_slots) {
    const int per_xcd = (tiles + 7) / 8;
    if (split_slots == 0 || per_xcd <= split_slots) return per_xcd * 8;
    const int rounds = (per_xcd + split_slots - 1) / split_slots * split_slots, halves = per_xcd + split_slots / 2;
    return (rounds < halves ? rounds : halves) * 8;
}

// ---- dispatch inside a product -----------------------------------------------------------------------------
// The pairs of a layer are sorted by expert (stable) so that each expert's rows are one group.  For up to a
// few thousand pairs a workgroup finds what it needs of that from the P keys itself -- the groups' bounds
// and the pairs of its own tile's rows -- and a launch of 5-11 us that does nothing else is saved for 1-6 us
// more of the product (measured, layer of 300 tokens, 432 x 1152: 31.3 -> 27.4 us; 2048 tokens, 432 x 1152:
// 47.3 -> 41.6; 777 tokens, 1440 x 3840: 98.3 -> 93.5; 4096 tokens, 720 x 1920: 123.5 -> 116.0).  Every tile
// counts again: at 2048 tokens, 2048 x 5632, three rounds of tiles, it is even (310 us), so the line lies at the
// keys that the threads of one workgroup hold.  A thread holds neighbouring keys, as many as another (a multiple of 4), so that order by
// thread is order by pair.
constexpr int kKeyChunks = 4;
__device__ __forceinline__ int lanes_below(unsigned long long mask) {  // set bits of mask below this lane
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
#else
    return 0;
#endif
}
template <int NTHR>
struct PairKeys {
    int k[kKeyChunks][4];
    int chunks;  // of 4 keys, of every thread (wave-uniform)

    __device__ __forceinline__ int pair(int c) const { return ((int)threadIdx.x * chunks + c) * 4; }  // of k[c][0]

    __device__ __forceinline__ void load(const int32_t* __restrict__ keys, int P) {
        chunks = (P + 4 * NTHR - 1) / (4 * NTHR);
#pragma unroll
        for (int c = 0; c < kKeyChunks; ++c) {
            const int p = pair(c);
            int4 v = make_int4(-1, -1, -1, -1);
            if (c < chunks) {
                if (p + 3 < P) {
                    v = *reinterpret_cast<const int4*>(keys + p);
                } else {
                    if (p < P) v.x = keys[p];
                    if (p + 1 < P) v.y = keys[p + 1];
                    if (p + 2 < P) v.z = keys[p + 2];
                }
            }
            k[c][0] = v.x, k[c][1] = v.y, k[c][2] = v.z, k[c][3] = v.w;
        }
    }

    // Lane e: keys of the wave that are expert e, e < 8.  Counted per lane in the eight bytes of a word (16 keys at most), then
    // summed over the wave in fields of 16 bits, four registers of two.
    __device__ __forceinline__ int count_eight() const {
        unsigned lo = 0, hi = 0;
#pragma unroll
        for (int c = 0; c < kKeyChunks; ++c) {
            if (c >= chunks) break;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const unsigned f = (unsigned)k[c][j], one = 1u << (f * 8 & 31);
                lo += f < 4 ? one : 0;
                hi += f - 4 < 4 ? one : 0;
            }
        }
        const int lane = threadIdx.x & (kWave - 1);
        auto sum = [&](unsigned v) {  // of a 16-bit field over the wave
            int s = (int)v;
            s += dpp_i32<kDppSwap1>(s);
            s += dpp_i32<kDppSwap2>(s);
            s += dpp_i32<kDppHalfMirror>(s);
            s += dpp_i32<kDppMirror>(s);
            return (MOE_READLANE(s, 0) + MOE_READLANE(s, 16)) + (MOE_READLANE(s, 32) + MOE_READLANE(s, 48));
        };
        const int lo02 = sum(lo & 0x00ff00ffu), lo13 = sum(lo >> 8 & 0x00ff00ffu), hi02 = sum(hi & 0x00ff00ffu), hi13 = sum(hi >> 8 & 0x00ff00ffu);
        const int both = lane & 1 ? (lane & 4 ? hi13 : lo13) : (lane & 4 ? hi02 : lo02);
        return lane & 2 ? (int)((unsigned)both >> 16) : both & 0xffff;
    }

    // group bounds in lane e of every wave (as group_bounds); s_count [waves][kMaxExperts] receives every wave's count of every
    // expert.  Where a thread holds more than four keys (from 2049 pairs on with 512 threads, from 1025 on with 256), up to 8 experts, the lanes' counts are
    // added up in registers: LDS atomics meet on few addresses, and the
    // more where experts are chosen unevenly (4096 skewed pairs of 8 experts 2500 clocks, 1650 now; 16 experts even 2048 tokens of 1024 / 2816 188.9 / 191.6).
    // Below, atomics without a branch: 2400 clocks of 1024 pairs, 1040 now.  With the sums over lanes in find_tile and here, and all arguments
    // in one place (expert_gemm_pp.hip), a tile's way to its first fill went from 5650 to 4050 clocks there, from 7260 to 3880 at 4096 pairs; whole layer, us,
    // before / now: 300 tokens of 432 / 1152 26.1 / 24.6, 512 tokens of 1024 / 2816 53.1 / 51.6, 64 tokens, 4 of 16 experts, 66.2 / 61.5, 200
    // tokens of 2048 / 5632 121.4 / 119.3, 777 tokens of 1440 / 3840 92.4 / 90.4, 2048 skewed tokens of 432 / 1152 46.4 / 40.6, 4096 tokens of
    // 1024 / 2816 178.3 / 174.0, 2048 tokens of 2048 / 5632 308.9 / 306.7 (the power limit).
    __device__ __forceinline__ void bounds(int E, int (*s_count)[kMaxExperts], int& lo, int& hi) const {
        constexpr int NW = NTHR / kWave;
        const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
        int* const count = s_count[wave];
        if (E <= 8 && chunks > 1) {
            count[lane] = count_eight();  // (lanes from E on: not read)
        } else {
            count[lane] = 0;  // (a wave's LDS operations complete in order)
#pragma unroll
            for (int c = 0; c < kKeyChunks; ++c) {
                if (c >= chunks) break;
#pragma unroll
                for (int j = 0; j < 4; ++j) {  // (no key: nothing, to an address of the lane's own)
                    const bool is = (unsigned)k[c][j] < (unsigned)E;
                    atomicAdd(&count[is ? k[c][j] : lane], is ? 1 : 0);
                }
            }
        }
        __syncthreads();
        int total = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) total += s_count[w][lane];
        total = lane < E ? total : 0;
        hi = wave_scan(total);
        lo = hi - total;
    }

    // pairs of rows [first, first + n) of expert e's group (counted from its start) to s_pair[0 .. n), n <= room; what is not asked for goes to
    // s_pair[room .. room + 64), an address per lane, with no branch around a write.  (Behind a wave's fills straight into LDS its LDS operations
    // wait: 3000 clocks of a tile here, 1200 with the fills behind; the fills came first all the same, as the weights are what a tile waits for: whole layer
    // 0.7 % faster in the geometric mean of 15.)
    __device__ __forceinline__ void rows(int e, int first, int n, int room, const int (*s_count)[kMaxExperts], int* s_pair) const {
        constexpr int NW = NTHR / kWave;
        const int wave = threadIdx.x / kWave;
        int at = -first, mine = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const int before = s_count[w][e];
            at += w < wave ? before : 0;
        }
#pragma unroll
        for (int c = 0; c < kKeyChunks; ++c) {
            if (c >= chunks) break;
#pragma unroll
            for (int j = 0; j < 4; ++j) mine += k[c][j] == e ? 1 : 0;
        }
#pragma unroll
        for (int b = 0; b < 5; ++b) {  // 4 chunks at most
            if (b == 3 && chunks == 1) break;
            at += lanes_below(__ballot(mine >> b & 1)) << b;
        }
#pragma unroll
        for (int c = 0; c < kKeyChunks; ++c) {
            if (c >= chunks) break;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool is = k[c][j] == e;
                s_pair[is && (unsigned)at < (unsigned)n ? at : room + ((int)threadIdx.x & (kWave - 1))] = pair(c) + j;
                at += is ? 1 : 0;
            }
        }
        __syncthreads();
    }
};
inline bool dispatch_in_product(int P, int threads) { return P <= kKeyChunks * 4 * threads; }

// fp32 problems (expert_gemm_f32.hip)
constexpr int kF32DispatchThreads = 256;  // threads of its workgroups
int run_gemm_f32(GemmArgs& g, bool swiglu, hipStream_t st);
// bf16 products, fills straight into LDS (expert_gemm_pp.hip)
constexpr int kPpThreads = 512;
bool gemm_pp_supported(const GemmArgs& g);
int run_gemm_pp(GemmArgs& g, bool swiglu, hipStream_t st);
// Parts, up to parts_max, into which it is worth cutting the k-steps of a plain product of P rows in E groups
// (k_parts above)
int gemm_pp_split(long long P, int E, int N, int K, int parts_max, bool parts_f32, bool sum_launch);
// bf16 products of few rows per group (expert_gemm_few.hip)
bool gemm_few_rows(long long P, int top_k);
// Parts of K, at least parts_min, in which these kernels take a plain product of P rows, or 0 if that is more than parts_max
// or they do not take it
int gemm_few_split(long long P, int N, int K, int parts_min, int parts_max);
bool gemm_few_supported(const GemmArgs& g);
int run_gemm_few(const GemmArgs& g, bool swiglu, hipStream_t st);
int launch_sum_parts(const float* parts, int q, long long n, void* out, hipStream_t st);

}  // namespace moe
