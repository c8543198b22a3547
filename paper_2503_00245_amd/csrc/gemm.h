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
    void* C1;           // PLAIN only, deep kernel: second product (A1 . B1) of the same shape, or NULL
    int N;
    const int32_t* offsets;  // [E+1]
    const int32_t* row_map;  // [P] or NULL
    int row_div;
    int E;
    int P;
    int m_tiles_max;
    int n_tiles;        // n-tiles of the launch (twice those of one product when C1 is set)
    // SWIGLU, deep kernel: per-token rows added to the two accumulators before the activation
    // (the token of sorted slot s is row_map[s] / row_div), [*, N] in the activation type, or NULL
    const void* add0;
    const void* add1;
    int n_inner;        // tile order inside an expert: blocks of this many n-tiles (0 or 1: n-tile outer, m-tiles inner)
    int split_slots;    // workgroups one XCD runs at a time; > 0: the tiles of its last, partial round are cut
                        // into upper and lower halves when both halves still fit in one round (set by the launcher)
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
};

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
template <typename NTiles>
__device__ __forceinline__ bool find_tile(const int32_t* __restrict__ offsets, int E, int P, int BM,
                                          NTiles n_tiles_of, int& e_out, int& row0, int& row_end,
                                          int& nt_out, int n_inner = 0, int split_slots = 0) {
#if defined(__HIP_DEVICE_COMPILE__)
    // Lane e of every wave fetches group e's bounds with ONE vector load (E <= 64); the sums below
    // then run on scalar registers through readlane.  (A loop of dependent scalar loads over the
    // offsets cost 2.6-3.3 us per tile here, a twentieth of a tile's whole duration.)
    const int lane = threadIdx.x & (kWave - 1);
    int lo = 0, hi = 0;
    if (lane < E) {
        lo = group_begin(offsets, lane);
        hi = group_end(offsets, lane, P);
    }
    const int cnt = (hi - lo + BM - 1) / BM;  // m-tiles of group `lane` (0 beyond E)
    int total = 0;
    for (int e = 0; e < E; ++e) total += __builtin_amdgcn_readlane(cnt, e);
#else
    int total = 0;
    for (int e = 0; e < E; ++e)
        total += (group_end(offsets, e, P) - group_begin(offsets, e) + BM - 1) / BM;
#endif
    const int n_tiles = n_tiles_of(total);
    total *= n_tiles;
    const int per_xcd = (total + 7) / 8;
    const int slot = blockIdx.x >> 3;
    const int first = (blockIdx.x & 7) * per_xcd;               // this XCD's first tile
    const int mine = max(0, min(per_xcd, total - first));       // and how many it has
    int local_tile = slot, half = -1;
    if (split_slots > 0) {
        const int whole = (mine / split_slots) * split_slots;   // tiles in full rounds
        const int rem = mine - whole;
        if (whole > 0 && rem > 0 && 2 * rem <= split_slots && slot >= whole) {
            const int idx = slot - whole;
            local_tile = whole + idx / 2;
            half = idx & 1;
        }
    }
    if (local_tile >= mine) return false;
    const int L = first + local_tile;
    int before = 0;
    for (int e = 0; e < E; ++e) {
#if defined(__HIP_DEVICE_COMPILE__)
        const int mtiles = __builtin_amdgcn_readlane(cnt, e);
#else
        const int mtiles = (group_end(offsets, e, P) - group_begin(offsets, e) + BM - 1) / BM;
#endif
        const int here = mtiles * n_tiles;
        if (L < before + here) {
#if defined(__HIP_DEVICE_COMPILE__)
            const int prev = __builtin_amdgcn_readlane(lo, e), next = __builtin_amdgcn_readlane(hi, e);
#else
            const int prev = group_begin(offsets, e), next = group_end(offsets, e, P);
#endif
            const int local = L - before;
            e_out = e;
            // blocks of n_inner n-tiles: block outer, the expert's m-tiles in the middle, the
            // block's n-tiles inner (n_inner = 1: n-tile outer, m-tiles inner)
            const int nb = max(n_inner, 1);
            const int full = (n_tiles / nb) * nb * mtiles;  // tiles in whole blocks
            int mt, nt;
            if (local < full) {
                const int rem = local % (mtiles * nb);
                mt = rem / nb;
                nt = (local / (mtiles * nb)) * nb + rem % nb;
            } else {
                const int nb_tail = n_tiles % nb;
                const int rem = local - full;
                mt = rem / nb_tail;
                nt = (n_tiles / nb) * nb + rem % nb_tail;
            }
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
        before += here;
    }
    return false;
}

// fp32 problems (expert_gemm_f32.hip)
int run_gemm_f32(GemmArgs& g, bool swiglu, hipStream_t st);
// bf16 products, fills straight into LDS (expert_gemm_pp.hip)
bool gemm_pp_supported(const GemmArgs& g);
int run_gemm_pp(GemmArgs& g, bool swiglu, hipStream_t st);
// Parts into which it is worth cutting the k-steps of a plain product of P rows in E groups (k_parts above)
int gemm_pp_split(long long P, int E, int N, int K, bool parts_f32, bool sum_launch);
int launch_sum_parts(const float* parts, int q, long long n, void* out, hipStream_t st);

}  // namespace moe
