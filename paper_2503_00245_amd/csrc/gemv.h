// Single-token stages that live in a file of their own (expert_gemv_one.hip), as expert_gemv.hip calls them.
#pragma once

#include "common.h"

namespace moe {

constexpr int kOneWaves = 16;  // waves of a workgroup: 4 per SIMD, so a wave may hold 128 registers
constexpr int kOneCus = 256;

// Units beyond the last whole turn of all waves, spread over the workgroups: which of them is the w-th wave's of a workgroup.  Neighbours lie on one
// XCD (workgroups go to the XCDs in turn).
__host__ __device__ inline int place_in_rest(int block, int w, int blocks) {
    return w * blocks + (blocks % 8 == 0 ? (block & 7) * (blocks >> 3) + (block >> 3) : block);
}
// Order of decode_first_kernel's units (pair, row) on the waves of `blocks` workgroups: 0, waves first, so that a workgroup's rows and results are
// neighbours; -1, workgroups first, so that no CU has more than another of the units beyond the last whole turn of all waves; the number of
// whole turns, waves first and the rest alone on place_in_rest.  Waves first in one turn (400 / 1072 8.2 us for the layer, 8.4 workgroups first),
// where there is no rest, and where it fills more than three quarters of the waves (1472 / 3952, 1.93 turns, 18.2 / 18.3).  Otherwise
// (whole layer, us, waves first / workgroups first / the rest alone)
//   - the rest alone in rows that are no whole cache lines, of which neighbours share one: 2040 / 5552, 2.71 turns, 27.6 / 28.2 / 27.6, 1400 / 3760,
//     1.84, 17.4 / 17.7 / 17.4, 2016 / 5376, 4 experts, 5.25, 50.5 / 49.7 / 49.1; and in short ones: 1024 / 2816, 1.38, 12.1 / 12.1 / 11.9, 960 / 2560,
//     1.25, 11.5 / 11.4 / 11.1, 832 / 2240 10.6 / 10.5 / 10.2, 1088 / 2880 14.1 / 13.8 / 13.6;
//   - workgroups first in longer ones: even from 2.5 KB on (1280 / 3456 16.1 / 16.0 / 16.0, 1920 / 5184 25.4 / 25.2 / 25.2), and at 2048 / 5632 27.7 /
//     27.6 / 27.7, one expert 18.2 / 16.8 / 17.1, a shared base's 5632 rows on 3968 waves 25.4 / 22.1 / 22.6.
inline int first_stage_turns(long long units, int blocks, int row_bytes) {
    const long long waves = (long long)blocks * kOneWaves, rest = units % waves;
    if (units <= waves || rest == 0 || 4 * rest > 3 * waves) return 0;
    return row_bytes % 128 == 0 && row_bytes > 2560 ? -1 : (int)(units / waves);
}
// Order of a pair's rows of rank factors on its `waves` waves (decode_hidden_kernel): 0, waves first, so that neighbouring rows are a workgroup's; -1,
// workgroups first, so that the last turn's rows lie on all CUs; the number of whole turns, waves first and the rest alone on place_in_rest.
//   Rows of whole cache lines (whole layer, us, 2 of 8 experts, waves first / workgroups first): 2048 / 5632 of rank 1024, 2.75 turns, 27.9 / 27.5,
//   1024 / 2816 of 512, 1.38, 16.5 / 16.1, 1704 / 4544 of 576, 2.22, 22.8 / 22.3; 1920 / 5120 of 960, 4 experts, 5 whole turns, 40.5 / 40.0.
//   Other rows, of which neighbours share a line (waves first / workgroups first / the rest alone): 2040 / 5552 of 1016, 2.71, 28.3 / 28.2 / 27.9,
//   1800 / 4800 of 600, 2.34, 23.4 / 23.1 / 22.8, 1984 / 5312 of 264, 4 experts, 5.19, 26.0 / 26.2 / 25.7, 1536 / 4096 of 264, 2 whole turns,
//   17.3 / 17.6 / 17.3.
// Waves first in one turn, and where the last one fills more than three quarters of them (1440 / 3840 of 720, 1.88, 21.4 / 21.5).
inline int hidden_turns(int rows, int waves, int k, int row_bytes) {
    const int rest = rows % waves;
    if (rows <= waves || 4 * rest > 3 * waves) return 0;
    if (row_bytes % 128 == 0) return -1;
    // (where k does not divide the waves, the last workgroup lacks a wave of some pairs: none whose place is below this)
    return rest > 0 && rest < kOneWaves / k * kOneCus ? rows / waves : 0;
}

// Route the token x [d], then out0[j] = W0[expert j] x and out1[j] = W1[expert j] x, or, with SwiGLU,
// out0[j] = silu(W0 x) * (W1 x).
struct FirstStage {
    const void* x;
    const float *router_w, *router_b;
    const void *W0, *W1;  // [E, rows, d]
    long long stride;     // elements between experts
    int rows, d, E, k;
    int32_t* idx;         // [k], written
    float* gate;          // [k], written
    float *out0, *out1;   // [k][rows]
    void* out0_act;       // SwiGLU: [k][rows] in the activation type, written instead of out0 (or NULL)
    // without SwiGLU, beside those: base0 = base_W0 x, base1 = base_W1 x (or NULL)
    const void *base_W0, *base_W1;  // [base_rows, d]
    float *base0, *base1;
    int base_rows;
    int route_blocks;     // set by the launcher, as are these (first_stage_turns)
    int turns, base_turns;
};
bool decode_first_supported(const moe_shape& s);
int launch_decode_first(int act_dtype, const FirstStage& a, bool swiglu, hipStream_t st);

// y[row] = sum_j gate_j <W[expert j][row, :], v_j> (+ residual[row])
struct LastStage {
    const void* W;      // [E, rows, n]
    long long stride;
    const void* v;      // [k][n], fp32 or in the activation type
    int rows, n, E, k;
    int slices;         // waves per (row, pair); set by the launcher
    const int32_t* idx;
    const float* gate;
    const void* residual;
    void* y;
};
bool decode_last_supported(int act_dtype, bool v_f32, int rows, int n, int k);
int launch_decode_last(int act_dtype, bool v_f32, LastStage a, hipStream_t st);

// Layers with a shared base: after a first stage that also forms base0 = W_gate x and base1 = W_up x,
//   low rank (hidden)  h_j and their mix      mid  td_j = R_d h_j, y0 = W_down mix      low rank  y
struct LowRankStage {
    const void *L0, *L1;     // [E, rows, r]
    long long stride;
    const float *t0, *t1;    // [k][r]
    float* b0;               // [rows]; hidden: replaced by the mix, or NULL (no base)
    const float* b1;         // [rows] (hidden)
    float* h;                // [k][rows] (hidden)
    int rows, r, E, k;
    int lanes;               // lanes per row; set by the launcher
    const int32_t* idx;
    const float* gate;
    const void* residual;
    void* y;
};
struct MidStage {
    const void *rd, *w_down;  // [E, r, n], [d, n]
    long long stride;
    const float *h, *mix;     // [k][n], [n]
    float *td, *y0;           // [k][r], [d]
    int n, r, d, E, k;
    int slices;               // waves per row; set by the launcher
    const int32_t* idx;
};
// or, where the rank-down products' partial sums are few (decode_base_parts_supported),
//   base hidden  h_j, their mix and, per workgroup's share of the rows, partial sums of R_d h_j      base last  y
struct BaseHiddenStage {
    const void *L0, *L1, *rd;  // [E, rows, r] twice, [E, r, rows]
    const float *t0, *t1;      // [k][r]
    float* b0;                 // [rows]; replaced by the mix
    const float* b1;           // [rows]
    float* parts;              // [blocks][k][r]
    int rows, r, E, k;
    int lanes;                 // lanes per row; set by the launcher
    const int32_t* idx;
    const float* gate;
};
struct BaseLastStage {
    const void *w_down, *ld;   // [rows, n], [E, rows, r]
    const float *mix, *parts;  // [n], [blocks][k][r]
    int rows, n, r, E, k;
    int slices;                // waves per row; set by the launcher
    const int32_t* idx;
    const float* gate;
    const void* residual;
    void* y;
};
bool decode_base_parts_supported(const moe_shape& s);
// tg, tu [k][r] and the parts take the place of the hidden vectors: at most k (d_ff + 3 r) floats
int launch_decode_base_hidden(BaseHiddenStage a, hipStream_t st);
int launch_decode_base_last(BaseLastStage a, hipStream_t st);
bool decode_base_supported(const moe_shape& s);
inline size_t decode_base_bytes(const moe_shape& s) { return 2 * sizeof(float) * (size_t)s.d_ff; }
int launch_decode_low_rank(LowRankStage a, bool hidden, hipStream_t st);
int launch_decode_mid(MidStage a, hipStream_t st);

// Rank experts without a base: first stage, hidden (fp32 hidden vectors), mid with d = 0, last stage.
bool decode_rank_supported(const moe_shape& s);
int launch_decode_hidden(const LowRankStage& a, hipStream_t st);

}  // namespace moe
