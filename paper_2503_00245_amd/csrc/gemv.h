// Single-token stages that live in a file of their own (expert_gemv_one.hip), as expert_gemv.hip calls them.
#pragma once

#include "common.h"

namespace moe {

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

}  // namespace moe
