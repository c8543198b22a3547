// Shared device/host helpers of the gfx950 MoE library (internal; not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "moe.h"

namespace moe {

constexpr int kWave = 64;        // CDNA wavefront width
constexpr int kMaxExperts = 64;  // one lane per expert in the router's selection step

typedef __bf16 bf16_t;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// ---- storage-type traits: VEC elements per 16-byte load -------------------------------
template <typename T>
struct Store;
template <>
struct Store<float> {
    static constexpr int VEC = 4;
    typedef f32x4 vec_t;
    static __device__ __forceinline__ float get(const vec_t& v, int i) { return v[i]; }
    static __device__ __forceinline__ float to_f32(float v) { return v; }
    static __device__ __forceinline__ float from_f32(float v) { return v; }
};
template <>
struct Store<bf16_t> {
    static constexpr int VEC = 8;
    typedef bf16x8 vec_t;
    static __device__ __forceinline__ float get(const vec_t& v, int i) { return (float)v[i]; }
    static __device__ __forceinline__ float to_f32(bf16_t v) { return (float)v; }
    static __device__ __forceinline__ bf16_t from_f32(float v) { return (bf16_t)v; }  // RNE
};

// ---- wavefront reductions: every lane gets the result --------------------------------------
// Within a row of 16 lanes the exchange is done with DPP modifiers (register-to-register,
// no LDS round trip): swap neighbours, swap pairs, mirror within 8, mirror within 16.  After
// those four steps every lane of a row holds the row's result; the four rows are then
// combined with two cross-lane permutes (xor 16, xor 32).
constexpr int kDppSwap1 = 0xB1;        // quad_perm [1,0,3,2]
constexpr int kDppSwap2 = 0x4E;        // quad_perm [2,3,0,1]
constexpr int kDppHalfMirror = 0x141;  // lane i <-> 7 - i within 8
constexpr int kDppMirror = 0x140;      // lane i <-> 15 - i within 16

template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}
template <int CTRL>
__device__ __forceinline__ int dpp_i32(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, false);
}

__device__ __forceinline__ float wave_sum(float v) {
    v += dpp_f32<kDppSwap1>(v);
    v += dpp_f32<kDppSwap2>(v);
    v += dpp_f32<kDppHalfMirror>(v);
    v += dpp_f32<kDppMirror>(v);
    v += __shfl_xor(v, 16, kWave);
    v += __shfl_xor(v, 32, kWave);
    return v;
}

// silu(z) = z / (1 + e^-z) with the hardware reciprocal (1 ulp) in place of an IEEE division:
// the epilogue of a 256 x 256 SwiGLU tile evaluates it 64 times per lane.
__device__ __forceinline__ float silu_f32(float z) {
#if defined(__HIP_DEVICE_COMPILE__)
    return z * __builtin_amdgcn_rcpf(1.0f + __expf(-z));
#else
    return z / (1.0f + __expf(-z));
#endif
}

// Sum of v over this lane and those below it
__device__ __forceinline__ int wave_scan(int v) {
#if defined(__HIP_DEVICE_COMPILE__)
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);  // within a row of 16 lanes: from 1, 2, 4 and 8 lanes below
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);  // the last lane of rows 0 and 2 to rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);  // lane 31 to rows 2 and 3
#endif
    return v;
}

// ---- host side ---------------------------------------------------------------------------
inline hipStream_t as_stream(void* s) { return reinterpret_cast<hipStream_t>(s); }

inline int launch_status() { return hipGetLastError() == hipSuccess ? MOE_OK : MOE_ERR_LAUNCH; }

// Kernels that use more than the default 64 KB of dynamic LDS need the limit raised once per
// device.  `done` is a per-kernel bit mask of the devices already set up (the only state the
// library keeps; a race merely repeats the call).
inline int allow_dynamic_lds(const void* kernel, size_t bytes, std::atomic<uint64_t>& done) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return MOE_ERR_LAUNCH;
    const uint64_t bit = 1ull << (dev & 63);
    if (done.load(std::memory_order_acquire) & bit) return MOE_OK;
    if (hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) != hipSuccess)
        return MOE_ERR_LAUNCH;
    done.fetch_or(bit, std::memory_order_release);
    return MOE_OK;
}

#if defined(__HIP_DEVICE_COMPILE__)
#define MOE_READLANE(v, l) __builtin_amdgcn_readlane(v, l)
#else
#define MOE_READLANE(v, l) (v)
#endif
// a / b for a >= 0, b > 0: the estimate is off by a few hundred at most (2^31 times the rounding of the three
// float steps), the second one, of the remainder, by one.  The compiler's integer division is forty
// dependent instructions, and a workgroup makes half a dozen before its first load.
__host__ __device__ __forceinline__ int quick_div(int a, int b) {
#if defined(__HIP_DEVICE_COMPILE__)
    const float inv = __builtin_amdgcn_rcpf((float)b);
    int q = (int)((float)a * inv);
    int r = (int)((unsigned)a - (unsigned)q * (unsigned)b);
    const int more = (int)((float)r * inv);
    q += more, r -= more * b;
    q += (r >= b ? 1 : 0) - (r < 0 ? 1 : 0);
    return q;
#else
    return a / b;
#endif
}
__host__ __device__ __forceinline__ int uniform_div(int a, int b) {  // wave-uniform a, b
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_readfirstlane(quick_div(a, b));
#else
    return a / b;
#endif
}

// A device pointer in a kernel's argument list, as a number: a launch takes longer on the host for every argument of pointer type
// (a call of two launches that waits for the host: 8.9-9.3 us with six of them, 8.4-8.7 with the same as numbers).
typedef unsigned long long ptr_arg;
inline ptr_arg as_arg(const void* p) { return reinterpret_cast<ptr_arg>(p); }
template <typename T>
__device__ __forceinline__ T* from_arg(ptr_arg a) {
    return (T*)(__attribute__((address_space(1))) T*)a;
}

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

inline size_t elt_size(int act_dtype) { return act_dtype == MOE_F32 ? 4 : 2; }

inline size_t round_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// Optional per-stage timing (moe_forward_timed): an event before the first stage and after
// every stage kernel, all on the launch stream.  A null timer costs nothing.
struct StageTimer {
    hipStream_t st;
    hipEvent_t ev[MOE_MAX_STAGES + 1];
    const char* name[MOE_MAX_STAGES];
    int n;
};
inline void stage_mark(StageTimer* t, const char* name) {
    if (!t || t->n >= MOE_MAX_STAGES) return;
    t->name[t->n] = name;
    (void)hipEventRecord(t->ev[t->n + 1], t->st);
    t->n += 1;
}

// Shape check shared by every entry point: MOE_OK, MOE_ERR_INVALID or MOE_ERR_UNSUPPORTED.
int validate_shape(const moe_shape* s);

// ---- per-stage launchers (each file owns its kernels) ---------------------------------------
int launch_route(const moe_shape& s, const void* x, const float* rw, const float* rb,
                 int32_t* topk_idx, float* topk_gate, float* probs, hipStream_t st);

// scratch: permute_scratch_bytes at least; more, up to 256 counts per expert, makes for more and shorter chunks
size_t permute_scratch_bytes(int P, int E);
int launch_permute(int P, int E, const int32_t* topk_idx, int32_t* offsets, int32_t* perm,
                   int32_t* inv_perm, void* scratch, size_t scratch_bytes, hipStream_t st);
int launch_gather_rows(const moe_shape& s, const int32_t* perm, const void* x, void* x_perm,
                       hipStream_t st);

// addend: optional second per-token term [T, d] (beside the residual), in the activation type, or, with
// addend_parts > 1, the sum of that many fp32 partial outputs [T, d], one after the other.
// y_parts > 1: y_perm holds that many partial outputs [P, d], fp32 or in the activation type, one after the
// other, to be added.
int launch_combine(const moe_shape& s, const void* y_perm, const int32_t* inv_perm,
                   const float* topk_gate, const void* residual, void* y, hipStream_t st,
                   const void* addend = nullptr, int y_parts = 1, bool y_parts_f32 = true, int addend_parts = 1);

// Products whose k-steps are cut into parts to fill the chip, by shape (bf16): the final down projection
// (parts [P, d], fp32 if down_f32, else in the activation type, added by the combine), the rank-down product of weight-decomposed
// experts (fp32 parts [P, r], added by a kernel of its own) and the down projection of a shared base
// (fp32 parts [T, d], added by the combine).  1: not cut.
constexpr int kMaxParts = 4;
struct SplitPlan {
    int down, rank_down, base_down;
    bool down_f32;
};
bool down_cut_supported(const moe_shape& s);
bool few_two_tokens(const moe_shape& s);  // two tokens take the prefill's stages
// down_bytes, rank_bytes: room for the down projection's and the rank-down product's outputs
SplitPlan split_plan(const moe_shape& s, size_t down_bytes, size_t rank_bytes);

// Scratch of the expert FFN, in the activation type except for the parts.  The order is that of memory:
// rank_parts ([rank_down][P, r] fp32) starts at tg, which is consumed by then, as are bg and bu, and runs on
// into y_perm, not yet written, and the room for parts behind it; base_parts ([base_down][T, d] fp32) starts at h and
// ends before y_perm.
struct FfnScratch {
    void *td, *z, *h, *tg, *tu, *bg, *bu;
    float *rank_parts, *base_parts;
};
struct FfnLayout {  // byte offsets
    size_t td, z, h, tg, tu, bg, bu, end;
};
FfnLayout ffn_layout(const moe_shape& s);
inline FfnScratch ffn_scratch(const moe_shape& s, void* base) {
    const FfnLayout l = ffn_layout(s);
    char* b = static_cast<char*>(base);
    return FfnScratch{b + l.td, b + l.z, b + l.h, b + l.tg, b + l.tu, b + l.bg, b + l.bu,
                      reinterpret_cast<float*>(b + l.tg), reinterpret_cast<float*>(b + l.h)};
}

// Grouped expert FFN on P sorted rows.  a_row_map/a_row_div: optional gather of the input
// rows (row of sorted slot s is x[a_row_map[s] / a_row_div]); NULL = x is already grouped.
// keys: NULL, or the pairs' experts [P]: then a_row_map, offsets and inv_perm are not read but written, by the
// first product (only where ffn_takes_keys).
bool ffn_takes_keys(const moe_shape& s, const int32_t* keys);
// plan: NULL = nothing is cut, y_perm is one output [P, d].  Otherwise y_perm has room for plan->down outputs (of plan->down_f32) and
// receives that many.
inline size_t ffn_scratch_bytes(const moe_shape& s) { return ffn_layout(s).end; }
int launch_expert_ffn(const moe_shape& s, const moe_weights& w, const void* x,
                      int32_t* a_row_map, int a_row_div, int32_t* offsets,
                      void* y_perm, void* scratch, hipStream_t st, StageTimer* timer = nullptr,
                      const SplitPlan* plan = nullptr, const int32_t* keys = nullptr, int32_t* inv_perm = nullptr);

// Shared-base experts M_e = M0 + L_e R_e (Sec. 2.2, Eq. 1 with a base shared by all experts), prefill,
// with the token of every sorted slot known: the base products run once per token instead
// of once per (token, expert) pair.  y_perm [P, d] receives only the low-rank part of the down
// projection and y_base [T, d] the shared part, to be added in the combine.
bool token_base_supported(const moe_shape& s);
int launch_expert_ffn_token_base(const moe_shape& s, const moe_weights& w, const void* x,
                                 int32_t* perm, int32_t* inv_perm, const float* topk_gate,
                                 int32_t* offsets, void* y_perm, void* y_base, void* scratch,
                                 hipStream_t st, StageTimer* timer, const SplitPlan& plan, const int32_t* keys);

// Small fp32 layer of dense experts in two launches, every token with every expert; h: token_layer_bytes of scratch.
constexpr size_t kTokenLayerBytes = 4u << 20;       // at most that
bool token_layer_f32_shape(const moe_shape& s);      // whatever the number of tokens
bool token_layer_f32_supported(const moe_shape& s);
inline size_t token_layer_bytes(const moe_shape& s) { return sizeof(float) * (size_t)s.n_experts * s.n_tokens * s.d_ff; }
int launch_token_layer_f32(const moe_shape& s, const moe_weights& w, const void* x, int32_t* idx, float* gate, float* h,
                           const void* residual, void* y, hipStream_t st, StageTimer* timer);

// Single-token layer: routed, experts chosen on the device from topk_idx, weights streamed once.
// base_scratch: decode_base_bytes (gemv.h) for a layer with a shared base, or NULL.
size_t decode_scratch_bytes(const moe_shape& s, int n_tokens);
int launch_decode(const moe_shape& s, const moe_weights& w, const void* x, int32_t* topk_idx,
                  float* topk_gate, void* y, void* scratch, float* base_scratch, hipStream_t st,
                  StageTimer* timer = nullptr);

}  // namespace moe
