// Gate-weighted combine back to token order:
//   y[t,:] = sum_{j<k} gate[t,j] * y_perm[inv_perm[t*k+j], :]  (+ residual[t,:]) (+ addend[t,:])
// y_perm may come as several partial outputs (a down projection whose k-steps were cut into parts):
// then y_perm[s,:] stands for the sum of the parts' rows s, added here in part order.
// (Sec. 1 / Sec. 2.1: the gate sets each selected expert's contribution.)  One workgroup
// per token, 16-byte loads, fp32 accumulation in ascending j, one rounding at the store.
#include <type_traits>

#include "common.h"

namespace moe {

enum { ADD_NONE, ADD_ONE, ADD_PARTS };  // no addend, one of type T, several fp32 parts of one

// PARTS: partial outputs of y_perm, of type Y (known at compile time, so that the loads of a row are all in flight
// together: 8 tokens of a 1024 / 2816 layer 38.9 -> 37.1 us)
// ADD: the addend's form.  (Known at compile time: the four fp32 parts that only a layer with a base has are 32 registers, and from 65 on a
// CU holds less than eight workgroups.  2048 tokens of 2048, a workgroup each, with / without them: one expert 4.92 / 4.35 us, two 5.95 / 5.53.)
template <typename T, typename Y, int PARTS, int ADD>
__global__ __launch_bounds__(256) void combine_kernel(ptr_arg a_inv, ptr_arg a_gate, ptr_arg a_perm, int d, int k, int P, int addend_parts,
                                                      ptr_arg a_residual, ptr_arg a_addend, ptr_arg a_y) {
    const int32_t* const inv_perm = from_arg<const int32_t>(a_inv);
    const float* const gate = from_arg<const float>(a_gate);
    const Y* const y_perm = from_arg<const Y>(a_perm);
    const T *const residual = from_arg<const T>(a_residual), *const addend = from_arg<const T>(a_addend);
    T* const y = from_arg<T>(a_y);
    typedef Store<T> S;
    constexpr int VEC = S::VEC, YV = VEC / Store<Y>::VEC;  // loads of y_perm per chunk of y
    typedef typename S::vec_t vec_t;
    const int t = blockIdx.x;
    for (int i = threadIdx.x * VEC; i < d; i += blockDim.x * VEC) {
        float acc[VEC];
#pragma unroll
        for (int q = 0; q < VEC; ++q) acc[q] = 0.f;
        // Everything that a chunk needs is requested ahead of the sums: the residual, a shared part, and two pairs' rows at a time.  (One
        // after the other they were up to four memory latencies: 16384 tokens of 2048, two experts, 36.6 us, 33.9 now, 8192 tokens of 720,
        // eight experts, 32.0 and 23.9; layer of 8 tokens on a shared base of 2048 / 5632 65.4 and 63.8, of 24 tokens, 4 of 16 experts, 43.1 and 42.5.
        // fp32 rows of 2048, four experts: 512 tokens 5.2 and 4.7, 1024 tokens 8.3 and 7.5, 8192 tokens 65.9 and 65.0; only where rows and results are about what
        // the memory-side cache holds, 4096 tokens, is it 25.5 and 25.9.)
        vec_t res{}, add{};
        f32x4 add_part[ADD == ADD_PARTS ? kMaxParts : 1][VEC / 4] = {};
        if (residual) res = *reinterpret_cast<const vec_t*>(residual + (size_t)t * d + i);
        if constexpr (ADD == ADD_PARTS) {
            const float* a = reinterpret_cast<const float*>(addend) + (size_t)t * d + i;
#pragma unroll
            for (int part = 0; part < kMaxParts; ++part)
                if (part < addend_parts)
#pragma unroll
                    for (int q = 0; q < VEC / 4; ++q) add_part[part][q] = reinterpret_cast<const f32x4*>(a + (size_t)part * gridDim.x * d)[q];
        } else if constexpr (ADD == ADD_ONE) {
            add = *reinterpret_cast<const vec_t*>(addend + (size_t)t * d + i);
        }
        auto pairs = [&](int j, auto n) {
            constexpr int N = decltype(n)::value;
            float g[N];
            typename Store<Y>::vec_t v[N][PARTS][YV];
#pragma unroll
            for (int p = 0; p < N; ++p) {
                const int s = min(max(inv_perm[(size_t)t * k + j + p], 0), P - 1);
                g[p] = gate[(size_t)t * k + j + p];
                const Y* row = y_perm + (size_t)s * d + i;
#pragma unroll
                for (int part = 0; part < PARTS; ++part, row += (size_t)P * d)
#pragma unroll
                    for (int q = 0; q < YV; ++q) v[p][part][q] = reinterpret_cast<const typename Store<Y>::vec_t*>(row)[q];
            }
#pragma unroll
            for (int p = 0; p < N; ++p)
#pragma unroll
                for (int part = 0; part < PARTS; ++part)
#pragma unroll
                    for (int q = 0; q < VEC; ++q) acc[q] = fmaf(g[p], Store<Y>::get(v[p][part][q / Store<Y>::VEC], q % Store<Y>::VEC), acc[q]);
        };
        int j = 0;
        for (; j + 2 <= k; j += 2) pairs(j, std::integral_constant<int, 2>{});
        if (j < k) pairs(j, std::integral_constant<int, 1>{});
        if (residual) {
#pragma unroll
            for (int q = 0; q < VEC; ++q) acc[q] += S::get(res, q);
        }
        if constexpr (ADD == ADD_PARTS) {
#pragma unroll
            for (int part = 0; part < kMaxParts; ++part)
                if (part < addend_parts)
#pragma unroll
                    for (int q = 0; q < VEC; ++q) acc[q] += add_part[part][q / 4][q % 4];
        } else if constexpr (ADD == ADD_ONE) {
#pragma unroll
            for (int q = 0; q < VEC; ++q) acc[q] += S::get(add, q);
        }
        vec_t o;
#pragma unroll
        for (int q = 0; q < VEC; ++q) o[q] = S::from_f32(acc[q]);
        *reinterpret_cast<vec_t*>(y + (size_t)t * d + i) = o;
    }
}

template <typename T, typename Y, int PARTS>
static int combine_on(const moe_shape& s, const void* y_perm, const int32_t* inv_perm, const float* topk_gate,
                      const void* residual, void* y, hipStream_t st, const void* addend, int addend_parts) {
    const auto kern = !addend            ? combine_kernel<T, Y, PARTS, ADD_NONE>
                      : addend_parts > 1 ? combine_kernel<T, Y, PARTS, ADD_PARTS>
                                         : combine_kernel<T, Y, PARTS, ADD_ONE>;
    hipLaunchKernelGGL(kern, dim3(s.n_tokens), dim3(256), 0, st, as_arg(inv_perm), as_arg(topk_gate),
                       as_arg(y_perm), s.d_model, s.top_k, s.n_tokens * s.top_k, addend_parts, as_arg(residual), as_arg(addend),
                       as_arg(y));
    return launch_status();
}

int launch_combine(const moe_shape& s, const void* y_perm, const int32_t* inv_perm,
                   const float* topk_gate, const void* residual, void* y, hipStream_t st,
                   const void* addend, int y_parts, bool y_parts_f32, int addend_parts) {
    if (s.n_tokens == 0) return MOE_OK;
    auto on = [&](auto run) { return run(s, y_perm, inv_perm, topk_gate, residual, y, st, addend, addend_parts); };
    if (s.act_dtype == MOE_F32) return y_parts == 1 ? on(combine_on<float, float, 1>) : MOE_ERR_INVALID;
    static_assert(kMaxParts == 4, "one to four parts");
    switch (y_parts) {
        case 1: return on(combine_on<bf16_t, bf16_t, 1>);
        case 2: return on(y_parts_f32 ? combine_on<bf16_t, float, 2> : combine_on<bf16_t, bf16_t, 2>);
        case 3: return on(y_parts_f32 ? combine_on<bf16_t, float, 3> : combine_on<bf16_t, bf16_t, 3>);
        case 4: return on(y_parts_f32 ? combine_on<bf16_t, float, 4> : combine_on<bf16_t, bf16_t, 4>);
        default: return MOE_ERR_INVALID;
    }
}

}  // namespace moe
