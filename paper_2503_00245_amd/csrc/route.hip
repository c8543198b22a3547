// Fused router: logits, softmax (Sec. 2.3 Eq. 2, temperature 1), top-k (Eq. 3) with
// lowest-index tie-break and gates renormalised over the k chosen.
//
// One workgroup per kRouteTok tokens.  Wave w accumulates the logits of experts w, w+W, ...
// for all of the group's tokens at once (each router row chunk is read once and reused),
// with 16-byte loads striding the rows and 64-lane butterflies; then wave w takes tokens
// w, w+W, ..., holds one logit per lane and runs k rounds of a (value, index) arg-max
// butterfly.  Everything stays in registers / LDS; only the k indices, k gates and
// (optionally) the E probabilities are written.
#include "router.h"

namespace moe {

constexpr int kRouteTokLarge = 4;  // ... from kRouteLargeFrom tokens on
constexpr int kRouteLargeFrom = 1024;

#ifndef MOE_ROUTE_NB_LARGE
#define MOE_ROUTE_NB_LARGE 2
#endif
// NB: router-row chunks a wave requests at once (4 for small batches, where the kernel is a chain
// of memory round trips; fewer for large ones, where registers per wave decide how many
// workgroups a CU holds)
// TOK: tokens per workgroup.  Every workgroup reads the whole router (E x d fp32) once, and with
// many tokens that re-read, not the token rows, is most of what the CUs pull in: at 2048 tokens of
// the 2048-wide, 8-expert router 11.1 us with four tokens per workgroup against 13.5 with two (and
// 11.2-12.1 with eight); at 512 tokens two are the faster (128 workgroups do not fill the chip).
template <typename T, int NB, int TOK>
__global__ __launch_bounds__(kRouteWaves* kWave) void route_kernel(
    ptr_arg x, ptr_arg rw, ptr_arg rb, int d, int E, int T_, int k, ptr_arg topk_idx, ptr_arg topk_gate, ptr_arg probs) {
    route_tokens<T, NB, TOK>(from_arg<const T>(x), from_arg<const float>(rw), from_arg<const float>(rb), from_arg<int32_t>(topk_idx),
                             from_arg<float>(topk_gate), from_arg<float>(probs), T_, d, E, k, blockIdx.x);
}

// Large batches: the whole router (E x d fp32) is staged in LDS once per workgroup and a wave
// owns TOK tokens at a time: it reads their rows once, the next chunk on its way while one is multiplied, takes the E router
// rows from LDS for all of them together and ends with one butterfly per token and expert, so lane e holds logit e and the
// selection follows in the same wave with no further exchange.  The multiply-adds of a logit run in the same order as in
// router_logits (lane l: elements [l*VEC, l*VEC+VEC) of every 64*VEC-wide chunk, ascending), so
// both kernels give bit-identical logits.  For E <= kRouteLdsMaxE and E * d * 4 bytes of LDS.
// (One token at a time read 64 KB of LDS and waited for its chunks one by one: 16384 tokens, 2048 wide, 8
// experts 42 us, 34 now.)
// Up to 8 experts a wave takes four tokens at a time, from 9 on as many as its registers hold without scratch: four of 12
// accumulators each (with 16 each, 28 bytes a lane went to scratch), two of 16, and three where that is all a wave has.  us, four with scratch /
// this, 2048 wide: 16 experts 9000 tokens 47.3 / 38.0, 12288 49.8 / 40.4, 16384 54.7 / 54.4, 32768 98.9 / 98.6; 12 experts 12288
// tokens 39.5 / 33.6, 16384 43.2 / 40.5, 32768 78.6 / 73.1 (three tokens at a time 56.4, 85.6); 9 experts, 512 wide, 16384 tokens 16.8 / 15.7.
constexpr int kRouteLdsMaxE = 16;
constexpr int kRouteLdsBytes = 128 * 1024;

template <typename T, int TOK, int MAXE>
__global__ __launch_bounds__(kRouteWaves* kWave) __attribute__((amdgpu_waves_per_eu(4, 4))) void route_lds_kernel(
    const T* __restrict__ x, const float* __restrict__ rw, const float* __restrict__ rb,
    int32_t* __restrict__ topk_idx, float* __restrict__ topk_gate, float* __restrict__ probs,
    int T_, int d, int E, int k, int tokens_per_wave) {
    typedef Store<T> S;
    constexpr int VEC = S::VEC;
    constexpr int CH = kWave * VEC;
    extern __shared__ __align__(16) float s_rw[];  // [E][d]
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int t_first = (blockIdx.x * kRouteWaves + wave) * tokens_per_wave, t_end = min(T_, t_first + tokens_per_wave);
    const int chunks = (d + CH - 1) / CH;  // the last one may be ragged: lanes beyond the row add nothing
    typename S::vec_t cur[TOK], nxt[TOK];
    auto load = [&](typename S::vec_t (&v)[TOK], int t, int c) {
        const int i = min(c * CH + lane * VEC, d - VEC);
#pragma unroll
        for (int u = 0; u < TOK; ++u) v[u] = *reinterpret_cast<const typename S::vec_t*>(x + (size_t)min(t + u, T_ - 1) * d + i);
    };
    load(cur, t_first, 0);
    for (int i = threadIdx.x; i < E * d / 4; i += kRouteWaves * kWave)
        reinterpret_cast<f32x4*>(s_rw)[i] = reinterpret_cast<const f32x4*>(rw)[i];
    __syncthreads();

    for (int t = t_first; t < t_end; t += TOK) {
        float acc[MAXE][TOK];
#pragma unroll
        for (int e = 0; e < MAXE; ++e)
#pragma unroll
            for (int u = 0; u < TOK; ++u) acc[e][u] = 0.f;
        for (int c = 0; c < chunks; ++c) {
            const bool last = c + 1 == chunks;
            load(nxt, last ? t + TOK : t, last ? 0 : c + 1);
            const int i = c * CH + lane * VEC;
            if (i < d) {
#pragma unroll
                for (int e = 0; e < MAXE; ++e) {
                    if (e >= E) continue;  // wave-uniform
                    const float* w = s_rw + e * d + i;
#pragma unroll
                    for (int q = 0; q < VEC; q += 4) {
                        const f32x4 wv = *reinterpret_cast<const f32x4*>(w + q);
#pragma unroll
                        for (int u = 0; u < TOK; ++u)
#pragma unroll
                            for (int j = 0; j < 4; ++j) acc[e][u] = fmaf(S::get(cur[u], q + j), wv[j], acc[e][u]);
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < TOK; ++u) cur[u] = nxt[u];
        }
#pragma unroll
        for (int u = 0; u < TOK; ++u) {
            float logit = 0.f;
#pragma unroll
            for (int e = 0; e < MAXE; ++e) {
                if (e >= E) continue;
                const float sum = wave_sum(acc[e][u]);
                if (lane == e) logit = sum + (rb ? rb[e] : 0.f);
            }
            if (t + u >= t_end) continue;
            const RouterPick r = router_select(lane, E, k, lane < E ? logit : 0.f);
            if (probs && lane < E) probs[(size_t)(t + u) * E + lane] = r.p / r.den;
            if (r.slot >= 0) {
                topk_idx[(size_t)(t + u) * k + r.slot] = lane;
                topk_gate[(size_t)(t + u) * k + r.slot] = r.p / r.sel_sum;
            }
        }
    }
}

template <typename T>
static int launch_route_lds(const moe_shape& s, const T* x, const float* rw, const float* rb,
                            int32_t* topk_idx, float* topk_gate, float* probs, hipStream_t st) {
    const size_t lds = (size_t)s.n_experts * s.d_model * sizeof(float);
    // up to two workgroups per CU, every wave with the same number of tokens
    const int waves = 2 * 256 * kRouteWaves;
    const int tokens_per_wave = (s.n_tokens + waves - 1) / waves;
    const int per_block = tokens_per_wave * kRouteWaves;
    dim3 grid((s.n_tokens + per_block - 1) / per_block), block(kRouteWaves * kWave);
    auto launch = [&](auto kern, std::atomic<uint64_t>& lds_allowed) {
        if (allow_dynamic_lds(reinterpret_cast<const void*>(kern), kRouteLdsBytes, lds_allowed) != MOE_OK) return (int)MOE_ERR_LAUNCH;
        hipLaunchKernelGGL(kern, grid, block, lds, st, x, rw, rb, topk_idx, topk_gate, probs, s.n_tokens, s.d_model, s.n_experts,
                           s.top_k, tokens_per_wave);
        return launch_status();
    };
    static std::atomic<uint64_t> allowed[5];
    if (s.n_experts <= 8)
        return tokens_per_wave > 2 ? launch(route_lds_kernel<T, 4, 8>, allowed[0]) : launch(route_lds_kernel<T, 2, 8>, allowed[1]);
    if (tokens_per_wave == 3) return launch(route_lds_kernel<T, 3, 16>, allowed[2]);
    if (tokens_per_wave > 3 && s.n_experts <= 12) return launch(route_lds_kernel<T, 4, 12>, allowed[3]);
    return launch(route_lds_kernel<T, 2, 16>, allowed[4]);
}

int launch_route(const moe_shape& s, const void* x, const float* rw, const float* rb,
                 int32_t* topk_idx, float* topk_gate, float* probs, hipStream_t st) {
    if (s.n_tokens == 0) return MOE_OK;
    // (measured on the 2048-wide, 8-expert router: 15.6 us against 12.7 at 2048 tokens, 34 against
    // 64 at 16384, 18 against 34 at 8192)
    if (s.n_tokens >= 8192 && s.n_experts <= kRouteLdsMaxE &&
        (size_t)s.n_experts * s.d_model * sizeof(float) <= (size_t)kRouteLdsBytes) {
        if (s.act_dtype == MOE_F32)
            return launch_route_lds<float>(s, (const float*)x, rw, rb, topk_idx, topk_gate, probs, st);
        return launch_route_lds<bf16_t>(s, (const bf16_t*)x, rw, rb, topk_idx, topk_gate, probs, st);
    }
    const bool small = s.n_tokens <= 256, large = s.n_tokens >= kRouteLargeFrom;
    const int tok = large ? kRouteTokLarge : kRouteTok;
    dim3 grid((s.n_tokens + tok - 1) / tok), block(kRouteWaves * kWave);
    auto launch = [&](auto kern) {
        hipLaunchKernelGGL(kern, grid, block, 0, st, as_arg(x), as_arg(rw), as_arg(rb), s.d_model, s.n_experts, s.n_tokens, s.top_k,
                           as_arg(topk_idx), as_arg(topk_gate), as_arg(probs));
    };
    if (s.act_dtype == MOE_F32) {
        if (small) launch(route_kernel<float, 4, kRouteTok>);
        else if (!large) launch(route_kernel<float, MOE_ROUTE_NB_LARGE, kRouteTok>);
        else launch(route_kernel<float, MOE_ROUTE_NB_LARGE, kRouteTokLarge>);
    } else {
        if (small) launch(route_kernel<bf16_t, 4, kRouteTok>);
        else if (!large) launch(route_kernel<bf16_t, MOE_ROUTE_NB_LARGE, kRouteTok>);
        else launch(route_kernel<bf16_t, MOE_ROUTE_NB_LARGE, kRouteTokLarge>);
    }
    return launch_status();
}

}  // namespace moe
