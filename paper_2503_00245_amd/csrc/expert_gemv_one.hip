// One token: the first and the last stage of the layer, each as one pass over weights that are all
// requested at once.
//
//   decode_first_kernel  routes the token and multiplies it with the two [rows, d] matrices of each
//                        selected expert (gate / up projection with SwiGLU, or the two rank factors)
//   decode_last_kernel   y = sum_j gate_j M_j h_j (+ residual) over the selected experts
//
// Both are bound by HBM: a CU has to keep its L1 full of requests from the first clock to the last.
#include <algorithm>

#include "gemv.h"
#include "router.h"

namespace moe {

constexpr int kOneWaves = 16;  // per workgroup: 4 per SIMD, so a wave may hold 128 registers
constexpr int kOneCus = 256;

// Every workgroup routes the token for itself: 64 KB of router rows from its L2 per CU, a wave per
// expert, and all of it in one round trip, in place of a launch that leaves 255 CUs idle.  With one
// workgroup per CU that is 16 MB out of the L2s.  A wave then takes (pair, row) units gw, gw + W, ...;
// it holds the token's row in registers and requests both rows of its next unit (8 KB at 2048 wide)
// before it sums the current one.
// NC: 1 KB chunks per row.
template <typename T, int NC, bool SWIGLU>
__global__ __launch_bounds__(kOneWaves* kWave) __attribute__((amdgpu_waves_per_eu(4, 4))) void decode_first_kernel(
    const FirstStage a) {
    typedef Store<T> S;
    typedef typename S::vec_t vec_t;
    constexpr int VEC = S::VEC, CH = kWave * VEC;
    __shared__ float s_logit[kMaxExperts];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int n = a.d;
    const T* x = static_cast<const T*>(a.x);

    // only the last chunk can be ragged (n is a multiple of VEC): lanes beyond it read the row's last
    // vector and count as zero
    int off[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) off[c] = min(c * CH + lane * VEC, n - VEC);
    const bool tail_in = (NC - 1) * CH + lane * VEC < n;
    vec_t xv[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) xv[c] = *reinterpret_cast<const vec_t*>(x + off[c]);

    auto load_x = [&](int, int i, float* out) {
        const vec_t v = *reinterpret_cast<const vec_t*>(x + i);
#pragma unroll
        for (int q = 0; q < VEC; ++q) out[q] = S::get(v, q);
    };
    for (int e = wave; e < a.E; e += kOneWaves) {
        const float b = a.router_b ? a.router_b[e] : 0.f;
        float acc[1];
        router_logits<VEC, 1, 4>(load_x, a.router_w + (size_t)e * n, n, lane, 1, acc);
        if (lane == 0) s_logit[e] = acc[0] + b;
    }
    __syncthreads();
    const RouterPick pick = router_select(lane, a.E, a.k, lane < a.E ? s_logit[lane] : 0.f);
    if (blockIdx.x == 0 && wave == 0 && pick.slot >= 0) {
        a.idx[pick.slot] = lane;
        a.gate[pick.slot] = pick.p / pick.sel_sum;
    }

    struct Unit {
        int j, row;  // pair, row; j >= k: none left
    };
    struct Rows {
        vec_t w0[NC], w1[NC];
    };
    const int stride = gridDim.x * kOneWaves;
    auto settle = [&](Unit u) {
        while (u.row >= a.rows && u.j < a.k) {
            u.row -= a.rows;
            ++u.j;
        }
        return u;
    };
    auto load = [&](Rows& r, const Unit& u) {
        const int e = max(__ffsll((unsigned long long)__ballot(pick.slot == u.j)) - 1, 0);
        const size_t at = (size_t)e * a.stride + (size_t)u.row * n;
        const T* p0 = static_cast<const T*>(a.W0) + at;
        const T* p1 = static_cast<const T*>(a.W1) + at;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            r.w0[c] = __builtin_nontemporal_load(reinterpret_cast<const vec_t*>(p0 + off[c]));
            r.w1[c] = __builtin_nontemporal_load(reinterpret_cast<const vec_t*>(p1 + off[c]));
        }
    };
    auto finish = [&](Rows& r, const Unit& u) {
        float s0 = 0.f, s1 = 0.f;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
#pragma unroll
            for (int q = 0; q < VEC; ++q) {
                const bool in = c + 1 < NC || tail_in;
                const float xq = S::get(xv[c], q);
                s0 = fmaf(in ? S::get(r.w0[c], q) : 0.f, xq, s0);
                s1 = fmaf(in ? S::get(r.w1[c], q) : 0.f, xq, s1);
            }
        }
        s0 = wave_sum(s0);
        s1 = wave_sum(s1);
        if (lane == 0) {
            const size_t at = (size_t)u.j * a.rows + u.row;
            if (SWIGLU) {
                const float h = silu_f32(s0) * s1;
                if (a.out0_act)
                    static_cast<T*>(a.out0_act)[at] = S::from_f32(h);
                else
                    a.out0[at] = h;
            } else {
                a.out0[at] = s0;
                a.out1[at] = s1;
            }
        }
    };
    // (x beyond the row's end: the last vector again; its weight is zero, so it must not be inf)
    if (!tail_in) {
#pragma unroll
        for (int q = 0; q < VEC; ++q) xv[NC - 1][q] = S::from_f32(0.f);
    }
    Rows r0, r1;
    Unit u0 = settle(Unit{0, (int)blockIdx.x * kOneWaves + wave});
    if (u0.j < a.k) load(r0, u0);
    while (u0.j < a.k) {
        const Unit u1 = settle(Unit{u0.j, u0.row + stride});
        if (u1.j < a.k) load(r1, u1);
        __builtin_amdgcn_sched_barrier(0);  // the requests stay ahead of the sums
        finish(r0, u0);
        if (u1.j >= a.k) break;
        u0 = settle(Unit{u1.j, u1.row + stride});
        if (u0.j < a.k) load(r0, u0);
        __builtin_amdgcn_sched_barrier(0);
        finish(r1, u1);
    }
}

// A wave takes one slice of one (row, pair): chunks slice, slice + slices, ... -- NC of them, all
// requested before the first is used, the hidden vector's ahead of the expert's id.  16 waves hold
// 16 / (k slices) rows; their sums meet in LDS and are added in slice and pair order.
// V: the stored type of the hidden vectors.
template <typename T, typename V, int NC>
__global__ __launch_bounds__(kOneWaves* kWave) __attribute__((amdgpu_waves_per_eu(4, 4))) void decode_last_kernel(
    const LastStage a) {
    typedef typename Store<T>::vec_t vec_t;
    typedef typename Store<V>::vec_t vvec_t;
    constexpr int VEC = Store<T>::VEC, CH = kWave * VEC, VL = VEC / Store<V>::VEC;
    __shared__ float s_part[kOneWaves];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int per_row = a.k * a.slices, rows_here = kOneWaves / per_row;
    const int local_row = wave / per_row, q = wave - local_row * per_row;
    const int j = q / a.slices, slice = q - j * a.slices;
    const int row = min((int)blockIdx.x * rows_here + local_row, a.rows - 1);
    const int n = a.n;

    int off[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) off[c] = min((slice + c * a.slices) * CH + lane * VEC, n - VEC);
    const bool tail_in = (slice + (NC - 1) * a.slices) * CH + lane * VEC < n;
    const V* v = static_cast<const V*>(a.v) + (size_t)j * n;
    vvec_t x[NC][VL];
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int l = 0; l < VL; ++l) x[c][l] = *reinterpret_cast<const vvec_t*>(v + off[c] + l * Store<V>::VEC);
    __builtin_amdgcn_sched_barrier(0);
    const int e = min(max(a.idx[j], 0), a.E - 1);
    const T* w = static_cast<const T*>(a.W) + (size_t)e * a.stride + (size_t)row * n;
    vec_t wv[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) wv[c] = __builtin_nontemporal_load(reinterpret_cast<const vec_t*>(w + off[c]));
    // what the last step needs beside the sums
    const int my_row = (int)blockIdx.x * rows_here + (int)threadIdx.x;
    const bool mine = (int)threadIdx.x < rows_here && my_row < a.rows;
    float res = 0.f;
    if (a.residual && mine) res = Store<T>::to_f32(static_cast<const T*>(a.residual)[my_row]);
    __builtin_amdgcn_sched_barrier(0);
    float s = 0.f;
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
            const bool in = c + 1 < NC || tail_in;
            const float xi = Store<V>::to_f32(x[c][i / Store<V>::VEC][i % Store<V>::VEC]);
            s = fmaf(in ? Store<T>::get(wv[c], i) : 0.f, in ? xi : 0.f, s);
        }
    s = wave_sum(s);
    if (lane == 0) s_part[wave] = s;
    __syncthreads();
    if (mine) {
        float total = 0.f;
        for (int jj = 0; jj < a.k; ++jj) {
            float sum = 0.f;
            for (int sl = 0; sl < a.slices; ++sl) sum += s_part[threadIdx.x * per_row + jj * a.slices + sl];
            total = fmaf(a.gate[jj], sum, total);
        }
        static_cast<T*>(a.y)[my_row] = Store<T>::from_f32(total + res);
    }
}

template <typename T>
static constexpr int chunks_of(int n) { return (n + kWave * Store<T>::VEC - 1) / (kWave * Store<T>::VEC); }

constexpr int kFirstMaxChunks = 4;
// The router is read once per CU: past 128 KB that read takes as long as the launch that it saves.
constexpr size_t kFirstMaxRouterBytes = 128 * 1024;

bool decode_first_supported(const moe_shape& s) {
    return s.n_tokens == 1 &&
           (s.act_dtype == MOE_F32 ? chunks_of<float>(s.d_model) : chunks_of<bf16_t>(s.d_model)) <= kFirstMaxChunks &&
           (size_t)s.n_experts * s.d_model * sizeof(float) <= kFirstMaxRouterBytes;
}

template <typename T, int NC>
static void launch_first_nc(const FirstStage& a, bool swiglu, dim3 grid, hipStream_t st) {
    const dim3 block(kOneWaves * kWave);
    if (swiglu)
        hipLaunchKernelGGL((decode_first_kernel<T, NC, true>), grid, block, 0, st, a);
    else
        hipLaunchKernelGGL((decode_first_kernel<T, NC, false>), grid, block, 0, st, a);
}

template <typename T>
static int launch_first_t(const FirstStage& a, bool swiglu, hipStream_t st) {
    const long long units = (long long)a.k * a.rows;
    const dim3 grid((unsigned)std::min<long long>(kOneCus, (units + kOneWaves - 1) / kOneWaves));
    switch (chunks_of<T>(a.d)) {
        case 1: launch_first_nc<T, 1>(a, swiglu, grid, st); break;
        case 2: launch_first_nc<T, 2>(a, swiglu, grid, st); break;
        case 3: launch_first_nc<T, 3>(a, swiglu, grid, st); break;
        case 4: launch_first_nc<T, 4>(a, swiglu, grid, st); break;
        default: return MOE_ERR_UNSUPPORTED;
    }
    return launch_status();
}

int launch_decode_first(int act_dtype, const FirstStage& a, bool swiglu, hipStream_t st) {
    return act_dtype == MOE_F32 ? launch_first_t<float>(a, swiglu, st) : launch_first_t<bf16_t>(a, swiglu, st);
}

// A wave's chunks with their part of the hidden vector: 128 registers hold 12 of them beside a vector in
// the weights' type, 8 beside an fp32 one that is twice as long.
template <typename T, typename V>
static constexpr int last_max_chunks() { return sizeof(V) > sizeof(T) ? 8 : 12; }

template <typename T, typename V, int NC>
static int launch_last_nc(const LastStage& a, int nc, hipStream_t st) {
    if constexpr (NC > last_max_chunks<T, V>()) {
        return MOE_ERR_UNSUPPORTED;
    } else {
        if (nc != NC) return launch_last_nc<T, V, NC + 1>(a, nc, st);
        const int rows_here = kOneWaves / (a.k * a.slices);
        const dim3 grid((a.rows + rows_here - 1) / rows_here), block(kOneWaves * kWave);
        hipLaunchKernelGGL((decode_last_kernel<T, V, NC>), grid, block, 0, st, a);
        return launch_status();
    }
}

// Slices per (row, pair): the fewest that fit the registers, then more while the stage has fewer waves
// than the chip holds and every slice keeps two chunks.  0: the stage is not one for this kernel.
template <typename T, typename V>
static int last_slices(int rows, int n, int k) {
    if (k > kOneWaves || kOneWaves % k) return 0;
    const int chunks = chunks_of<T>(n);
    int s = 1;
    while ((chunks + s - 1) / s > last_max_chunks<T, V>()) s *= 2;
    while ((long long)rows * k * s * 2 <= kOneCus * kOneWaves && chunks >= 4 * s) s *= 2;
    return k * s <= kOneWaves ? s : 0;
}

template <typename T, typename V>
static int launch_last_t(LastStage& a, hipStream_t st) {
    a.slices = last_slices<T, V>(a.rows, a.n, a.k);
    if (!a.slices) return MOE_ERR_UNSUPPORTED;
    return launch_last_nc<T, V, 1>(a, (chunks_of<T>(a.n) + a.slices - 1) / a.slices, st);
}

bool decode_last_supported(int act_dtype, bool v_f32, int rows, int n, int k) {
    if (act_dtype == MOE_F32) return last_slices<float, float>(rows, n, k) != 0;
    return (v_f32 ? last_slices<bf16_t, float>(rows, n, k) : last_slices<bf16_t, bf16_t>(rows, n, k)) != 0;
}

int launch_decode_last(int act_dtype, bool v_f32, LastStage a, hipStream_t st) {
    if (act_dtype == MOE_F32) return launch_last_t<float, float>(a, st);
    return v_f32 ? launch_last_t<bf16_t, float>(a, st) : launch_last_t<bf16_t, bf16_t>(a, st);
}

}  // namespace moe
