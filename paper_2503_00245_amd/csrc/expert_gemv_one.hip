// One token: the first and the last stage of the layer, each as one pass over weights that are all
// requested at once.
//
//   decode_first_kernel  routes the token and multiplies it with the two [rows, d] matrices of each
//                        selected expert (gate / up projection with SwiGLU, or the two rank factors)
//   decode_last_kernel   y = sum_j gate_j M_j h_j (+ residual) over the selected experts
//
// Both are bound by HBM: a CU has to keep its L1 full of requests from the first clock to the last.  What the first loads
// need stands at the head of every kernel's argument list: scalars there arrive in registers with the wave.
#include <algorithm>

#include "gemv.h"
#include "router.h"

namespace moe {

constexpr int kBaseSums = 256, kBasePairs = kBaseSums / 8;  // k r, k of decode_base_parts_supported

// Every workgroup routes the token for itself: 64 KB of router rows from its L2 per CU, a wave per
// expert, in place of a launch that leaves 255 CUs idle.  With one workgroup per CU that is 16 MB out of the L2s.  (The token's row comes
// first, then the router's, four chunks of a row at a time and a remainder of fewer one after the other: two round trips at 2048 wide, three at
// 1024, four at 1440.)  A wave then takes (pair, row) units in the order of first_stage_turns: it holds
// the token's row in registers and requests both rows of its next unit (8 KB at 2048 wide)
// before it sums the current one.  2048 x 5632, 92 MB: 18.9 us with the routing, where a router launch and
// a wave per row took 3.8 + 17.6; 1024 x 2816, 23 MB: 8.4 us for 3.1 + 8.9.  What is left beside the stream
// (5.6 TB/s) is the prologue, 2-2.5 us.
// NC: 1 KB chunks per row.  DEAL: some of the units are not dealt waves first.  (Known at compile time, and the rest's place worked out behind
// the first requests: the order's arithmetic ahead of them was 0.05-0.15 us of a layer of one turn, 456 x 1216, 2 of 4 experts, 8.18 / 8.04,
// 512 x 1376 of rank 256, one expert, 12.78 / 12.64.)
template <typename T, int NC, bool SWIGLU, bool DEAL>
__global__ __launch_bounds__(kOneWaves* kWave) __attribute__((amdgpu_waves_per_eu(4, 4))) void decode_first_kernel(
    ptr_arg ax, ptr_arg aw, ptr_arg ab, int n, int E, int route_blocks, const FirstStage a) {
    typedef Store<T> S;
    typedef typename S::vec_t vec_t;
    constexpr int VEC = S::VEC, CH = kWave * VEC;
    __shared__ float s_logit[kMaxExperts];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const T* x = from_arg<const T>(ax);
    const float *router_w = from_arg<const float>(aw), *router_b = from_arg<const float>(ab);
    // workgroups from route_blocks on: the shared base's rows, one matrix pair that needs no routing
    const bool base = !SWIGLU && (int)blockIdx.x >= route_blocks;
    const int first_block = base ? route_blocks : 0;
    const int blocks = base ? (int)gridDim.x - route_blocks : route_blocks;
    const int k = base ? 1 : a.k, rows = base ? a.base_rows : a.rows;
    const T* W0 = static_cast<const T*>(base ? a.base_W0 : a.W0);
    const T* W1 = static_cast<const T*>(base ? a.base_W1 : a.W1);
    float* out0 = base ? a.base0 : a.out0;
    float* out1 = base ? a.base1 : a.out1;

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
    int slot = lane == 0 ? 0 : -1;  // the pair whose expert this lane stands for
    float logit = 0.f, vmax = 0.f;
    if (!base) {
        for (int e = wave; e < E; e += kOneWaves) {
            const float b = router_b ? router_b[e] : 0.f;
            float acc[1];
            router_logits<VEC, 1, 4>(load_x, router_w + (size_t)e * n, n, lane, 1, acc);
            if (lane == 0) s_logit[e] = acc[0] + b;
        }
        __syncthreads();
        logit = lane < E ? s_logit[lane] : 0.f;
        slot = router_slots(lane, E, k, logit, vmax);
    }

    struct Unit {
        int j, row;  // pair, row; j >= k: none left
    };
    struct Rows {
        vec_t w0[NC], w1[NC];
    };
    const int stride = blocks * kOneWaves;
    auto settle = [&](Unit u) {
        while (u.row >= rows && u.j < k) {
            u.row -= rows;
            ++u.j;
        }
        return u;
    };
    auto load = [&](Rows& r, const Unit& u) {
        // (clamped: with NaN logits the lanes may disagree about a round, and lanes past E may win it)
        const int e = min(max(__ffsll((unsigned long long)__ballot(slot == u.j)) - 1, 0), E - 1);
        const size_t at = (size_t)e * a.stride + (size_t)u.row * n;
        const T* p0 = W0 + at;
        const T* p1 = W1 + at;
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
            const size_t at = (size_t)u.j * rows + u.row;
            if (SWIGLU) {
                const float h = silu_f32(s0) * s1;
                if (a.out0_act)
                    static_cast<T*>(a.out0_act)[at] = S::from_f32(h);
                else
                    out0[at] = h;
            } else {
                out0[at] = s0;
                out1[at] = s1;
            }
        }
    };
    // (x beyond the row's end: the last vector again; its weight is zero, so it must not be inf)
    if (!tail_in) {
#pragma unroll
        for (int q = 0; q < VEC; ++q) xv[NC - 1][q] = S::from_f32(0.f);
    }
    Rows r0, r1;
    const int in_order = (int)blockIdx.x - first_block;
    int turns = !DEAL ? 0 : base ? a.base_turns : a.turns;
    Unit u0 = settle(Unit{0, DEAL && turns < 0 ? wave * blocks + in_order : in_order * kOneWaves + wave});
    if (u0.j < k) load(r0, u0);
    if (blockIdx.x == 0 && wave == 0) {  // the gates, for the last stage: behind the first requests
        const RouterPick pick = router_weigh(lane, E, logit, slot, vmax);
        if (slot >= 0) {
            a.idx[slot] = lane;
            a.gate[slot] = pick.p / pick.sel_sum;
        }
    }
    const int to_rest = stride + place_in_rest(in_order, wave, blocks) - (in_order * kOneWaves + wave);  // (from the last whole turn; one at least)
    auto next = [&](const Unit& u) { return settle(Unit{u.j, u.row + (DEAL && --turns == 0 ? to_rest : stride)}); };
    while (u0.j < k) {
        const Unit u1 = next(u0);
        if (u1.j < k) load(r1, u1);
        __builtin_amdgcn_sched_barrier(0);  // the requests stay ahead of the sums
        finish(r0, u0);
        if (u1.j >= k) break;
        u0 = next(u1);
        if (u0.j < k) load(r0, u0);
        __builtin_amdgcn_sched_barrier(0);
        finish(r1, u1);
    }
}

// A wave takes one slice of one (row, pair): chunks slice, slice + slices, ... -- NC of them, all
// requested before the first is used, the hidden vector's ahead of the expert's id.  16 waves hold
// 16 / (k slices) rows; their sums meet in LDS and are added in slice and pair order.
// 2048 x 5632, 46 MB: 10.0 us for 10.7, 1024 x 2816: 5.2 for 5.9 (there eight chunks at a time left a
// remainder of up to three that came one after the other).
// V: the stored type of the hidden vectors.
template <typename T, typename V, int NC>
__global__ __launch_bounds__(kOneWaves* kWave) __attribute__((amdgpu_waves_per_eu(4, 4))) void decode_last_kernel(
    ptr_arg ai, ptr_arg av, ptr_arg aW, long long stride, int n, int k, int slices, int E, int rows,
    const LastStage a) {
    const int32_t* idx = from_arg<const int32_t>(ai);
    const T* W = from_arg<const T>(aW);
    typedef typename Store<T>::vec_t vec_t;
    typedef typename Store<V>::vec_t vvec_t;
    constexpr int VEC = Store<T>::VEC, CH = kWave * VEC, VL = VEC / Store<V>::VEC;
    __shared__ float s_part[kOneWaves];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int per_row = k * slices, rows_here = kOneWaves / per_row;
    const int local_row = wave / per_row, q = wave - local_row * per_row;
    const int j = q / slices, slice = q - j * slices;
    const int row = min((int)blockIdx.x * rows_here + local_row, rows - 1);

    int off[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) off[c] = min((slice + c * slices) * CH + lane * VEC, n - VEC);
    const bool tail_in = (slice + (NC - 1) * slices) * CH + lane * VEC < n;
    const V* v = from_arg<const V>(av) + (size_t)j * n;
    vvec_t x[NC][VL];
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int l = 0; l < VL; ++l) x[c][l] = *reinterpret_cast<const vvec_t*>(v + off[c] + l * Store<V>::VEC);
    __builtin_amdgcn_sched_barrier(0);
    const int e = min(max(idx[j], 0), E - 1);
    const T* w = W + (size_t)e * stride + (size_t)row * n;
    vec_t wv[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) wv[c] = __builtin_nontemporal_load(reinterpret_cast<const vec_t*>(w + off[c]));
    // what the last step needs beside the sums
    const int my_row = (int)blockIdx.x * rows_here + (int)threadIdx.x;
    const bool mine = (int)threadIdx.x < rows_here && my_row < rows;
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
        for (int jj = 0; jj < k; ++jj) {
            float sum = 0.f;
            for (int sl = 0; sl < slices; ++sl) sum += s_part[threadIdx.x * per_row + jj * slices + sl];
            total = fmaf(a.gate[jj], sum, total);
        }
        static_cast<T*>(a.y)[my_row] = Store<T>::from_f32(total + res);
    }
}

// ---- a shared base (M_e = M0 + L_e R_e) ---------------------------------------------------------------
// The base's products are the bytes of the layer and none of them waits for the low-rank ones: they run
// beside the rank products in the first launch and beside the rank-down product in the third, and two
// launches of this kernel add the low-rank part.  64 / lanes rows per wave (a row of L is r long: 128
// bytes at rank 64), two pairs' rows requested at once.
// (2048 x 5632, rank 128: layer 27.0 us.  Rank 64: 25.4 us, 40.8 in five launches one after the other, and 21.8 in three, as below.)
//   HIDDEN: h_j = silu(b0 + L0_j t0_j) * (b1 + L1_j t1_j) and their mix b0 <- sum_j gate_j h_j; without a
//           base (b0 NULL) the hidden vectors alone
//   else:   y = b0 + sum_j gate_j L0_j t0_j (+ residual)
constexpr int kLowRankWaves = 4;
template <typename T, bool HIDDEN>
__global__ __launch_bounds__(kLowRankWaves* kWave) void decode_low_rank_kernel(
    ptr_arg ai, ptr_arg aL, ptr_arg at0, long long stride, int r, int rows, int k, int lanes, int E,
    const LowRankStage a) {
    const int32_t* idx = from_arg<const int32_t>(ai);
    const T* L0 = from_arg<const T>(aL);
    const float* t0 = from_arg<const float>(at0);
    typedef typename Store<T>::vec_t vec_t;
    constexpr int VEC = Store<T>::VEC;
    const int lane = threadIdx.x & (kWave - 1);
    const int group = lane / lanes, sub = lane - group * lanes, per_wave = kWave / lanes;
    const int row_at = ((int)blockIdx.x * kLowRankWaves + (int)(threadIdx.x / kWave)) * per_wave + group;
    const int row = min(row_at, rows - 1);
    const bool mine = sub == 0 && row_at < rows;
    const bool base = !HIDDEN || a.b0;
    const float b0 = base ? a.b0[row] : 0.f, b1 = HIDDEN && base ? a.b1[row] : 0.f;
    float res = 0.f;
    if (!HIDDEN && a.residual) res = Store<T>::to_f32(static_cast<const T*>(a.residual)[row]);
    float mix = 0.f;
    for (int j0 = 0; j0 < k; j0 += 2) {
        float acc[2][2] = {{0.f, 0.f}, {0.f, 0.f}};
        const T* l[2][2];
        const float* t[2][2];
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int j = min(j0 + p, k - 1);
            const int e = min(max(idx[j], 0), E - 1);
            const size_t at = (size_t)e * stride + (size_t)row * r;
            l[p][0] = L0 + at;
            t[p][0] = t0 + (size_t)j * r;
            l[p][1] = HIDDEN ? static_cast<const T*>(a.L1) + at : l[p][0];
            t[p][1] = HIDDEN ? a.t1 + (size_t)j * r : t[p][0];
        }
        for (int i = sub * VEC; i < r; i += lanes * VEC) {
            vec_t w[2][2];
            f32x4 v[2][2][VEC / 4];
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int m = 0; m < (HIDDEN ? 2 : 1); ++m) {
                    w[p][m] = __builtin_nontemporal_load(reinterpret_cast<const vec_t*>(l[p][m] + i));
#pragma unroll
                    for (int q = 0; q < VEC / 4; ++q) v[p][m][q] = *reinterpret_cast<const f32x4*>(t[p][m] + i + 4 * q);
                }
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int m = 0; m < (HIDDEN ? 2 : 1); ++m)
#pragma unroll
                    for (int q = 0; q < VEC; ++q) acc[p][m] = fmaf(Store<T>::get(w[p][m], q), v[p][m][q / 4][q % 4], acc[p][m]);
        }
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            for (int o = 1; o < lanes; o *= 2) {
                acc[p][0] += __shfl_xor(acc[p][0], o, kWave);
                if (HIDDEN) acc[p][1] += __shfl_xor(acc[p][1], o, kWave);
            }
            if (j0 + p < k) {
                const float g = a.gate[j0 + p];
                if (HIDDEN) {
                    const float h = silu_f32(b0 + acc[p][0]) * (b1 + acc[p][1]);
                    if (mine) a.h[(size_t)(j0 + p) * rows + row] = h;
                    mix = fmaf(g, h, mix);
                } else {
                    mix = fmaf(g, acc[p][0], mix);
                }
            }
        }
    }
    if (!mine) return;
    if (HIDDEN) {
        if (base) a.b0[row] = mix;  // read above by this group of lanes alone
    } else
        static_cast<T*>(a.y)[row] = Store<T>::from_f32(b0 + mix + res);
}

// ---- rank experts without a base (M_e = L_e R_e) --------------------------------------------------------
// h_j = silu(L0_j t0_j) * (L1_j t1_j) for rows of r > 256: a wave belongs to one pair, whose two rank vectors
// it keeps in registers, and requests both rows of its next unit before it sums the current one.
// turns: the order of the units (hidden_turns); DEAL: it is not 0 (a layer of one turn, 720 / 1936 of rank 264, 14.4 us without this / 14.2).
// NC: 1 KB chunks per row.
template <typename T, int NC, bool DEAL>
__global__ __launch_bounds__(kOneWaves* kWave) __attribute__((amdgpu_waves_per_eu(4, 4))) void decode_hidden_kernel(
    ptr_arg ai, ptr_arg aL0, ptr_arg aL1, long long stride, int n, int rows, int k, int E, int waves /* per pair */, int turns,
    const LowRankStage a) {
    const int32_t* idx = from_arg<const int32_t>(ai);
    typedef Store<T> S;
    typedef typename S::vec_t vec_t;
    constexpr int VEC = S::VEC, CH = kWave * VEC;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int at = DEAL && turns < 0 ? wave * (int)gridDim.x + (int)blockIdx.x : (int)blockIdx.x * kOneWaves + wave;
    int row = uniform_div(at, k);
    const int j = at - row * k;
    if (row >= waves || row >= rows) return;
    int off[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) off[c] = min(c * CH + lane * VEC, n - VEC);
    const bool tail_in = (NC - 1) * CH + lane * VEC < n;
    const int e = min(max(idx[j], 0), E - 1);
    const T* L0 = from_arg<const T>(aL0) + (size_t)e * stride;
    const T* L1 = from_arg<const T>(aL1) + (size_t)e * stride;
    float* h = a.h + (size_t)j * rows;
    struct Rows {
        vec_t w0[NC], w1[NC];
    };
    auto load = [&](Rows& r, int i) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            r.w0[c] = __builtin_nontemporal_load(reinterpret_cast<const vec_t*>(L0 + (size_t)i * n + off[c]));
            r.w1[c] = __builtin_nontemporal_load(reinterpret_cast<const vec_t*>(L1 + (size_t)i * n + off[c]));
        }
    };
    Rows r0, r1;
    load(r0, row);
    f32x4 t0[NC][VEC / 4], t1[NC][VEC / 4];
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int q = 0; q < VEC / 4; ++q) {
            t0[c][q] = *reinterpret_cast<const f32x4*>(a.t0 + (size_t)j * n + off[c] + 4 * q);
            t1[c][q] = *reinterpret_cast<const f32x4*>(a.t1 + (size_t)j * n + off[c] + 4 * q);
            if (c + 1 == NC && !tail_in) t0[c][q] = t1[c][q] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    auto finish = [&](Rows& r, int i) {
        float s0 = 0.f, s1 = 0.f;
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int q = 0; q < VEC; ++q) {
                const bool in = c + 1 < NC || tail_in;
                s0 = fmaf(in ? S::get(r.w0[c], q) : 0.f, t0[c][q / 4][q % 4], s0);
                s1 = fmaf(in ? S::get(r.w1[c], q) : 0.f, t1[c][q / 4][q % 4], s1);
            }
        s0 = wave_sum(s0);
        s1 = wave_sum(s1);
        if (lane == 0) h[i] = silu_f32(s0) * s1;
    };
    const int to_rest = waves + place_in_rest((int)blockIdx.x, uniform_div(wave, k), kOneCus) - row;  // (from the last whole turn)
    auto next_of = [&](int i) { return i + (DEAL && --turns == 0 ? to_rest : waves); };
    for (;;) {
        const int next = next_of(row);
        if (next < rows) load(r1, next);
        __builtin_amdgcn_sched_barrier(0);  // the requests stay ahead of the sums
        finish(r0, row);
        if (next >= rows) return;
        row = next_of(next);
        if (row < rows) load(r0, row);
        __builtin_amdgcn_sched_barrier(0);
        finish(r1, next);
        if (row >= rows) return;
    }
}

// td_j = R_d,j h_j for every pair, and y0 = M0_down mix: rows of one length against fp32 vectors, `slices`
// waves each, NC chunks a wave and all of them requested at once.  (d = 0: the pairs alone)
constexpr int kMidWaves = 8;
template <typename T, int NC>
__global__ __launch_bounds__(kMidWaves* kWave) __attribute__((amdgpu_waves_per_eu(4, 8))) void decode_mid_kernel(
    ptr_arg ai, ptr_arg ard, ptr_arg aw, long long stride, int n, int slices, int r, int k, int d, int E,
    const MidStage a) {
    const int32_t* idx = from_arg<const int32_t>(ai);
    typedef typename Store<T>::vec_t vec_t;
    constexpr int VEC = Store<T>::VEC, CH = kWave * VEC, VL = VEC / 4;
    __shared__ float s_part[kMidWaves];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int slice = wave % slices, rows_here = kMidWaves / slices;
    const int low = k * r, units = low + d;
    const int u_at = (int)blockIdx.x * rows_here + wave / slices, u = min(u_at, units - 1);
    int off[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) off[c] = min((slice + c * slices) * CH + lane * VEC, n - VEC);
    const bool tail_in = (slice + (NC - 1) * slices) * CH + lane * VEC < n;
    const float* v;
    const T* w;
    float* out;
    if (u < low) {
        const int j = u / r, e = min(max(idx[j], 0), E - 1);
        w = from_arg<const T>(ard) + (size_t)e * stride + (size_t)(u - j * r) * n;
        v = a.h + (size_t)j * n;
        out = a.td + u;
    } else {
        w = from_arg<const T>(aw) + (size_t)(u - low) * n;
        v = a.mix;
        out = a.y0 + (u - low);
    }
    vec_t wv[NC];
    f32x4 x[NC][VL];
#pragma unroll
    for (int c = 0; c < NC; ++c) wv[c] = __builtin_nontemporal_load(reinterpret_cast<const vec_t*>(w + off[c]));
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int l = 0; l < VL; ++l) x[c][l] = *reinterpret_cast<const f32x4*>(v + off[c] + 4 * l);
    __builtin_amdgcn_sched_barrier(0);
    float s = 0.f;
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
            const bool in = c + 1 < NC || tail_in;
            s = fmaf(in ? Store<T>::get(wv[c], i) : 0.f, in ? x[c][i / 4][i % 4] : 0.f, s);
        }
    s = wave_sum(s);
    if (lane == 0) s_part[wave] = s;
    __syncthreads();
    if (slice == 0 && lane == 0 && u_at < units) {
        float sum = 0.f;
        for (int sl = 0; sl < slices; ++sl) sum += s_part[wave + sl];
        *out = sum;
    }
}

// ---- a shared base, rank-down products in parts ---------------------------------------------------------------
// td_j = R_d,j h_j is a sum over the hidden rows, so a workgroup that forms 64 of them adds up its share of all k r
// sums while it has them, from columns of R_d that it requested at its start, and the last stage, every workgroup of
// which needs all of td, adds up the workgroups' shares (45 KB at 2048 x 5632, rank 64) under its stream of base
// rows: a launch less, and no hidden vectors in memory.  2048 x 5632, rank 64: 10.0 + 4.4 + 8.7 us in the trace, layer 23.9 -> 21.9; 12 shapes of 400 to
// 2048 wide, 2 and 4 experts, 1.07 times as fast (geometric mean, 1.03 the least).  Up to 64 sums per hidden row of a workgroup and
// pair: longer ranks would take more hidden rows a workgroup, or the parts more room than the vectors whose place they take (128
// rows a workgroup, rank 128: 512 x 1400 14.6 -> 19.0, 2048 x 5632 27.0 -> 28.0).
//   decode_base_hidden_kernel  h_j and their mix as decode_low_rank_kernel, parts[block][j][:] = R_d,j[:, its rows] h_j
//   decode_base_last_kernel    y = W_down mix + sum_j gate_j L_d,j td_j (+ residual)
// NQ: 64 rows of the k R_d's each.
constexpr int kBaseRows = 64;
template <typename T, int NQ>
__global__ __launch_bounds__(8 * kBaseRows) void decode_base_hidden_kernel(
    ptr_arg ai, ptr_arg ard, ptr_arg aL0, ptr_arg aL1, int r, int rows, int k, int lanes, int E, const BaseHiddenStage a) {
    typedef typename Store<T>::vec_t vec_t;
    constexpr int VEC = Store<T>::VEC, FB = kBaseRows, THREADS = 8 * FB, CHUNKS = FB / VEC;  // 16-byte chunks of a row of R_d here
    static_assert(THREADS / CHUNKS == 64 && CHUNKS == 8, "64 rows of R_d at a time, a row in eight lanes");
    __shared__ f32x4 s_h[kBasePairs][FB / 4];
    const int32_t* idx = from_arg<const int32_t>(ai);
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int f0 = (int)blockIdx.x * FB, kr = k * r;
    const int my_e = min(max(idx[min(lane, k - 1)], 0), E - 1);  // lane j: the j-th expert
    // the columns of R_d: nothing of what they meet is needed to request them
    const int chunk = threadIdx.x % CHUNKS;
    const bool chunk_in = f0 + chunk * VEC < rows;  // (rows is a multiple of VEC)
    vec_t rd[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int at = min((int)threadIdx.x / CHUNKS + q * 64, kr - 1), j = quick_div(at, r);
        const int e = __shfl(my_e, j, kWave);
        rd[q] = __builtin_nontemporal_load(reinterpret_cast<const vec_t*>(
            from_arg<const T>(ard) + ((size_t)e * r + (at - j * r)) * rows + min(f0 + chunk * VEC, rows - VEC)));
    }
    __builtin_amdgcn_sched_barrier(0);
    const int group = lane / lanes, sub = lane & (lanes - 1), per_wave = kWave / lanes;
    for (int local = wave * per_wave + group; local < FB; local += THREADS / lanes) {
        const int row = min(f0 + local, rows - 1);
        const bool mine = sub == 0 && f0 + local < rows;
        const float b0 = a.b0[row], b1 = a.b1[row];
        const int i = min(sub * VEC, r - VEC);
        const bool in = sub * VEC < r;
        float mix = 0.f;
        for (int j0 = 0; j0 < k; j0 += 2) {
            vec_t w[2][2];
            f32x4 v[2][2][VEC / 4];
            float g[2];
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const int j = min(j0 + p, k - 1), e = MOE_READLANE(my_e, j);
                const size_t at = ((size_t)e * rows + row) * r + i;
                w[p][0] = __builtin_nontemporal_load(reinterpret_cast<const vec_t*>(from_arg<const T>(aL0) + at));
                w[p][1] = __builtin_nontemporal_load(reinterpret_cast<const vec_t*>(from_arg<const T>(aL1) + at));
#pragma unroll
                for (int q = 0; q < VEC / 4; ++q) {
                    v[p][0][q] = *reinterpret_cast<const f32x4*>(a.t0 + (size_t)j * r + i + 4 * q);
                    v[p][1][q] = *reinterpret_cast<const f32x4*>(a.t1 + (size_t)j * r + i + 4 * q);
                }
                g[p] = a.gate[j];
            }
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                float acc[2] = {0.f, 0.f};
#pragma unroll
                for (int m = 0; m < 2; ++m)
#pragma unroll
                    for (int q = 0; q < VEC; ++q) acc[m] = fmaf(in ? Store<T>::get(w[p][m], q) : 0.f, in ? v[p][m][q / 4][q % 4] : 0.f, acc[m]);
                for (int o = 1; o < lanes; o *= 2) {
                    acc[0] += __shfl_xor(acc[0], o, kWave);
                    acc[1] += __shfl_xor(acc[1], o, kWave);
                }
                if (j0 + p < k) {
                    const float h = silu_f32(b0 + acc[0]) * (b1 + acc[1]);
                    if (sub == 0) reinterpret_cast<float*>(&s_h[j0 + p][0])[local] = mine ? h : 0.f;
                    mix = fmaf(g[p], h, mix);
                }
            }
        }
        if (mine) a.b0[row] = mix;  // read above by this group of lanes alone
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int at = min((int)threadIdx.x / CHUNKS + q * 64, kr - 1), j = quick_div(at, r);
        const f32x4 lo = s_h[j][chunk * 2], hi = s_h[j][chunk * 2 + 1];
        float s = 0.f;
#pragma unroll
        for (int c = 0; c < 4; ++c) s = fmaf(chunk_in ? Store<T>::get(rd[q], c) : 0.f, lo[c], s);
#pragma unroll
        for (int c = 0; c < 4; ++c) s = fmaf(chunk_in ? Store<T>::get(rd[q], 4 + c) : 0.f, hi[c], s);
        s += dpp_f32<kDppSwap1>(s);
        s += dpp_f32<kDppSwap2>(s);
        s += dpp_f32<kDppHalfMirror>(s);
        if (chunk == 0 && (int)threadIdx.x / CHUNKS + q * 64 < kr) a.parts[(size_t)blockIdx.x * kr + at] = s;
    }
}

// A wave takes a slice of a base row, all its chunks requested before anything else but the parts.
template <typename T, int NC>
__global__ __launch_bounds__(kOneWaves* kWave) __attribute__((amdgpu_waves_per_eu(4, 4))) void decode_base_last_kernel(
    ptr_arg aw, ptr_arg ap, ptr_arg av, ptr_arg ai, ptr_arg ag, int n, int slices, int r, int k, int blocks, int rows, const BaseLastStage a) {
    typedef typename Store<T>::vec_t vec_t;
    constexpr int VEC = Store<T>::VEC, CH = kWave * VEC, VL = VEC / 4, NB = 4;
    __shared__ f32x4 s_sum[kOneWaves * kWave];
    __shared__ float s_td[kBaseSums], s_part[kOneWaves];
    const int32_t* idx = from_arg<const int32_t>(ai);
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int local_row = uniform_div(wave, slices), slice = wave - local_row * slices, rows_here = uniform_div(kOneWaves, slices);
    const int row = min((int)blockIdx.x * rows_here + local_row, rows - 1);
    // the parts: thread (share, four sums) adds up blocks share, share + shares, ...
    const int kr = k * r, quads = kr / 4, shares = min(uniform_div(kOneWaves * kWave, quads), (blocks + NB - 1) / NB);
    const int share = quick_div(threadIdx.x, quads), quad = (int)threadIdx.x - share * quads;
    const f32x4* const parts = from_arg<const f32x4>(ap) + quad;
    const bool adds = share < shares;
    f32x4 pv[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) pv[b] = parts[(size_t)min(share + b * shares, blocks - 1) * quads];
    // the low-rank rows' place and gate (lane: 8 of the k r elements; thread: one of them)
    const int l_at = min(lane * VEC, kr - VEC), l_j = quick_div(l_at, r), l_e = idx[l_j];
    const int t_at = min((int)threadIdx.x, kr - 1);
    const float gate = from_arg<const float>(ag)[quick_div(t_at, r)];
    int off[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) off[c] = min((slice + c * slices) * CH + lane * VEC, n - VEC);
    const bool tail_in = (slice + (NC - 1) * slices) * CH + lane * VEC < n;
    const T* w = from_arg<const T>(aw) + (size_t)row * n;
    vec_t wv[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) wv[c] = __builtin_nontemporal_load(reinterpret_cast<const vec_t*>(w + off[c]));
    __builtin_amdgcn_sched_barrier(0);
    f32x4 sum = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int b = 0; b < NB; ++b)
        if (adds && share + b * shares < blocks) sum += pv[b];
    for (int b = share + NB * shares; adds && b < blocks; b += shares) sum += parts[(size_t)b * quads];
    if (adds) s_sum[share * quads + quad] = sum;
    const int e = min(max(l_e, 0), a.E - 1);
    const vec_t l = __builtin_nontemporal_load(
        reinterpret_cast<const vec_t*>(static_cast<const T*>(a.ld) + ((size_t)e * rows + row) * r + (l_at - l_j * r)));
    f32x4 x[NC][VL];
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int i = 0; i < VL; ++i) x[c][i] = *reinterpret_cast<const f32x4*>(from_arg<const float>(av) + off[c] + 4 * i);
    const int my_row = (int)blockIdx.x * rows_here + (int)threadIdx.x;
    const bool mine = (int)threadIdx.x < rows_here && my_row < rows;
    // (not conditional, or the compiler waits for it, and all before it, where the branch ends; w_down: any valid place)
    const T res = *(a.residual ? static_cast<const T*>(a.residual) + min(my_row, rows - 1) : from_arg<const T>(aw));
    __syncthreads();
    if ((int)threadIdx.x < kr) {
        const float* const sums = reinterpret_cast<const float*>(s_sum) + threadIdx.x;
        float td = 0.f;
        for (int i = 0; i < shares; ++i) td += sums[i * kr];
        s_td[threadIdx.x] = gate * td;
    }
    __syncthreads();
    float s = 0.f;
    if (slice == 0 && lane * VEC < kr) {
#pragma unroll
        for (int i = 0; i < VEC; ++i) s = fmaf(Store<T>::get(l, i), s_td[lane * VEC + i], s);
    }
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
            const bool in = c + 1 < NC || tail_in;
            s = fmaf(in ? Store<T>::get(wv[c], i) : 0.f, in ? x[c][i / 4][i % 4] : 0.f, s);
        }
    s = wave_sum(s);
    if (lane == 0) s_part[wave] = s;
    __syncthreads();
    if (mine) {
        float total = a.residual ? Store<T>::to_f32(res) : 0.f;
        for (int sl = 0; sl < slices; ++sl) total += s_part[threadIdx.x * slices + sl];
        static_cast<T*>(a.y)[my_row] = Store<T>::from_f32(total);
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
    const bool deal = a.turns || a.base_turns;
    const auto kern = swiglu ? (deal ? decode_first_kernel<T, NC, true, true> : decode_first_kernel<T, NC, true, false>)
                             : (deal ? decode_first_kernel<T, NC, false, true> : decode_first_kernel<T, NC, false, false>);
    hipLaunchKernelGGL(kern, grid, block, 0, st, as_arg(a.x), as_arg(a.router_w), as_arg(a.router_b), a.d, a.E, a.route_blocks, a);
}

template <typename T>
static int launch_first_t(FirstStage a, bool swiglu, hipStream_t st) {
    const long long units = (long long)a.k * a.rows;
    a.route_blocks = (int)std::min<long long>(kOneCus, (units + kOneWaves - 1) / kOneWaves);
    const int base_blocks = a.base_W0 ? std::max(kOneCus / 2, kOneCus - a.route_blocks) : 0;
    const int row_bytes = a.d * (int)sizeof(T);
    a.turns = first_stage_turns(units, a.route_blocks, row_bytes);
    a.base_turns = base_blocks ? first_stage_turns(a.base_rows, base_blocks, row_bytes) : 0;
    const dim3 grid(a.route_blocks + base_blocks);
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
        hipLaunchKernelGGL((decode_last_kernel<T, V, NC>), grid, block, 0, st, as_arg(a.idx), as_arg(a.v), as_arg(a.W), a.stride, a.n, a.k, a.slices, a.E, a.rows, a);
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

static int mid_slices(int units, int n) {
    const int chunks = chunks_of<bf16_t>(n);
    int s = 1;
    while ((chunks + s - 1) / s > last_max_chunks<bf16_t, float>()) s *= 2;
    while ((long long)units * s * 2 <= kOneCus * kOneWaves && chunks >= 4 * s) s *= 2;
    return s <= kMidWaves ? s : 0;
}

template <int NC>
static int launch_mid_nc(const MidStage& a, int nc, hipStream_t st) {
    if constexpr (NC > last_max_chunks<bf16_t, float>()) {
        return MOE_ERR_UNSUPPORTED;
    } else {
        if (nc != NC) return launch_mid_nc<NC + 1>(a, nc, st);
        const int rows_here = kMidWaves / a.slices;
        const dim3 grid((a.k * a.r + a.d + rows_here - 1) / rows_here), block(kMidWaves * kWave);
        hipLaunchKernelGGL((decode_mid_kernel<bf16_t, NC>), grid, block, 0, st, as_arg(a.idx), as_arg(a.rd), as_arg(a.w_down), a.stride, a.n, a.slices, a.r, a.k, a.d, a.E, a);
        return launch_status();
    }
}

// (the output's fp32 sums go where the base's up product lay: no wider than that)
bool decode_base_supported(const moe_shape& s) {
    return decode_first_supported(s) && s.act_dtype == MOE_BF16 && token_base_supported(s) && s.d_model <= s.d_ff &&
           (long long)s.top_k * s.rank + s.d_model < (1 << 24) && mid_slices(s.top_k * s.rank + s.d_model, s.d_ff) != 0;
}

// Slices per base row: as many as there are CUs for, a chunk at least to each
static int base_slices(int rows, int n) {
    const int chunks = chunks_of<bf16_t>(n);
    int s = 1;
    while ((chunks + s - 1) / s > last_max_chunks<bf16_t, float>()) s *= 2;
    while ((long long)rows * s * 2 <= kOneCus * kOneWaves && chunks >= 2 * s && s < kOneWaves) s *= 2;
    return s <= kOneWaves ? s : 0;
}

bool decode_base_parts_supported(const moe_shape& s) {
    return decode_base_supported(s) && s.rank <= kBaseRows && s.top_k * s.rank <= kBaseSums && base_slices(s.d_model, s.d_ff) != 0;
}

int launch_decode_base_hidden(BaseHiddenStage a, hipStream_t st) {
    a.lanes = 1;
    while (a.lanes * Store<bf16_t>::VEC < a.r) a.lanes *= 2;
    const auto kern = a.k * a.r <= 64    ? decode_base_hidden_kernel<bf16_t, 1>
                      : a.k * a.r <= 128 ? decode_base_hidden_kernel<bf16_t, 2>
                                         : decode_base_hidden_kernel<bf16_t, 4>;
    hipLaunchKernelGGL(kern, dim3((a.rows + kBaseRows - 1) / kBaseRows), dim3(8 * kBaseRows), 0, st, as_arg(a.idx), as_arg(a.rd), as_arg(a.L0), as_arg(a.L1),
                       a.r, a.rows, a.k, a.lanes, a.E, a);
    return launch_status();
}

template <int NC>
static int launch_base_last_nc(const BaseLastStage& a, int nc, hipStream_t st) {
    if constexpr (NC > last_max_chunks<bf16_t, float>()) {
        return MOE_ERR_UNSUPPORTED;
    } else {
        if (nc != NC) return launch_base_last_nc<NC + 1>(a, nc, st);
        const int rows_here = kOneWaves / a.slices;
        hipLaunchKernelGGL((decode_base_last_kernel<bf16_t, NC>), dim3((a.rows + rows_here - 1) / rows_here), dim3(kOneWaves * kWave), 0, st, as_arg(a.w_down),
                           as_arg(a.parts), as_arg(a.mix), as_arg(a.idx), as_arg(a.gate), a.n, a.slices, a.r, a.k, (a.n + kBaseRows - 1) / kBaseRows, a.rows, a);
        return launch_status();
    }
}
int launch_decode_base_last(BaseLastStage a, hipStream_t st) {
    a.slices = base_slices(a.rows, a.n);
    if (!a.slices) return MOE_ERR_UNSUPPORTED;
    return launch_base_last_nc<1>(a, (chunks_of<bf16_t>(a.n) + a.slices - 1) / a.slices, st);
}

int launch_decode_mid(MidStage a, hipStream_t st) {
    a.slices = mid_slices(a.k * a.r + a.d, a.n);
    if (!a.slices) return MOE_ERR_UNSUPPORTED;
    return launch_mid_nc<1>(a, (chunks_of<bf16_t>(a.n) + a.slices - 1) / a.slices, st);
}

int launch_decode_low_rank(LowRankStage a, bool hidden, hipStream_t st) {
    a.lanes = 1;
    while (a.lanes < kWave && a.lanes * Store<bf16_t>::VEC < a.r) a.lanes *= 2;
    const int per_block = kLowRankWaves * (kWave / a.lanes);
    const dim3 grid((a.rows + per_block - 1) / per_block), block(kLowRankWaves * kWave);
    if (hidden)
        hipLaunchKernelGGL((decode_low_rank_kernel<bf16_t, true>), grid, block, 0, st, as_arg(a.idx), as_arg(a.L0), as_arg(a.t0), a.stride, a.r, a.rows, a.k, a.lanes, a.E, a);
    else
        hipLaunchKernelGGL((decode_low_rank_kernel<bf16_t, false>), grid, block, 0, st, as_arg(a.idx), as_arg(a.L0), as_arg(a.t0), a.stride, a.r, a.rows, a.k, a.lanes, a.E, a);
    return launch_status();
}

constexpr int kHiddenMaxChunks = 3;  // (decode_hidden_kernel) two rank vectors and two units of two rows in 128 registers

bool decode_rank_supported(const moe_shape& s) {
    return decode_first_supported(s) && s.act_dtype == MOE_BF16 && s.rank > 0 && !(s.flags & MOE_FLAG_SHARED_BASE) &&
           s.top_k <= kOneCus && chunks_of<bf16_t>(s.rank) <= kHiddenMaxChunks && mid_slices(s.top_k * s.rank, s.d_ff) != 0;
}

int launch_decode_hidden(const LowRankStage& a, hipStream_t st) {
    if (a.r <= kWave / 2 * Store<bf16_t>::VEC) return launch_decode_low_rank(a, true, st);  // two and more rows per wave
    const long long units = (long long)a.k * a.rows;
    const dim3 grid((unsigned)std::min<long long>(kOneCus, (units + kOneWaves - 1) / kOneWaves)), block(kOneWaves * kWave);
    const int waves = (int)grid.x * kOneWaves / a.k;
    const int chunks = chunks_of<bf16_t>(a.r);
    if (chunks > kHiddenMaxChunks) return MOE_ERR_UNSUPPORTED;
    const int turns = hidden_turns(a.rows, waves, a.k, a.r * (int)sizeof(bf16_t));
    const auto kern = chunks == 1   ? (turns ? decode_hidden_kernel<bf16_t, 1, true> : decode_hidden_kernel<bf16_t, 1, false>)
                      : chunks == 2 ? (turns ? decode_hidden_kernel<bf16_t, 2, true> : decode_hidden_kernel<bf16_t, 2, false>)
                                    : (turns ? decode_hidden_kernel<bf16_t, 3, true> : decode_hidden_kernel<bf16_t, 3, false>);
    hipLaunchKernelGGL(kern, grid, block, 0, st, as_arg(a.idx), as_arg(a.L0), as_arg(a.L1), a.stride, a.r, a.rows, a.k, a.E, waves, turns, a);
    return launch_status();
}

}  // namespace moe
