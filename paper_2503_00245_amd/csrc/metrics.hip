// Routing-trace statistics the paper defines on the router's outputs:
//   - hard expert replacements H_e, H (Sec. 2.3, Eq. 4) and floor(H/2) of Eq. 5;
//   - the forward value of the block-wise expert selection loss (Eq. 4-7);
//   - set changes and expert loads under the offloading rule of Sec. 3.4.2;
//   - "Delta Uniform" (Sec. 3.2 metric list, Table 3, Fig. 6): per-layer divergence of the
//     realised expert balance from the uniform one, and its mean over layers.
// All integer work uses integer atomics (order-independent, hence deterministic); the one
// floating-point reduction (Eq. 6) sums fixed shares of the tokens in a fixed order and adds the
// shares' sums, again in a fixed order; both in fp64, but for the four differences of one load.
// What bounds these kernels is launches: each dependent one costs 4-5 us however little it does, and
// the data (2 MB for 24 layers of 2048 tokens) is read in about that time.  So every entry point is
// one or two launches, and what is left of serial work runs on a workgroup instead of a thread
// (all four calls on 24 x 2048 tokens, 2 of 8 experts: 120 us before, 28 now; on short traces, one launch each, 18).
#include "common.h"

namespace moe {

constexpr int kMetricThreads = 256;

// 64-bit mask of the experts selected for one token; entries outside [0, E) are dropped.
__device__ __forceinline__ unsigned long long expert_mask(const int32_t* __restrict__ s, int K,
                                                          int E) {
    unsigned long long m = 0;
    for (int j = 0; j < K; ++j) {
        const int e = s[j];
        if ((unsigned)e < (unsigned)E) m |= 1ull << e;
    }
    return m;
}

__global__ __launch_bounds__(kMetricThreads) void zero_counters_kernel(ptr_arg ap, int n, ptr_arg aq) {
    unsigned long long *const p = from_arg<unsigned long long>(ap), *const q = from_arg<unsigned long long>(aq);
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
    if (q && i == 0) *q = 0;
}

// Expert sets that differ between tokens i and i + 1 of the flattened [B, T] tokens (0 when token i
// is its sequence's last, or lies at or beyond `end`).
__device__ __forceinline__ unsigned long long replaced_set(const int32_t* __restrict__ S, int i, int end,
                                                           int T, int K, int E) {
    if (i >= end || i % T == T - 1) return 0ull;
    const int32_t* s0 = S + (size_t)i * K;
    return expert_mask(s0, K, E) ^ expert_mask(s0 + K, K, E);
}

// One thread per token: H_e[e] += [e in S(b,t+1)] xor [e in S(b,t)], H += the same over all e.  He and H
// start at zero.  (H is added here, one atomic per workgroup, and not by a kernel of its own: a
// dependent launch costs 4-5 us, whatever it does.)
__global__ __launch_bounds__(kMetricThreads) void replacements_kernel(
    ptr_arg aS, int B, int T, int K, int E, ptr_arg aHe, ptr_arg aH) {
    const int32_t* const S = from_arg<const int32_t>(aS);
    unsigned long long *const He = from_arg<unsigned long long>(aHe), *const H = from_arg<unsigned long long>(aH);
    __shared__ int s_cnt[kMaxExperts];
    if (threadIdx.x < kMaxExperts) s_cnt[threadIdx.x] = 0;
    __syncthreads();
    unsigned long long diff =
        replaced_set(S, blockIdx.x * kMetricThreads + threadIdx.x, B * T, T, K, E);
    while (diff) {
        const int e = __ffsll((long long)diff) - 1;
        atomicAdd(&s_cnt[e], 1);
        diff &= diff - 1;
    }
    __syncthreads();
    if (threadIdx.x < kMaxExperts) {  // one wave
        const int c = s_cnt[threadIdx.x];
        if (c) atomicAdd(&He[threadIdx.x], (unsigned long long)c);
        int all = c;
#pragma unroll
        for (int m = 1; m < kWave; m <<= 1) all += __shfl_xor(all, m, kWave);
        if (threadIdx.x == 0 && all) atomicAdd(H, (unsigned long long)all);
    }
}

// Partial sums of a workgroup's share of the tokens, soft part |W[b,t+1,e] - W[b,t,e]| and hard part
// (number of replaced experts), to soft_part[block] and hard_part[block].  Nothing is accumulated in memory,
// so nothing has to be cleared first.
__global__ __launch_bounds__(kMetricThreads) void bles_partial_kernel(
    ptr_arg aW, ptr_arg aS, int B, int T, int K, int E, int tokens_per_block, int vec, ptr_arg a_soft, ptr_arg a_hard) {
    const float* const W = from_arg<const float>(aW);
    const int32_t* const S = from_arg<const int32_t>(aS);
    double* const soft_part = from_arg<double>(a_soft);
    int* const hard_part = from_arg<int>(a_hard);
    __shared__ double s_soft[kMetricThreads / kWave];
    __shared__ int s_hard[kMetricThreads / kWave];
    const int t0 = blockIdx.x * tokens_per_block;
    const int t1 = min(B * T, t0 + tokens_per_block);
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    int hard = 0;
    for (int i = t0 + threadIdx.x; i < t1; i += kMetricThreads) hard += __popcll(replaced_set(S, i, t1, T, K, E));
    double soft = 0.0;
    if (vec) {  // rows of W are whole, aligned 16-byte chunks
        const int q = E / 4;
        const f32x4* w = reinterpret_cast<const f32x4*>(W);
        for (int c = t0 * q + threadIdx.x; c < t1 * q; c += kMetricThreads) {
            if ((c / q) % T == T - 1) continue;
            const f32x4 v = w[c + q] - w[c];
            soft += (double)((fabsf(v[0]) + fabsf(v[1])) + (fabsf(v[2]) + fabsf(v[3])));
        }
    } else {
        for (int c = t0 * E + threadIdx.x; c < t1 * E; c += kMetricThreads)
            if ((c / E) % T != T - 1) soft += (double)fabsf(W[c + E] - W[c]);
    }
#pragma unroll
    for (int m = 1; m < kWave; m <<= 1) {
        soft += __shfl_xor(soft, m, kWave);
        hard += __shfl_xor(hard, m, kWave);
    }
    if (lane == 0) {
        s_soft[wave] = soft;
        s_hard[wave] = hard;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kMetricThreads / kWave; ++w) {
            soft += s_soft[w];
            hard += s_hard[w];
        }
        soft_part[blockIdx.x] = soft;
        hard_part[blockIdx.x] = hard;
    }
}

// out = {H, H_norm, L, L_norm, loss} (Eq. 5, 6, 7)
__device__ __forceinline__ void write_bles(double* out, double L, unsigned long long H, int B, int T, int K) {
    const double Hn = T > 1 ? (double)(H / 2) / ((double)B * K * (T - 1)) : 0.0;
    const double Ln = L / ((double)B * T);
    out[0] = (double)H;
    out[1] = Hn;
    out[2] = L;
    out[3] = Ln;
    out[4] = Hn * Ln;
}

// One workgroup: thread i adds the partials
// i, i + 256, ... in fp64 and the threads meet in a fixed tree (deterministic).  (One thread adding
// all of them was a chain of 1536 dependent load-and-adds at 24 x 2048 tokens: 64 us.)
__global__ __launch_bounds__(kMetricThreads) void bles_finalize_kernel(
    ptr_arg a_soft, ptr_arg a_hard, int nblocks, int B, int T, int K, ptr_arg a_out) {
    const double* const soft_part = from_arg<const double>(a_soft);
    const int* const hard_part = from_arg<const int>(a_hard);
    double* const out = from_arg<double>(a_out);
    __shared__ double s_soft[kMetricThreads];
    __shared__ unsigned long long s_hard[kMetricThreads];
    double L = 0.0;
    unsigned long long H = 0;
    for (int i = threadIdx.x; i < nblocks; i += kMetricThreads) {
        L += soft_part[i];
        H += (unsigned)hard_part[i];
    }
    s_soft[threadIdx.x] = L;
    s_hard[threadIdx.x] = H;
    __syncthreads();
    for (int off = kMetricThreads / 2; off > 0; off >>= 1) {
        if (threadIdx.x < off) {
            s_soft[threadIdx.x] += s_soft[threadIdx.x + off];
            s_hard[threadIdx.x] += s_hard[threadIdx.x + off];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) write_bles(out, s_soft[0], s_hard[0], B, T, K);
}

// ---- short traces: one workgroup, one launch ------------------------------------------------------------------
// What takes two launches for want of a sum over workgroups takes one where a single workgroup reads the whole trace in less
// time than the other launch costs on the GPU.  Several turns' loads are requested together: none is conditional.
constexpr int kOneThreads = 1024, kOneWaves = kOneThreads / kWave, kOneTurns = 4;
// Up to here lane e counts expert e by ballots, above by LDS atomics (3072 tokens, 4 and 8 experts, 3.2 and 3.7 us against 5.3 and
// 5.1; 2048 tokens, 16 experts, 4.6 against 3.6)
constexpr int kBallotExperts = 8;

// Experts replaced after token i of the n = B T (two at least), K of them selected per token
template <int K>
__device__ __forceinline__ unsigned long long replaced_after(const int32_t* __restrict__ S, int i, int n, int T, int E) {
    const int32_t* s0 = S + (size_t)min(i, n - 2) * K;
    const unsigned long long d = expert_mask(s0, K, E) ^ expert_mask(s0 + K, K, E);
    return i < n - 1 && i % T != T - 1 ? d : 0ull;
}

template <int K>
__global__ __launch_bounds__(kOneThreads) void replacements_one_kernel(ptr_arg aS, int B, int T, int E, ptr_arg aHe, ptr_arg aH) {
    const int32_t* const S = from_arg<const int32_t>(aS);
    __shared__ int s_cnt[kOneWaves][kMaxExperts];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave, n = B * T;
    s_cnt[wave][lane] = 0;
    __syncthreads();
    int mine = 0;
    for (int i0 = wave * kWave; i0 < n; i0 += kOneTurns * kOneThreads) {
        unsigned long long d[kOneTurns];
#pragma unroll
        for (int u = 0; u < kOneTurns; ++u) d[u] = replaced_after<K>(S, i0 + lane + u * kOneThreads, n, T, E);
        if (E <= kBallotExperts) {
            for (int e = 0; e < E; ++e) {
                int c = 0;
#pragma unroll
                for (int u = 0; u < kOneTurns; ++u) c += __popcll(__ballot(d[u] >> e & 1));
                mine += lane == e ? c : 0;
            }
        } else {
#pragma unroll
            for (int u = 0; u < kOneTurns; ++u)
                for (; d[u]; d[u] &= d[u] - 1) atomicAdd(&s_cnt[wave][__ffsll((long long)d[u]) - 1], 1);
        }
    }
    if (E <= kBallotExperts) s_cnt[wave][lane] = mine;
    __syncthreads();
    if (wave != 0) return;
    unsigned long long c = 0;
    for (int w = 0; w < kOneWaves; ++w) c += (unsigned)s_cnt[w][lane];
    if (lane < E) from_arg<unsigned long long>(aHe)[lane] = c;
#pragma unroll
    for (int m = 1; m < kWave; m <<= 1) c += __shfl_xor(c, m, kWave);
    if (lane == 0) *from_arg<unsigned long long>(aH) = c;
}

template <int K>
__global__ __launch_bounds__(kOneThreads) void bles_one_kernel(ptr_arg aW, ptr_arg aS, int B, int T, int E, int vec, ptr_arg a_out) {
    const float* const W = from_arg<const float>(aW);
    const int32_t* const S = from_arg<const int32_t>(aS);
    __shared__ double s_soft[kOneWaves];
    __shared__ unsigned long long s_hard[kOneWaves];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave, n = B * T;
    unsigned long long hard = 0;
    for (int i0 = threadIdx.x; i0 < n; i0 += kOneTurns * kOneThreads)
#pragma unroll
        for (int u = 0; u < kOneTurns; ++u) hard += __popcll(replaced_after<K>(S, i0 + u * kOneThreads, n, T, E));
    double soft = 0.0;
    const int q = vec ? E / 4 : E, last = (n - 2) * q + q - 1;  // chunks of a row, the last one with a successor
    for (int c0 = threadIdx.x; c0 <= last; c0 += kOneTurns * kOneThreads) {
        float d[kOneTurns];
#pragma unroll
        for (int u = 0; u < kOneTurns; ++u) {
            const int c = min(c0 + u * kOneThreads, last);
            if (vec) {  // rows of W are whole, aligned 16-byte chunks
                const f32x4* w = reinterpret_cast<const f32x4*>(W) + c;
                const f32x4 v = w[q] - w[0];
                d[u] = (fabsf(v[0]) + fabsf(v[1])) + (fabsf(v[2]) + fabsf(v[3]));
            } else {
                d[u] = fabsf(W[c + q] - W[c]);
            }
        }
#pragma unroll
        for (int u = 0; u < kOneTurns; ++u) {
            const int c = c0 + u * kOneThreads;
            if (c <= last && (c / q) % T != T - 1) soft += (double)d[u];
        }
    }
#pragma unroll
    for (int m = 1; m < kWave; m <<= 1) {
        soft += __shfl_xor(soft, m, kWave);
        hard += __shfl_xor(hard, m, kWave);
    }
    if (lane == 0) {
        s_soft[wave] = soft;
        s_hard[wave] = hard;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int w = 1; w < kOneWaves; ++w) {
        soft += s_soft[w];
        hard += s_hard[w];
    }
    write_bles(from_arg<double>(a_out), soft, hard, B, T, K);
}

constexpr int kOneLayers = 2 * kOneWaves;  // layers of a trace at most

// Waves take layers in turn.  The sums are those of the kernels below, in the same order.
__global__ __launch_bounds__(kOneThreads) void balance_one_kernel(
    ptr_arg a_trace, int L, int TK, int E, ptr_arg a_counts, ptr_arg a_delta, ptr_arg a_mean) {
    const int32_t* const trace = from_arg<const int32_t>(a_trace);
    double* const delta = from_arg<double>(a_delta);
    __shared__ int s_cnt[kOneWaves][kMaxExperts];
    __shared__ double s_dev[kOneWaves][kMaxExperts], s_delta[kOneLayers];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    for (int l0 = 0; l0 < L; l0 += kOneWaves) {  // (in step: the waves meet at the barriers)
        const int l = l0 + wave;
        s_cnt[wave][lane] = 0;
        __syncthreads();
        if (l < L) {
            const int32_t* tr = trace + (size_t)l * TK;
            for (int i0 = lane; i0 < TK; i0 += 2 * kOneTurns * kWave) {
                int e[2 * kOneTurns];
#pragma unroll
                for (int u = 0; u < 2 * kOneTurns; ++u) e[u] = tr[min(i0 + u * kWave, TK - 1)];
#pragma unroll
                for (int u = 0; u < 2 * kOneTurns; ++u)
                    if (i0 + u * kWave < TK && (unsigned)e[u] < (unsigned)E) atomicAdd(&s_cnt[wave][e[u]], 1);
            }
        }
        __syncthreads();
        if (l < L && lane < E) {
            const unsigned long long c = (unsigned)s_cnt[wave][lane];
            from_arg<unsigned long long>(a_counts)[(size_t)l * E + lane] = c;
            const double dev = (double)c / (double)TK - 1.0 / (double)E;
            s_dev[wave][lane] = dev < 0 ? -dev : dev;
        }
        __syncthreads();
        if (l < L && lane == 0) {
            double dl = 0.0;
#pragma unroll 8
            for (int e = 0; e < E; ++e) dl += s_dev[wave][e];
            if (delta) delta[l] = dl;
            s_delta[l] = dl;
        }
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    double total = 0.0;
    for (int l = 0; l < L; ++l) total += s_delta[l];
    *from_arg<double>(a_mean) = total / (double)L;
}

// Where that pays.  The host saves 2.5-3 us a call (two launches 7-8 us, one 4.6-5.2), but a call behind other work, or in a graph, costs
// its time on the GPU alone: the lines lie where that is longer by some half a microsecond at most.  In a graph of 64 calls, us a
// call, two launches / one:
//   replacements, 2 of 8 experts: 1024 tokens 3.9 / 3.2, 3072 3.9 / 3.7, 4096 3.9 / 4.0, 8192 3.8 / 5.7.  With atomics it matters how
//     often an expert is replaced: 2 of 16, random / the same four at every token: 1024 tokens 3.8 / 2.7 and 4.5 / 5.3, 2048 3.9 / 3.6 and
//     4.5 / 8.8, 3072 3.9 / 4.4 (1 of 16 3.7 / 3.2).  Four of 8 experts a token, whose loads are no constant number: 64 tokens 4.0 / 4.8; 4 of 16, 1024 tokens, 4.3 / 7.9
//   loss, 2 of 8: 2048 tokens 4.8 / 4.2, 3072 4.9 / 5.4, 4096 4.9 / 6.3; 2 of 16: 1024 tokens 5.1 / 4.1, 2048 5.1 / 5.5; 2 of 64: 256 tokens 6.1 /
//     3.8, 1024 6.5 / 8.0; 2 of 7, rows no whole chunks: 585 tokens 5.3 / 3.8, 2048 5.6 / 7.6
//   balance, random / Zipf / all tokens with the same experts, where the LDS atomics meet: 16 layers of 64 tokens, 2 of 2, 3.8 / 3.5 each;
//     2 layers of 1024, 2 of 4, 4.0 / 3.5, 4.1 / 3.5, 4.2 / 3.7; 8 of 512, 2 of 8, 4.3 / 3.7, 4.3 / 4.8, 4.3 / 5.6; 16 of 256 4.3 / 4.0, 4.3 / 5.1, 4.3 /
//     6.0; 16 of 512, 1 of 8, 4.4 / 4.0, 4.3 / 6.2, 4.4 / 9.4; two turns of the waves: 24 of 64, 4 of 16, 4.7 / 4.3, 27 of 64, 2 of 8, 4.2 / 4.6,
//     24 of 170 4.1 / 4.7, 24 of 341 4.4 / 6.5; 9 of 179, 8 of 8, 4.1 / 3.7; one layer, one wave, of 2048 3.9 / 4.7
constexpr int kOneTokens = 4096, kOneManyTokens = 3072, kOneChunks = 6144, kOnePairs = 16384, kOneLayerPairs = 2048;
// many: more experts than ballots are for, or layers than waves
static bool short_trace(int L, int T, bool many) { return (long long)L * T <= (many ? kOneManyTokens : kOneTokens); }

constexpr int kLayerThreads = 1024;  // kernels with one workgroup per layer
// Up to this many pairs a layer is one workgroup's: it reads 128 KB in about the 9 us that clearing the
// counters first and the second launch would add.
constexpr int kOneChunkPairs = 32768;

// one workgroup per layer: adjacent-token set comparisons (the resident set after token t is
// always S_t, so the rule's state is just the previous token's selection)
__global__ __launch_bounds__(kLayerThreads) void offload_kernel(
    ptr_arg a_trace, int T, int K, int E, ptr_arg a_changes, ptr_arg a_loads) {
    const int32_t* const trace = from_arg<const int32_t>(a_trace);
    unsigned long long *const changes = from_arg<unsigned long long>(a_changes), *const loads = from_arg<unsigned long long>(a_loads);
    __shared__ int s_ch, s_ld;
    if (threadIdx.x == 0) {
        s_ch = 0;
        s_ld = 0;
    }
    __syncthreads();
    const int32_t* tr = trace + (size_t)blockIdx.x * T * K;
    int ch = 0, ld = 0;
    for (int t = threadIdx.x; t < T; t += kLayerThreads) {
        const unsigned long long cur = expert_mask(tr + (size_t)t * K, K, E);
        const unsigned long long prev = t > 0 ? expert_mask(tr + (size_t)(t - 1) * K, K, E) : 0ull;
        if (cur != prev) {
            ch += 1;
            ld += __popcll(cur & ~prev);
        }
    }
#pragma unroll
    for (int m = 1; m < kWave; m <<= 1) {
        ch += __shfl_xor(ch, m, kWave);
        ld += __shfl_xor(ld, m, kWave);
    }
    if ((threadIdx.x & (kWave - 1)) == 0) {
        atomicAdd(&s_ch, ch);
        atomicAdd(&s_ld, ld);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        changes[blockIdx.x] = (unsigned long long)s_ch;
        loads[blockIdx.x] = (unsigned long long)s_ld;
    }
}

// counts[l][e] = pairs of layer l that chose expert e.  Grid: x = chunks of a layer, y = layers.  ONE: a
// single chunk, whose workgroup stores the layer's counts; otherwise they are added to counts, which
// start at zero.  Every wave counts in LDS of its own.
template <bool ONE>
__global__ __launch_bounds__(kLayerThreads) void balance_count_kernel(
    ptr_arg a_trace, int TK, int E, ptr_arg a_counts) {
    const int32_t* const trace = from_arg<const int32_t>(a_trace);
    unsigned long long* const counts = from_arg<unsigned long long>(a_counts);
    __shared__ int s_cnt[kLayerThreads / kWave][kMaxExperts];
    const int wave = threadIdx.x / kWave;
    for (int i = threadIdx.x; i < kLayerThreads / kWave * kMaxExperts; i += kLayerThreads) (&s_cnt[0][0])[i] = 0;
    __syncthreads();
    const int32_t* tr = trace + (size_t)blockIdx.y * TK;
    const int stride = gridDim.x * kLayerThreads;
    for (int i = blockIdx.x * kLayerThreads + threadIdx.x; i < TK; i += stride) {
        const int e = tr[i];
        if ((unsigned)e < (unsigned)E) atomicAdd(&s_cnt[wave][e], 1);
    }
    __syncthreads();
    if (threadIdx.x < E) {
        unsigned long long c = 0;
        for (int w = 0; w < kLayerThreads / kWave; ++w) c += s_cnt[w][threadIdx.x];
        unsigned long long* at = &counts[(size_t)blockIdx.y * E + threadIdx.x];
        if (ONE) *at = c;
        else if (c) atomicAdd(at, c);
    }
}

// delta[l] = sum_e | counts[l][e] / (T K) - 1/E |, summed in ascending e; mean = (sum_l delta[l]) / L
// in ascending l.  One workgroup, a thread per layer (kMetricThreads layers at a time): the fp64
// divisions, E per layer, are what takes time, and the layers' are independent.
__global__ __launch_bounds__(kMetricThreads) void balance_finalize_kernel(
    ptr_arg a_counts, int L, int TK, int E, ptr_arg a_delta, ptr_arg a_mean) {
    const unsigned long long* const counts = from_arg<const unsigned long long>(a_counts);
    double *const delta = from_arg<double>(a_delta), *const mean = from_arg<double>(a_mean);
    __shared__ double s_delta[kMetricThreads];
    double total = 0.0;
    for (int l0 = 0; l0 < L; l0 += kMetricThreads) {
        const int l = l0 + threadIdx.x;
        if (l < L) {
            double dl = 0.0;
#pragma unroll 4
            for (int e = 0; e < E; ++e) {
                const double dev = (double)counts[(size_t)l * E + e] / (double)TK - 1.0 / (double)E;
                dl += dev < 0 ? -dev : dev;
            }
            if (delta) delta[l] = dl;
            s_delta[threadIdx.x] = dl;
        }
        __syncthreads();
        if (threadIdx.x == 0)
            for (int i = 0; i < min(L - l0, kMetricThreads); ++i) total += s_delta[i];
        __syncthreads();
    }
    if (threadIdx.x == 0) *mean = total / (double)L;
}

}  // namespace moe

using namespace moe;

static int check_trace_shape(int B, int T, int K, int E) {
    if (B < 1 || T < 1 || K < 1 || E < 1 || K > E) return MOE_ERR_INVALID;
    if (E > kMaxExperts) return MOE_ERR_UNSUPPORTED;
    if ((long long)B * T * (long long)(E > K ? E : K) >= (1ll << 31)) return MOE_ERR_UNSUPPORTED;
    return MOE_OK;
}

extern "C" {

int moe_expert_replacements(const int32_t* S, int32_t B, int32_t T, int32_t K, int32_t E,
                            int64_t* H_e, int64_t* H, void* stream) {
    int rc = check_trace_shape(B, T, K, E);
    if (rc != MOE_OK) return rc;
    if (!S || !H_e || !H) return MOE_ERR_INVALID;
    hipStream_t st = as_stream(stream);
    unsigned long long* he = reinterpret_cast<unsigned long long*>(H_e);
    unsigned long long* h = reinterpret_cast<unsigned long long*>(H);
    if (T > 1 && K <= 2 && short_trace(B, T, E > kBallotExperts)) {
        const auto kern = K == 1 ? replacements_one_kernel<1> : replacements_one_kernel<2>;
        hipLaunchKernelGGL(kern, dim3(1), dim3(kOneThreads), 0, st, as_arg(S), B, T, E, as_arg(he), as_arg(h));
        return launch_status();
    }
    hipLaunchKernelGGL(zero_counters_kernel, dim3(1), dim3(kMetricThreads), 0, st, as_arg(he), E, as_arg(h));
    if (T > 1)
        hipLaunchKernelGGL(replacements_kernel, dim3((B * T - 1) / kMetricThreads + 1), dim3(kMetricThreads), 0, st,
                           as_arg(S), B, T, K, E, as_arg(he), as_arg(h));
    return launch_status();
}

size_t moe_bles_workspace_bytes(int32_t B, int32_t T, int32_t E) {
    if (check_trace_shape(B, T, 1, E) != MOE_OK) return 0;
    const long long n = (long long)B * (T > 1 ? T - 1 : 0) * E;
    const size_t nblocks = (size_t)((n + kMetricThreads - 1) / kMetricThreads);
    // [E+1] u64 replacement counters, then one float per block
    return round_up(sizeof(unsigned long long) * (kMaxExperts + 1), 256) +
           round_up(sizeof(float) * (nblocks ? nblocks : 1), 256);
}

int moe_bles_loss(const float* probs, const int32_t* S, int32_t B, int32_t T, int32_t K, int32_t E,
                  double* out, void* workspace, size_t workspace_bytes, void* stream) {
    int rc = check_trace_shape(B, T, K, E);
    if (rc != MOE_OK) return rc;
    if (!probs || !S || !out) return MOE_ERR_INVALID;
    if (!workspace || workspace_bytes < moe_bles_workspace_bytes(B, T, E)) return MOE_ERR_WORKSPACE;
    hipStream_t st = as_stream(stream);
    const int vec = E % 4 == 0 && aligned16(probs) ? 1 : 0;  // rows are whole 16-byte chunks
    if (T > 1 && K <= 2 && short_trace(B, T, false) && B * T * E / (vec ? 4 : 1) <= kOneChunks) {
        const auto kern = K == 1 ? bles_one_kernel<1> : bles_one_kernel<2>;
        hipLaunchKernelGGL(kern, dim3(1), dim3(kOneThreads), 0, st, as_arg(probs), as_arg(S), B, T, E, vec, as_arg(out));
        return launch_status();
    }
    // 12 bytes of partial sums per workgroup; the size query has room for 4 per 256 differences of W beside 768
    // bytes, and a workgroup takes at least 1024 elements, more where that is too many workgroups (T = 2)
    char* const first = reinterpret_cast<char*>(round_up(reinterpret_cast<uintptr_t>(workspace), sizeof(double)));
    const size_t room = moe_bles_workspace_bytes(B, T, E) - sizeof(double);
    const int max_blocks = (int)min(room / (sizeof(double) + sizeof(int)), (size_t)1 << 30);
    double* soft_part = reinterpret_cast<double*>(first);
    int* hard_part = nullptr;
    int nblocks = 0;
    if (T > 1) {
        const int tokens_per_block = max(max(kMetricThreads / 2, (4 * kMetricThreads + E - 1) / E), (B * T - 1) / max_blocks + 1);
        nblocks = (B * T - 1) / tokens_per_block + 1;
        hard_part = reinterpret_cast<int*>(soft_part + nblocks);
        hipLaunchKernelGGL(bles_partial_kernel, dim3(nblocks), dim3(kMetricThreads), 0, st, as_arg(probs), as_arg(S), B, T, K, E,
                           tokens_per_block, vec, as_arg(soft_part), as_arg(hard_part));
    }
    hipLaunchKernelGGL(bles_finalize_kernel, dim3(1), dim3(kMetricThreads), 0, st, as_arg(soft_part), as_arg(hard_part), nblocks, B, T, K,
                       as_arg(out));
    return launch_status();
}

int moe_offload_counters(const int32_t* trace, int32_t L, int32_t T, int32_t K, int32_t E,
                         int64_t* changes, int64_t* loads, void* stream) {
    int rc = check_trace_shape(L, T, K, E);
    if (rc != MOE_OK) return rc;
    if (!trace || !changes || !loads) return MOE_ERR_INVALID;
    hipLaunchKernelGGL(offload_kernel, dim3(L), dim3(kLayerThreads), 0, as_stream(stream), as_arg(trace), T,
                       K, E, as_arg(changes), as_arg(loads));
    return launch_status();
}

int moe_delta_uniform(const int32_t* trace, int32_t L, int32_t T, int32_t K, int32_t E,
                      int64_t* counts, double* delta, double* mean, void* stream) {
    int rc = check_trace_shape(L, T, K, E);
    if (rc != MOE_OK) return rc;
    if (!trace || !counts || !mean) return MOE_ERR_INVALID;
    if ((long long)L * E >= (1ll << 31)) return MOE_ERR_UNSUPPORTED;
    hipStream_t st = as_stream(stream);
    unsigned long long* cnt = reinterpret_cast<unsigned long long*>(counts);
    const int TK = T * K;  // < 2^31 by check_trace_shape
    if (L <= kOneLayers && short_trace(L, T, L > kOneWaves) && TK <= kOneLayerPairs && (long long)L * TK <= kOnePairs) {
        hipLaunchKernelGGL(balance_one_kernel, dim3(1), dim3(kOneThreads), 0, st, as_arg(trace), L, TK, E, as_arg(cnt), as_arg(delta), as_arg(mean));
        return launch_status();
    }
    if (TK <= kOneChunkPairs) {
        hipLaunchKernelGGL(balance_count_kernel<true>, dim3(1, L), dim3(kLayerThreads), 0, st, as_arg(trace), TK, E, as_arg(cnt));
    } else {
        const int n = L * E;
        hipLaunchKernelGGL(zero_counters_kernel, dim3((n + kMetricThreads - 1) / kMetricThreads), dim3(kMetricThreads), 0,
                           st, as_arg(cnt), n, as_arg(nullptr));
        const int chunks = min(64, (TK + 4 * kLayerThreads - 1) / (4 * kLayerThreads));
        hipLaunchKernelGGL(balance_count_kernel<false>, dim3(chunks, L), dim3(kLayerThreads), 0, st, as_arg(trace), TK, E, as_arg(cnt));
    }
    hipLaunchKernelGGL(balance_finalize_kernel, dim3(1), dim3(kMetricThreads), 0, st, as_arg(cnt), L, TK, E, as_arg(delta), as_arg(mean));
    return launch_status();
}

}  // extern "C"
