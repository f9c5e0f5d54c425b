// Token selection of the speculative step: Eq. 1 draws, Eq. 2 acceptance test, Eq. 3 resample, rollback.
#pragma once
#include "sdfp_common.hip.h"

namespace sdfp {

// ---- token selection (Eq. 1 draws, Eq. 2 test, Eq. 3 resample) -----------------------------------------
struct Uni { float u[2 * MAX_K + 2]; };

// The soft-max statistics and inverse-CDF draws of a vocabulary row are float64 work (a boundary decision has to match
// the oracle's): at 32000 to 128256 entries a single workgroup spent 45 to 112 us per draw and 120 to 370 us per accept
// on it, with 255 compute units idle.  So a row is cut into at most SEL_CHUNKS chunks of `len` entries, a workgroup
// each; the last one to arrive adds the chunks' sums in ascending order, finds the chunk in which the cumulative sum
// crosses the target and scans that chunk alone.  (One kernel and a last-arriver counter instead of two kernels: the
// counter costs less than the gap between two dependent launches.)  Measured at 32000 entries: a draw 73-89 -> 11 us, an
// accept with K = 6 270 -> 22 us (statistics 5, the rest 17): what is left is latency, three dependent round
// trips through memory and a few float64 exponentials.
constexpr int SEL_THREADS = 256;
constexpr int SEL_CHUNKS = SEL_THREADS;      // the last workgroup holds one chunk per thread
constexpr int SEL_ROWS = 2 * MAX_K + 1;      // rows whose statistics an accept needs: p_0 .. p_K, q_0 .. q_{K-1}
struct SelBuf {                              // workspace of the selection kernels
    float* mx;          // [SEL_ROWS][SEL_CHUNKS] chunk maxima
    double* sum;        // [SEL_ROWS][SEL_CHUNKS] chunk sums of exp((z - chunk maximum) / T)
    double* wres;       // [SEL_CHUNKS] chunk sums of the residual max(0, p - q)
    double* wp;         // [SEL_CHUNKS] chunk sums of p
    unsigned* counter;  // arrivals, left at 0
};
__host__ __device__ constexpr size_t sel_buf_bytes() {
    return (size_t)SEL_ROWS * SEL_CHUNKS * (sizeof(float) + sizeof(double)) + 2 * SEL_CHUNKS * sizeof(double);
}
// entries per chunk: 512 -- two per thread, enough workgroups for 32000 entries (63) to take one round of memory latency
// and a few float64 exponentials -- or as many as it takes to stay within SEL_CHUNKS chunks
__host__ __device__ constexpr int sel_chunk_len(int V) {
    const int need = (V + SEL_CHUNKS - 1) / SEL_CHUNKS;
    return need <= 512 ? 512 : (need + SEL_THREADS - 1) / SEL_THREADS * SEL_THREADS;
}

__device__ __forceinline__ void st_coh(double* p, double v) {
    __hip_atomic_store(as_global(reinterpret_cast<unsigned long long*>(p)), (unsigned long long)__double_as_longlong(v),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double ld_coh(const double* p) {
    return __longlong_as_double((long long)__hip_atomic_load(as_global(reinterpret_cast<const unsigned long long*>(p)),
                                                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

// helpers for a workgroup of SEL_THREADS; sh: SEL_THREADS / 64 doubles of LDS; every thread gets the result
__device__ __forceinline__ double wave_sum_d(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
}
__device__ __forceinline__ double block_sum_d(double v, double* sh) {
    v = wave_sum_d(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < SEL_THREADS / 64; ++w) s += sh[w];
    return s;
}
__device__ __forceinline__ float block_max_f(float v, double* sh) {
    v = wave_max(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = (double)v;
    __syncthreads();
    float s = -INFINITY;
#pragma unroll
    for (int w = 0; w < SEL_THREADS / 64; ++w) s = fmaxf(s, (float)sh[w]);
    return s;
}
// sums of the threads before this one (threads in ascending order); *total: of all
__device__ __forceinline__ double block_exclusive_sum(double v, double* sh, double* total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double inc = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const double t = __shfl_up(inc, off);
        if (lane >= off) inc += t;
    }
    double before = __shfl_up(inc, 1);
    if (lane == 0) before = 0.0;
    __syncthreads();
    if (lane == 63) sh[wave] = inc;
    __syncthreads();
    double base = 0.0, tot = 0.0;
#pragma unroll
    for (int w = 0; w < SEL_THREADS / 64; ++w) { if (w < wave) base += sh[w]; tot += sh[w]; }
    *total = tot;
    return base + before;
}
// The first thread whose range (before, before + v] holds `target`, i.e. before + v > target; SEL_THREADS if none.
__device__ __forceinline__ int block_first_crossing(bool crosses, int* sh_first) {
    __syncthreads();
    if (threadIdx.x == 0) *sh_first = SEL_THREADS;
    __syncthreads();
    if (crosses) atomicMin(sh_first, (int)threadIdx.x);
    __syncthreads();
    return *sh_first;
}

// Inverse CDF by one workgroup: thread c holds the weight `cw` of chunk c (0 past the last one), w(j) is the weight of
// entry j.  Returns the smallest j with w_0 + ... + w_j > u * sum(w) (entries added in index order, chunk by chunk; the
// last entry if round-off leaves no crossing) in all threads; *total_out: sum(w).
template <class W>
__device__ __forceinline__ int chunked_inv_cdf(double cw, int V, int len, double u, const W& w, double* sh, double* total_out) {
    __shared__ int s_first, s_tok;
    __shared__ double s_run;
    double total;
    double before = block_exclusive_sum(cw, sh, &total);
    *total_out = total;
    const double target = u * total;
    const int chunk = block_first_crossing(before + cw > target, &s_first);
    if (chunk == SEL_THREADS) return V - 1;                     // uniform
    if ((int)threadIdx.x == chunk) s_run = before;
    // inside the chunk: thread t takes len / SEL_THREADS consecutive entries
    const int per = len / SEL_THREADS, hi = min(V, (chunk + 1) * len);
    const int j0 = min(hi, chunk * len + (int)threadIdx.x * per), j1 = min(hi, j0 + per);
    double s = 0.0;
    for (int j = j0; j < j1; ++j) s += w(j);
    double chunk_total;
    before = block_exclusive_sum(s, sh, &chunk_total) + s_run;  // (the barriers in there order s_run's write)
    const int owner = block_first_crossing(j0 < j1 && before + s > target, &s_first);
    if (threadIdx.x == 0) s_tok = hi - 1;
    __syncthreads();
    if ((int)threadIdx.x == owner) {
        int tok = j1 - 1;
        for (int j = j0; j < j1; ++j) {
            before += w(j);
            if (before > target) { tok = j; break; }
        }
        s_tok = tok;
    }
    __syncthreads();
    return s_tok;
}

// maximum and sum of exp((z - maximum) / T) of chunk c of a row.  A chunk whose entries are all -inf (masked or overflowed
// logits) has the sum 0: exp(-inf - -inf) would be NaN and take the whole row with it.  (Its maximum stays -inf, which
// gives it the weight exp(-inf) = 0 where the chunks are combined; a row that is -inf throughout stays NaN there.)
__device__ __forceinline__ void chunk_stats(const float* __restrict__ z, int V, int len, int c, double invT, double* sh, float* mx_out,
                                            double* sum_out) {
    const int lo = c * len, hi = min(V, lo + len);
    float mx = -INFINITY;
    for (int j = lo + threadIdx.x; j < hi; j += SEL_THREADS) mx = fmaxf(mx, z[j]);
    mx = block_max_f(mx, sh);
    const double ref = mx > -INFINITY ? (double)mx : 0.0;
    double s = 0.0;
    for (int j = lo + threadIdx.x; j < hi; j += SEL_THREADS) s += exp(((double)z[j] - ref) * invT);
    *sum_out = block_sum_d(s, sh);
    *mx_out = mx;
}
// true in every thread of the last workgroup to arrive (the others are done); leaves the counter at 0
__device__ __forceinline__ bool sel_last_arrival(unsigned* counter, int n) {
    __shared__ unsigned s_last;
    stores_done();
    __syncthreads();
    if (threadIdx.x == 0) {
        s_last = atomic_inc_g(counter) == (unsigned)(n - 1) ? 1u : 0u;
        if (s_last) st_coh(counter, 0u);
    }
    __syncthreads();
    return s_last != 0u;
}

// draw one token from soft-max(z / T) by inverse CDF: draft draws (Eq. 1) and the prefill's first token.  Grid: the chunks.
__global__ __launch_bounds__(SEL_THREADS) void k_pick_sample(const float* __restrict__ z, int V, int len, float temperature, float u,
                                                             SelBuf b, DevState* st, int dst, int off) {
    __shared__ double sh[SEL_THREADS / 64];
    const double invT = 1.0 / (double)temperature;
    const int n = gridDim.x, tid = threadIdx.x;
    float mx; double sum;
    chunk_stats(z, V, len, blockIdx.x, invT, sh, &mx, &sum);
    if (tid == 0) { st_coh(b.mx + blockIdx.x, mx); st_coh(b.sum + blockIdx.x, sum); }
    if (!sel_last_arrival(b.counter, n)) return;
    const float cm = tid < n ? ld_coh(b.mx + tid) : -INFINITY;
    const float gm = block_max_f(cm, sh);
    const double cw = tid < n ? ld_coh(b.sum + tid) * exp(((double)cm - (double)gm) * invT) : 0.0;
    double tot;
    const int tok = chunked_inv_cdf(cw, V, len, (double)u, [&](int j) { return exp(((double)z[j] - (double)gm) * invT); }, sh, &tot);
    if (tid == 0) {
        if (dst == ROWS_DRAFT) st->d[off] = tok;
        else st->amax[off] = tok;
    }
}

__device__ __forceinline__ void commit_tokens(DevState* st, int* out_tokens, int n, int x, int K) {
    for (int i = 0; i <= n; ++i) {
        const int t = (i < n) ? st->d[i] : x;
        if (st->n_out < st->max_out) out_tokens[st->n_out++] = t;
        else st->overflow = 1;
    }
    st->n_acc = n; st->x = x;
    st->steps += 1; st->drafted += K; st->accepted += n; st->examined += n + (n < K ? 1 : 0);
}

// greedy accept: n = first i with d[i] != arg-max of target row i (else K); x = arg-max of row n
__global__ void k_accept_greedy(DevState* st, int* out_tokens) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    const int K = st->K;
    int n = K;
    for (int i = 0; i < K; ++i)
        if (st->d[i] != st->amax[i]) { n = i; break; }
    commit_tokens(st, out_tokens, n, st->amax[n], K);
}

// chunk statistics of the rows an accept needs: grid (chunks, 2 K + 1), row r <= K of zp, row r - K - 1 of zq behind them
__global__ __launch_bounds__(SEL_THREADS) void k_sel_stats(const float* __restrict__ zq, const float* __restrict__ zp, int V, int len,
                                                           float temperature, int K, SelBuf b) {
    __shared__ double sh[SEL_THREADS / 64];
    const int r = blockIdx.y;
    const float* z = r <= K ? zp + (size_t)r * V : zq + (size_t)(r - K - 1) * V;
    float mx; double sum;
    chunk_stats(z, V, len, blockIdx.x, 1.0 / (double)temperature, sh, &mx, &sum);
    if (threadIdx.x == 0) { b.mx[r * SEL_CHUNKS + blockIdx.x] = mx; b.sum[r * SEL_CHUNKS + blockIdx.x] = sum; }
}

// sampling accept: Eq. 2 test per draft token, then Eq. 3 resample or the bonus draw from p_K.  Grid: the chunks; every
// workgroup reduces the statistics of all rows and finds n by itself, then sums its chunk of the row that is drawn from.
__global__ __launch_bounds__(SEL_THREADS) void k_accept_sample(const float* __restrict__ zq, const float* __restrict__ zp, int V,
                                                               int len, float temperature, int K, Uni un, SelBuf b, DevState* st,
                                                               int* out_tokens) {
    __shared__ double sh[SEL_THREADS / 64];
    __shared__ float s_mx[SEL_ROWS];
    __shared__ double s_sum[SEL_ROWS];
    __shared__ int s_n;
    const int n_chunks = gridDim.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const double invT = 1.0 / (double)temperature;
    for (int r = wave; r < 2 * K + 1; r += SEL_THREADS / 64) {   // a wave per row
        float m[SEL_CHUNKS / 64], mx = -INFINITY;
#pragma unroll
        for (int i = 0; i < SEL_CHUNKS / 64; ++i) {
            m[i] = i * 64 + lane < n_chunks ? b.mx[r * SEL_CHUNKS + i * 64 + lane] : -INFINITY;
            mx = fmaxf(mx, m[i]);
        }
        mx = wave_max(mx);
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < SEL_CHUNKS / 64; ++i)
            if (i * 64 + lane < n_chunks) s += b.sum[r * SEL_CHUNKS + i * 64 + lane] * exp(((double)m[i] - (double)mx) * invT);
        s = wave_sum_d(s);
        if (lane == 0) { s_mx[r] = mx; s_sum[r] = s; }
    }
    if (tid == 0) s_n = K;
    __syncthreads();
    if (tid < K) {   // accept d_i iff u_i q_i(d_i) < p_i(d_i); n = the first that fails
        const int t = st->d[tid];
        const double p = exp(((double)zp[(size_t)tid * V + t] - (double)s_mx[tid]) * invT) / s_sum[tid];
        const double q = exp(((double)zq[(size_t)tid * V + t] - (double)s_mx[K + 1 + tid]) * invT) / s_sum[K + 1 + tid];
        if (!((double)un.u[tid] * q < p)) atomicMin(&s_n, tid);
    }
    __syncthreads();
    const int n = s_n;
    const bool residual = n < K;
    const float *rp = zp + (size_t)n * V, *rq = zq + (size_t)(residual ? n : 0) * V;
    const double mp = (double)s_mx[n], Sp = s_sum[n], mq = residual ? (double)s_mx[K + 1 + n] : 0.0, Sq = residual ? s_sum[K + 1 + n] : 1.0;
    auto w_p = [&](int j) { return exp(((double)rp[j] - mp) * invT) / Sp; };
    auto w_res = [&](int j) { return fmax(0.0, w_p(j) - exp(((double)rq[j] - mq) * invT) / Sq); };
    {
        const int lo = blockIdx.x * len, hi = min(V, lo + len);
        double a = 0.0, r = 0.0;
        for (int j = lo + tid; j < hi; j += SEL_THREADS) { a += w_p(j); if (residual) r += w_res(j); }
        a = block_sum_d(a, sh);
        r = block_sum_d(r, sh);
        if (tid == 0) { st_coh(b.wp + blockIdx.x, a); st_coh(b.wres + blockIdx.x, r); }
    }
    if (!sel_last_arrival(b.counter, n_chunks)) return;
    int x;
    double tot = 0.0;
    if (residual) x = chunked_inv_cdf(tid < n_chunks ? ld_coh(b.wres + tid) : 0.0, V, len, (double)un.u[K], w_res, sh, &tot);
    if (!residual || !(tot > 0.0))   // no rejection, or p == q to the last bit: a draw from p
        x = chunked_inv_cdf(tid < n_chunks ? ld_coh(b.wp + tid) : 0.0, V, len, (double)un.u[K], w_p, sh, &tot);
    if (tid == 0) commit_tokens(st, out_tokens, n, x, K);
}

// in-place KV rollback: keep the pending token's and the n accepted drafts' entries
__global__ void k_rollback(DevState* st) {
    if (threadIdx.x == 0 && blockIdx.x == 0) { st->P += st->n_acc + 1; st->t_last = st->x; }
}

// after the prompt forward: commit the first generated token
__global__ void k_commit_first(DevState* st, int* out_tokens, int n_prompt) {
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        st->P = n_prompt; st->t_last = st->amax[0]; st->n_out = 1; out_tokens[0] = st->amax[0];
        st->n_acc = 0; st->x = st->amax[0]; st->K = 0; st->overflow = 0;
        st->steps = 0; st->drafted = 0; st->accepted = 0; st->examined = 0;
    }
}
__global__ void k_set_k(DevState* st, int K) {
    if (threadIdx.x == 0 && blockIdx.x == 0) st->K = K;
}
__global__ void k_set_pending(DevState* st, int P, int tok) {
    if (threadIdx.x == 0 && blockIdx.x == 0) { st->P = P; st->t_last = tok; }
}
struct DraftBlock { int d[MAX_K]; };
__global__ void k_set_draft(DevState* st, DraftBlock b, int K) {
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        for (int i = 0; i < K; ++i) st->d[i] = b.d[i];
        st->K = K;
    }
}
__global__ void k_zero_u32(unsigned* p, int n) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = 0u;
}

}  // namespace sdfp
