// Accept/reject kernels of the verify step and the draft's token pick.
//
// Greedy rule (Section 2.2; Appendix A.1 "Generated Tokens"): keep the longest prefix of candidates
// that equal the target's own argmax, then emit the target's argmax at the first mismatch (or after
// all k).  Stochastic rule (the speculative-sampling works cited in Section 2.2): keep candidate i
// while u * q_i(c_i) < p_{i-1}(c_i); then draw from max(0, p_n - q_{n+1}) renormalised, or from p_k
// when all were kept.  All reductions over the vocabulary are wavefront shuffles + one LDS hop;
// running sums for the inverse-CDF draw are taken in ascending token id (register path: 4096 ids per sweep; general path:
// runs of 64 granules of four ids; short rows: 1024 ids per sweep).
#include "common.h"

namespace sv {

// ---- Philox4x32-10 (Salmon et al., SC'11): counter-based, so a draw depends only on
// (seed, round, sequence, position) and not on batch split or thread mapping ------------------
__device__ inline void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                     uint32_t k1, uint32_t out[4]) {
    const uint32_t M0 = 0xD2511F53u, M1 = 0xCD9E8D57u;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        uint32_t h0 = __umulhi(M0, c0), l0 = M0 * c0;
        uint32_t h1 = __umulhi(M1, c2), l1 = M1 * c2;
        uint32_t n0 = h1 ^ c1 ^ k0, n2 = h0 ^ c3 ^ k1;
        c0 = n0; c1 = l1; c2 = n2; c3 = l0;
        k0 += 0x9E3779B9u; k1 += 0xBB67AE85u;
    }
    out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}
__device__ inline float word_to_uniform(uint32_t w) { return (float)(w >> 8) * 5.9604644775390625e-8f; }
// word 0: draft draw, word 1: acceptance test, word 2: residual / bonus draw of position i
__device__ inline float philox_uniform(uint64_t seed, uint32_t round, uint32_t seq, uint32_t i, int word) {
    uint32_t o[4];
    philox4x32_10(round, seq, i, 0u, (uint32_t)seed, (uint32_t)(seed >> 32), o);
    return word_to_uniform(o[word]);
}

__global__ void philox_uniforms_kernel(uint64_t seed, uint32_t round, uint32_t seq_base, int B, int k,
                                       float* __restrict__ out) {
    int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= B * (k + 1)) return;
    int b = idx / (k + 1), i = idx % (k + 1);
    uint32_t o[4];
    philox4x32_10(round, seq_base + b, (uint32_t)i, 0u, (uint32_t)seed, (uint32_t)(seed >> 32), o);
    out[3 * idx + 0] = word_to_uniform(o[0]);
    out[3 * idx + 1] = word_to_uniform(o[1]);
    out[3 * idx + 2] = word_to_uniform(o[2]);
}
hipError_t launch_philox_uniforms(uint64_t seed, uint32_t round, uint32_t seq_base, int B, int k,
                                  float* out, hipStream_t st) {
    int n = B * (k + 1);
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(philox_uniforms_kernel, dim3((n + 255) / 256), dim3(256), 0, st, seed, round,
                       seq_base, B, k, out);
    return hipGetLastError();
}

// Softmax weights use the library's expf throughout.  One exp2 instruction on the rounded product x log2 e (its rounding
// error added to first order) was 10 % faster for 256 sequences of 6 candidates over 32000 ids, 105 against 117 us, but up to
// 2.3 x 2^-24 off where expf is 1.4, and it loses weights below 2^-126.

// =================================================================================================
// General path: long rows of any vocabulary size and alignment.  One workgroup of 1024 threads per sequence; a row is read in
// aligned 16-byte granules (elements outside the row count as -inf), several granules per thread in flight.
// The maximum and the normaliser of the two rows of a candidate come from one pass (running maximum per thread), the
// draw takes one pass for the sums of runs of 64 U granules and reads again only the run that holds the
// crossing.  What bounds it is the exponentials of one compute unit per row pair: 24 sequences of 5 candidates,
// 65537 ids, 1255 us as 256 threads with 4-byte loads and a pass per reduction, 93 as a launch of tests and one of draws, 71 with
// the draw in the workgroup that rejects (accept_ahead_generic_kernel).  The normaliser's error is 1.0 x 2^-24 on average (256 threads: 3.7).
// =================================================================================================
constexpr int WIDE_THREADS = 1024, WIDE_WAVES = WIDE_THREADS / 64, WIDE_RUNS = 1024;

struct WideShared {
    float red[2][WIDE_WAVES];
    int redi[WIDE_WAVES];
    float run[WIDE_RUNS];             // total of every run, then the sum in front of it
    float wave_tot[WIDE_WAVES];
    int pick, last, stop;
};

// a row of V floats at any alignment, as granules of four: granule g holds ids 4 g - off .. 4 g - off + 3
struct WideRow {
    const float* row;
    int V, off, n;
    __device__ WideRow(const float* r, int V_) : row(r), V(V_), off((int)(((uintptr_t)r >> 2) & 3)), n((V_ + off + 3) >> 2) {}
    __device__ float4 load(int g) const {
        const int id = 4 * g - off;
        if (g < n && id >= 0 && id + 3 < V) return *(const float4*)(row + id);
        float v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = g < n && id + j >= 0 && id + j < V ? row[id + j] : -INFINITY;
        return make_float4(v[0], v[1], v[2], v[3]);
    }
};

// running maximum and sum of exp((z - m) inv_tau) over what a thread has seen
struct MaxSum {
    float m = -INFINITY, s = 0.f;
    __device__ void take(const float4 (&v)[4], float inv_tau) {
        float mx = m;
#pragma unroll
        for (int q = 0; q < 4; ++q) mx = fmaxf(fmaxf(fmaxf(mx, v[q].x), fmaxf(v[q].y, v[q].z)), v[q].w);
        if (mx > m) { s *= expf((m - mx) * inv_tau); m = mx; }
        // (nothing but -inf and not-a-numbers so far: the former add nothing, one of the latter makes the sum one)
        const float at = m == -INFINITY ? 0.f : m;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            s += (expf((v[q].x - at) * inv_tau) + expf((v[q].y - at) * inv_tau)) +
                 (expf((v[q].z - at) * inv_tau) + expf((v[q].w - at) * inv_tau));
    }
};

// maximum and normaliser of one or two rows (b: may be the same row as a, then computed for nothing else)
template <bool TWO>
__device__ inline void wide_row_stats(const WideRow& a, const WideRow& b, float inv_tau, WideShared& sh, float* am, float* as,
                                      float* bm, float* bs) {
    constexpr int STEP = 4 * WIDE_THREADS;
    const int n = TWO ? max(a.n, b.n) : a.n;
    MaxSum x, y;
    float4 va[2][4], vb[2][4];
    auto request = [&](int buf, int g0) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            va[buf][q] = a.load(g0 + q * WIDE_THREADS + (int)threadIdx.x);
            if (TWO) vb[buf][q] = b.load(g0 + q * WIDE_THREADS + (int)threadIdx.x);
        }
    };
    request(0, 0);
    for (int g0 = 0; g0 < n; g0 += 2 * STEP) {              // the next four granules are requested ahead
        if (g0 + STEP < n) request(1, g0 + STEP);
        x.take(va[0], inv_tau);
        if (TWO) y.take(vb[0], inv_tau);
        if (g0 + STEP < n) {
            if (g0 + 2 * STEP < n) request(0, g0 + 2 * STEP);
            x.take(va[1], inv_tau);
            if (TWO) y.take(vb[1], inv_tau);
        }
    }
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    auto reduce = [&](const MaxSum& t, int slot, float* mo, float* so) {
        float m = wave_max(t.m);
        __syncthreads();
        if (lane == 0) sh.red[slot][wv] = m;
        __syncthreads();
        m = sh.red[slot][0];
#pragma unroll
        for (int w = 1; w < WIDE_WAVES; ++w) m = fmaxf(m, sh.red[slot][w]);
        float v = wave_sum(t.m == -INFINITY ? t.s : t.s * expf((t.m - m) * inv_tau));
        __syncthreads();
        if (lane == 0) sh.red[slot][wv] = v;
        __syncthreads();
        v = 0.f;
#pragma unroll
        for (int w = 0; w < WIDE_WAVES; ++w) v += sh.red[slot][w];
        *mo = m; *so = v;
    };
    reduce(x, 0, am, as);
    if (TWO) reduce(y, 1, bm, bs);
}

// argmax, lowest id on ties
__device__ inline int wide_argmax(const WideRow& a, WideShared& sh) {
    float bv = -INFINITY;
    int bi = 0x7fffffff;
    for (int g0 = 0; g0 < a.n; g0 += 4 * WIDE_THREADS) {
        float4 v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = a.load(g0 + q * WIDE_THREADS + (int)threadIdx.x);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int id = 4 * (g0 + q * WIDE_THREADS + (int)threadIdx.x) - a.off;
            const float x[4] = {v[q].x, v[q].y, v[q].z, v[q].w};
#pragma unroll
            for (int j = 0; j < 4; ++j) if (x[j] > bv) { bv = x[j]; bi = id + j; }
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        float ov = __shfl_xor(bv, o, 64);
        int oi = __shfl_xor(bi, o, 64);
        if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
    }
    __syncthreads();
    if ((threadIdx.x & 63) == 0) { sh.red[0][threadIdx.x >> 6] = bv; sh.redi[threadIdx.x >> 6] = bi; }
    __syncthreads();
    bv = sh.red[0][0]; bi = sh.redi[0];
#pragma unroll
    for (int w = 1; w < WIDE_WAVES; ++w)
        if (sh.red[0][w] > bv || (sh.red[0][w] == bv && sh.redi[w] < bi)) { bv = sh.red[0][w]; bi = sh.redi[w]; }
    return bi;
}

// Inverse CDF over non-negative weights: weight(g) gives the weights of granule g (ids 4 g - off + 0..3; 0 outside
// the row).  The smallest id whose running sum (ascending ids) exceeds u * total; if rounding leaves none, the
// largest id of positive weight.  *total_out: the total (0: no positive weight; result invalid).
template <typename F>
__device__ inline int wide_inverse_cdf(F weight, int n, int off, float u, WideShared& sh, float* total_out) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int U = (n + 64 * WIDE_RUNS - 1) / (64 * WIDE_RUNS), runs = (n + 64 * U - 1) / (64 * U);
    int last = -1;
    auto sum4 = [](const float4& w) { return (w.x + w.y) + (w.z + w.w); };
    auto see = [&](const float4& w, int g) {
        if (w.x > 0.f) last = max(last, 4 * g - off);
        if (w.y > 0.f) last = max(last, 4 * g - off + 1);
        if (w.z > 0.f) last = max(last, 4 * g - off + 2);
        if (w.w > 0.f) last = max(last, 4 * g - off + 3);
    };
    __syncthreads();
    sh.run[threadIdx.x] = 0.f;
    if (threadIdx.x == 0) { sh.pick = 0x7fffffff; sh.last = -1; }
    __syncthreads();
    for (int r0 = wv; r0 < runs; r0 += 4 * WIDE_WAVES) {             // four runs of a wavefront at a time
        float t[4] = {0.f, 0.f, 0.f, 0.f};
        for (int i = 0; i < U; ++i) {
            float4 w[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) w[q] = weight(((r0 + q * WIDE_WAVES) * U + i) * 64 + lane);
#pragma unroll
            for (int q = 0; q < 4; ++q) { t[q] += sum4(w[q]); see(w[q], ((r0 + q * WIDE_WAVES) * U + i) * 64 + lane); }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float v = wave_sum(t[q]);
            if (lane == 0 && r0 + q * WIDE_WAVES < runs) sh.run[r0 + q * WIDE_WAVES] = v;
        }
    }
    if (last >= 0) atomicMax(&sh.last, last);
    __syncthreads();
    // exclusive prefix of the runs' totals, one per thread
    const float mine = sh.run[threadIdx.x];
    float incl = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const float up = __shfl_up(incl, o, 64);
        if (lane >= o) incl += up;
    }
    if (lane == 63) sh.wave_tot[wv] = incl;
    __syncthreads();
    float before = 0.f, total = 0.f;
#pragma unroll
    for (int w = 0; w < WIDE_WAVES; ++w) { if (w < wv) before += sh.wave_tot[w]; total += sh.wave_tot[w]; }
    const float target = u * total, slack = 1e-4f * total;
    const float front = before + (incl - mine);
    // the run that holds the crossing, and its neighbours within the rounding of these sums
    const bool near = mine > 0.f && front <= target + slack && front + mine >= target - slack;
    __syncthreads();
    sh.run[threadIdx.x] = near ? front : -1.f;
    __syncthreads();
    int found = 0x7fffffff;
    for (int r = wv; r < runs; r += WIDE_WAVES) {
        float base = sh.run[r];
        if (base < 0.f) continue;                        // (wave-uniform)
        for (int i = 0; i < U; ++i) {
            const int g = (r * U + i) * 64 + lane;
            const float4 w = weight(g);
            const float local = sum4(w);
            float in = local;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const float up = __shfl_up(in, o, 64);
                if (lane >= o) in += up;
            }
            float c = base + (in - local);
            const float x[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                c += x[j];
                if (x[j] > 0.f && c > target) found = min(found, 4 * g - off + j);
            }
            base += __shfl(in, 63, 64);
        }
    }
    if (found != 0x7fffffff) atomicMin(&sh.pick, found);
    __syncthreads();
    *total_out = total;
    return sh.pick != 0x7fffffff ? sh.pick : (sh.last >= 0 ? sh.last : 0);
}
// the softmax weights of granule g of a row (0 for -inf entries, i.e. outside the row)
__device__ inline float4 wide_weights(const WideRow& r, int g, float m, float inv_tau, float inv_norm) {
    const float4 z = r.load(g);
    return make_float4(expf((z.x - m) * inv_tau) * inv_norm, expf((z.y - m) * inv_tau) * inv_norm,
                       expf((z.z - m) * inv_tau) * inv_norm, expf((z.w - m) * inv_tau) * inv_norm);
}

// the acceptance test of candidate i of sequence b (the rows' maxima and normalisers given): true = rejected
__device__ inline bool rejects(const AcceptArgs& a, int b, int i, float pm, float ps, float qm, float qs) {
    const int c = a.draft_tokens[b * a.k + i];
    if (c < 0 || c >= a.V) return true;              // an id outside the vocabulary is a rejected candidate
    const float pv = expf((a.p_logits[((int64_t)b * (a.k + 1) + i) * a.V + c] - pm) * a.inv_tau) / ps;
    const float qv = expf((a.q_logits[((int64_t)b * a.k + i) * a.V + c] - qm) * a.inv_tau) / qs;
    const float u = a.u_accept ? a.u_accept[b * a.k + i]
                               : philox_uniform(a.seed, a.round, a.seq_base + b, (uint32_t)(i + 1), 1);
    return !(u * qv < pv);
}

// greedy: early exit at the first mismatch
__global__ void __launch_bounds__(WIDE_THREADS)
accept_greedy_generic_kernel(AcceptArgs a) {
    __shared__ WideShared sh;
    const int b = blockIdx.x;
    const float* P = a.p_logits + (int64_t)b * (a.k + 1) * a.V;
    int n = 0, am;
    while (true) {
        am = wide_argmax(WideRow(P + (int64_t)n * a.V, a.V), sh);
        if (n < a.k && a.draft_tokens[b * a.k + n] == am) ++n; else break;
    }
    if (threadIdx.x == 0) {
        if (a.n_accepted) a.n_accepted[b] = n;
        if (a.next_token) a.next_token[b] = am;
    }
}

// the draw behind n kept candidates, from the residual of the two rows or (n == k) from the target's row
__device__ inline int wide_draw(const AcceptArgs& a, int b, int n, const WideRow& pr, const WideRow& qr, float pm, float ps,
                                float qm, float qs, WideShared& sh) {
    const int k = a.k, V = a.V;
    const float it = a.inv_tau, ipn = 1.0f / ps, iqn = 1.0f / qs;
    const float u = a.u_resample ? a.u_resample[b * (k + 1) + n]
                                 : philox_uniform(a.seed, a.round, a.seq_base + b, (uint32_t)n, 2);
    // (granules of the two rows differ where their alignments do: the residual takes q element by element then)
    auto wp = [&](int g) { return wide_weights(pr, g, pm, it, ipn); };
    auto wres = [&](int g) {
        float4 w = wide_weights(pr, g, pm, it, ipn), q;
        if (pr.off == qr.off) q = wide_weights(qr, g, qm, it, iqn);
        else {
            float z[4];
            const int id = 4 * g - pr.off;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool in = id + j >= 0 && id + j < V;
                z[j] = in ? expf((qr.row[in ? id + j : 0] - qm) * it) * iqn : 0.f;
            }
            q = make_float4(z[0], z[1], z[2], z[3]);
        }
        return make_float4(fmaxf(0.f, w.x - q.x), fmaxf(0.f, w.y - q.y), fmaxf(0.f, w.z - q.z), fmaxf(0.f, w.w - q.w));
    };
    float tot = 0.f;
    int nxt = 0;
    if (n < k) nxt = wide_inverse_cdf(wres, pr.n, pr.off, u, sh, &tot);
    if (n == k || !(tot > 0.f)) nxt = wide_inverse_cdf(wp, pr.n, pr.off, u, sh, &tot);    // (p == q everywhere: the target row)
    return nxt;
}

__global__ void __launch_bounds__(WIDE_THREADS)
accept_sample_generic_kernel(AcceptArgs a) {
    __shared__ WideShared sh;
    const int b = blockIdx.x, k = a.k, V = a.V;
    const float* P = a.p_logits + (int64_t)b * (k + 1) * V;
    const float* Q = a.q_logits + (int64_t)b * k * V;
    const float it = a.inv_tau;
    int n = 0;
    float pm = 0.f, ps = 1.f, qm = 0.f, qs = 1.f;
    // candidates are tested in order; each test needs the softmax normalisers of two rows
    while (true) {
        const WideRow p(P + (int64_t)n * V, V);
        if (n == k) { wide_row_stats<false>(p, p, it, sh, &pm, &ps, nullptr, nullptr); break; }
        wide_row_stats<true>(p, WideRow(Q + (int64_t)n * V, V), it, sh, &pm, &ps, &qm, &qs);
        if (threadIdx.x == 0) sh.stop = rejects(a, b, n, pm, ps, qm, qs);
        __syncthreads();
        const int stop = sh.stop;
        __syncthreads();
        if (stop) break;
        ++n;
    }
    const int nxt = wide_draw(a, b, n, WideRow(P + (int64_t)n * V, V), WideRow(Q + (int64_t)(n < k ? n : 0) * V, V), pm, ps, qm, qs, sh);
    if (threadIdx.x == 0) {
        if (a.n_accepted) a.n_accepted[b] = n;
        if (a.next_token) a.next_token[b] = nxt;
    }
}

// =================================================================================================
// Short rows of any vocabulary size and alignment: one workgroup of 256 threads per sequence, an element per thread and
// load, a pass over the row (in L1) per reduction.  Bound by the latency of its few steps, which four wavefronts
// go through faster than the sixteen of the general path: 16 sequences, 4 candidates, us per call as this and as
// the general path, first candidate rejected / all kept: 1001 ids 9 / 20 and 17 / 33, 2001 ids 14 / 30 and 18 / 36, 3001 ids
// 18 / 40 and 19 / 40, 4097 ids 24 / 51 and 21 / 44.
// =================================================================================================
constexpr int NARROW_THREADS = 256, NARROW_MAX_V = 3072;

__device__ inline float narrow_sum(float v, float* sh /*>=4*/) {
    v = wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    return sh[0] + sh[1] + sh[2] + sh[3];
}
__device__ inline float narrow_max(float v, float* sh) {
    v = wave_max(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    return fmaxf(fmaxf(sh[0], sh[1]), fmaxf(sh[2], sh[3]));
}
// argmax with lowest-index tie-break
__device__ inline int narrow_argmax(const float* __restrict__ z, int V, float* shv, int* shi) {
    float bv = -INFINITY;
    int bi = 0x7fffffff;
    for (int c = threadIdx.x; c < V; c += NARROW_THREADS) {
        float v = z[c];
        if (v > bv) { bv = v; bi = c; }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        float ov = __shfl_xor(bv, o, 64);
        int oi = __shfl_xor(bi, o, 64);
        if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
    }
    __syncthreads();
    if ((threadIdx.x & 63) == 0) { shv[threadIdx.x >> 6] = bv; shi[threadIdx.x >> 6] = bi; }
    __syncthreads();
    bv = shv[0]; bi = shi[0];
#pragma unroll
    for (int w = 1; w < 4; ++w)
        if (shv[w] > bv || (shv[w] == bv && shi[w] < bi)) { bv = shv[w]; bi = shi[w]; }
    return bi;
}

// Smallest id whose running sum of w(id) (ascending ids) exceeds target; if rounding leaves none,
// the largest id with positive weight.
template <typename F>
__device__ inline int narrow_inverse_cdf(F w, int V, float target, float* shf, int* shi) {
    float run = 0.f;
    int last_pos = -1;
    int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    for (int base = 0; base < V; base += NARROW_THREADS * 4) {
        int id0 = base + threadIdx.x * 4;
        float x[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            x[j] = id0 + j < V ? w(id0 + j) : 0.f;
            if (x[j] > 0.f) last_pos = id0 + j;
        }
        float local = (x[0] + x[1]) + (x[2] + x[3]);
        float incl = local;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            float up = __shfl_up(incl, o, 64);
            if (lane >= o) incl += up;
        }
        __syncthreads();
        if (lane == 63) shf[wv] = incl;
        __syncthreads();
        float wave_base = 0.f;
        for (int q = 0; q < wv; ++q) wave_base += shf[q];
        float seg_total = shf[0] + shf[1] + shf[2] + shf[3];
        incl += wave_base;
        bool over = run + incl > target;
        // lowest thread over the target
        unsigned long long bal = __ballot(over);
        __syncthreads();
        if (lane == 0) shi[wv] = bal ? (wv * 64 + (int)__ffsll((long long)bal) - 1) : 0x7fffffff;
        __syncthreads();
        int first = min(min(shi[0], shi[1]), min(shi[2], shi[3]));
        if (first != 0x7fffffff) {
            __syncthreads();
            if ((int)threadIdx.x == first) {
                float c = run + (incl - local);
                int pick = -1, lastp = -1;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    c += x[j];
                    if (x[j] > 0.f) lastp = id0 + j;
                    if (pick < 0 && c > target && x[j] > 0.f) pick = id0 + j;
                }
                shi[4] = pick >= 0 ? pick : (lastp >= 0 ? lastp : id0);
            }
            __syncthreads();
            return shi[4];
        }
        run += seg_total;
    }
    // no crossing found (target >= total after rounding): largest id of positive weight
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) last_pos = max(last_pos, __shfl_xor(last_pos, o, 64));
    __syncthreads();
    if (lane == 0) shi[wv] = last_pos;
    __syncthreads();
    int r = max(max(shi[0], shi[1]), max(shi[2], shi[3]));
    return r < 0 ? 0 : r;
}

// max and sum of exp((z - max) * inv_tau) of one row
__device__ inline void narrow_row_stats(const float* __restrict__ z, int V, float inv_tau, float* sh,
                                       float* out_max, float* out_sum) {
    float m = -INFINITY;
    for (int c = threadIdx.x; c < V; c += NARROW_THREADS) m = fmaxf(m, z[c]);
    m = narrow_max(m, sh);
    float s = 0.f;
    for (int c = threadIdx.x; c < V; c += NARROW_THREADS) s += expf((z[c] - m) * inv_tau);
    s = narrow_sum(s, sh);
    *out_max = m; *out_sum = s;
}

__global__ void __launch_bounds__(NARROW_THREADS)
accept_sample_narrow_kernel(AcceptArgs a) {
    __shared__ float shf[4];
    __shared__ int shi[5];
    __shared__ int sh_stop;
    int b = blockIdx.x, k = a.k, V = a.V;
    const float* P = a.p_logits + (int64_t)b * (k + 1) * V;
    const float* Q = a.q_logits + (int64_t)b * k * V;
    float it = a.inv_tau;
    int n = 0;
    float pm = 0.f, ps = 1.f, qm = 0.f, qs = 1.f;
    // candidates are tested in order; each test needs the softmax normalisers of two rows
    while (true) {
        narrow_row_stats(P + (int64_t)n * V, V, it, shf, &pm, &ps);
        if (n == k) break;
        narrow_row_stats(Q + (int64_t)n * V, V, it, shf, &qm, &qs);
        if (threadIdx.x == 0) sh_stop = rejects(a, b, n, pm, ps, qm, qs);
        __syncthreads();
        int stop = sh_stop;
        __syncthreads();
        if (stop) break;
        ++n;
    }
    const float* pr = P + (int64_t)n * V;
    const float* qr = n < k ? Q + (int64_t)n * V : nullptr;
    float ipn = 1.0f / ps, iqn = 1.0f / qs;
    auto wres = [&](int id) -> float {
        float pv = expf((pr[id] - pm) * it) * ipn;
        if (!qr) return pv;
        float qv = expf((qr[id] - qm) * it) * iqn;
        return fmaxf(0.f, pv - qv);
    };
    auto wp = [&](int id) -> float { return expf((pr[id] - pm) * it) * ipn; };
    float tot = 0.f;
    for (int c = threadIdx.x; c < V; c += NARROW_THREADS) tot += wres(c);
    tot = narrow_sum(tot, shf);
    float u = a.u_resample ? a.u_resample[b * (k + 1) + n]
                           : philox_uniform(a.seed, a.round, a.seq_base + b, (uint32_t)n, 2);
    int nxt;
    if (tot > 0.f) nxt = narrow_inverse_cdf(wres, V, u * tot, shf, shi);
    else {                                  // p == q everywhere: fall back to the target row
        float tp = 0.f;
        for (int c = threadIdx.x; c < V; c += NARROW_THREADS) tp += wp(c);
        tp = narrow_sum(tp, shf);
        nxt = narrow_inverse_cdf(wp, V, u * tp, shf, shi);
    }
    if (threadIdx.x == 0) {
        if (a.n_accepted) a.n_accepted[b] = n;
        if (a.next_token) a.next_token[b] = nxt;
    }
}

// =================================================================================================
// Fast path: vocabularies of up to 32768 ids (a multiple of 4, rows 16-byte aligned).  One workgroup
// of 1024 threads per sequence; a logits row is loaded once, 32 values per thread as 8 float4 (thread
// t of sweep s holds ids 4096 s + 4 t .. + 3, so running sums stay in ascending id order), and every
// reduction of that row (max, normaliser, residual total, inverse CDF) runs on the registers.  Candidates
// tested in turn, with early exit at the first rejected one, read each row they need exactly once: (2 n + 2) rows of V
// floats per sequence when n are kept (2 k + 1 when all are).  In turn a call is bound by the dependent chain of the sequence
// that keeps most, about 8 us a candidate at 32000 ids, not by bytes (256 sequences of 6 candidates: 117 us, 2.2 TB/s); with
// fewer sequences the candidates are tested at once (accept_ahead_kernel).
// =================================================================================================
constexpr int FAST_THREADS = 1024, FAST_WAVES = FAST_THREADS / 64, FAST_SWEEPS = 8;
constexpr int FAST_MAX_V = FAST_THREADS * 4 * FAST_SWEEPS;

struct FastShared {
    float red[FAST_WAVES];
    int redi[FAST_WAVES];
    float tot[FAST_SWEEPS * FAST_WAVES];     // wave totals of every sweep, then their exclusive prefix
    float total;
    int pick, last, stop;
};

__device__ inline void fast_load_row(const float* __restrict__ row, int V, float4 (&v)[FAST_SWEEPS]) {
#pragma unroll
    for (int s = 0; s < FAST_SWEEPS; ++s) {
        const int id = (s * FAST_THREADS + (int)threadIdx.x) * 4;
        v[s] = id < V ? *(const float4*)(row + id) : make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
    }
}
__device__ inline float fast_block_sum(float v, FastShared& sh) {
    v = wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh.red[threadIdx.x >> 6] = v;
    __syncthreads();
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < FAST_WAVES; ++w) t += sh.red[w];
    return t;
}
__device__ inline float fast_block_max(float v, FastShared& sh) {
    v = wave_max(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh.red[threadIdx.x >> 6] = v;
    __syncthreads();
    float t = sh.red[0];
#pragma unroll
    for (int w = 1; w < FAST_WAVES; ++w) t = fmaxf(t, sh.red[w]);
    return t;
}
// max and sum of exp((z - max) * inv_tau) of a row held in registers (padding is -inf: adds 0).  KEEP: the row becomes those
// exponentials, which a draw that follows needs again (not where candidates are tested in turn: most tests are not
// followed by one, and writing them back costs 2 % of a call of 256 sequences)
template <bool KEEP>
__device__ inline void fast_row_stats(float4 (&v)[FAST_SWEEPS], float inv_tau, FastShared& sh, float* out_max, float* out_sum) {
    float m = -INFINITY;
#pragma unroll
    for (int s = 0; s < FAST_SWEEPS; ++s) m = fmaxf(fmaxf(fmaxf(m, v[s].x), fmaxf(v[s].y, v[s].z)), v[s].w);
    m = fast_block_max(m, sh);
    float sum = 0.f;
#pragma unroll
    for (int s = 0; s < FAST_SWEEPS; ++s) {
        const float4 e = make_float4(expf((v[s].x - m) * inv_tau), expf((v[s].y - m) * inv_tau), expf((v[s].z - m) * inv_tau),
                                     expf((v[s].w - m) * inv_tau));
        if (KEEP) v[s] = e;
        sum += (e.x + e.y) + (e.z + e.w);
    }
    *out_max = m;
    *out_sum = fast_block_sum(sum, sh);
}
// argmax of a row held in registers, lowest id on ties
__device__ inline int fast_argmax(const float4 (&v)[FAST_SWEEPS], FastShared& sh) {
    float bv = -INFINITY;
    int bi = 0x7fffffff;
#pragma unroll
    for (int s = 0; s < FAST_SWEEPS; ++s) {
        const int id = (s * FAST_THREADS + (int)threadIdx.x) * 4;
        const float x[4] = {v[s].x, v[s].y, v[s].z, v[s].w};
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (x[j] > bv) { bv = x[j]; bi = id + j; }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        float ov = __shfl_xor(bv, o, 64);
        int oi = __shfl_xor(bi, o, 64);
        if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
    }
    __syncthreads();
    if ((threadIdx.x & 63) == 0) { sh.red[threadIdx.x >> 6] = bv; sh.redi[threadIdx.x >> 6] = bi; }
    __syncthreads();
    bv = sh.red[0]; bi = sh.redi[0];
#pragma unroll
    for (int w = 1; w < FAST_WAVES; ++w)
        if (sh.red[w] > bv || (sh.red[w] == bv && sh.redi[w] < bi)) { bv = sh.red[w]; bi = sh.redi[w]; }
    return bi;
}
// Inverse CDF over non-negative weights held in registers: the smallest id whose running sum (ascending
// ids) exceeds u * total, where total is the same running sum at the end; if rounding leaves none, the
// largest id of positive weight.  *total_out receives the total (0: no positive weight; result invalid).
__device__ inline int fast_inverse_cdf(const float4 (&wt)[FAST_SWEEPS], float u, FastShared& sh, float* total_out) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    float local[FAST_SWEEPS], excl[FAST_SWEEPS];
    __syncthreads();
#pragma unroll
    for (int s = 0; s < FAST_SWEEPS; ++s) {
        local[s] = (wt[s].x + wt[s].y) + (wt[s].z + wt[s].w);
        float incl = local[s];
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            float up = __shfl_up(incl, o, 64);
            if (lane >= o) incl += up;
        }
        excl[s] = incl - local[s];
        if (lane == 63) sh.tot[s * FAST_WAVES + wv] = incl;
    }
    if (threadIdx.x == 0) { sh.pick = 0x7fffffff; sh.last = -1; }
    __syncthreads();
    if (wv == 0) {      // exclusive prefix of the 128 (sweep, wavefront) totals, two per lane
        float v0 = sh.tot[2 * lane], v1 = sh.tot[2 * lane + 1];
        float pair = v0 + v1, incl = pair;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            float up = __shfl_up(incl, o, 64);
            if (lane >= o) incl += up;
        }
        sh.tot[2 * lane] = incl - pair;
        sh.tot[2 * lane + 1] = (incl - pair) + v0;
        if (lane == 63) sh.total = incl;
    }
    __syncthreads();
    const float total = sh.total, target = u * total;
    int found = 0x7fffffff, lastp = -1;
#pragma unroll
    for (int s = 0; s < FAST_SWEEPS; ++s) {
        const int id = (s * FAST_THREADS + (int)threadIdx.x) * 4;
        float c = sh.tot[s * FAST_WAVES + wv] + excl[s];
        const float x[4] = {wt[s].x, wt[s].y, wt[s].z, wt[s].w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            c += x[j];
            if (x[j] > 0.f) {
                lastp = id + j;
                if (c > target && found == 0x7fffffff) found = id + j;
            }
        }
    }
    if (found != 0x7fffffff) atomicMin(&sh.pick, found);
    if (lastp >= 0) atomicMax(&sh.last, lastp);
    __syncthreads();
    *total_out = total;
    return sh.pick != 0x7fffffff ? sh.pick : (sh.last >= 0 ? sh.last : 0);
}
__device__ inline float4 fast_softmax_weights(const float4& z, float m, float inv_tau, float inv_norm) {
    return make_float4(expf((z.x - m) * inv_tau) * inv_norm, expf((z.y - m) * inv_tau) * inv_norm,
                       expf((z.z - m) * inv_tau) * inv_norm, expf((z.w - m) * inv_tau) * inv_norm);
}
__device__ inline float4 fast_scaled(const float4& e, float f) { return make_float4(e.x * f, e.y * f, e.z * f, e.w * f); }

// The draw behind n kept candidates: from the residual of the rows p and q (n < k) or from p, with the rows' maxima and
// normalisers; KEPT: the rows are their exponentials already
template <bool KEPT>
__device__ inline int fast_draw(const AcceptArgs& a, int b, int n, const float4 (&p)[FAST_SWEEPS], const float4 (&q)[FAST_SWEEPS],
                                float pm, float ps, float qm, float qs, FastShared& sh) {
    const float it = a.inv_tau, ipn = 1.0f / ps, iqn = 1.0f / qs;
    auto weights = [&](const float4& v, float m, float inv) { return KEPT ? fast_scaled(v, inv) : fast_softmax_weights(v, m, it, inv); };
    float4 w[FAST_SWEEPS];
#pragma unroll
    for (int s = 0; s < FAST_SWEEPS; ++s) {
        w[s] = weights(p[s], pm, ipn);
        if (n < a.k) {
            const float4 x = weights(q[s], qm, iqn);
            w[s] = make_float4(fmaxf(0.f, w[s].x - x.x), fmaxf(0.f, w[s].y - x.y), fmaxf(0.f, w[s].z - x.z), fmaxf(0.f, w[s].w - x.w));
        }
    }
    const float u = a.u_resample ? a.u_resample[b * (a.k + 1) + n]
                                 : philox_uniform(a.seed, a.round, a.seq_base + b, (uint32_t)n, 2);
    float tot;
    int nxt = fast_inverse_cdf(w, u, sh, &tot);
    if (!(tot > 0.f)) {                     // p == q everywhere: fall back to the target row
#pragma unroll
        for (int s = 0; s < FAST_SWEEPS; ++s) w[s] = weights(p[s], pm, ipn);
        nxt = fast_inverse_cdf(w, u, sh, &tot);
    }
    return nxt;
}

__global__ void __launch_bounds__(FAST_THREADS)
accept_greedy_kernel(AcceptArgs a) {
    __shared__ FastShared sh;
    const int b = blockIdx.x;
    const float* P = a.p_logits + (int64_t)b * (a.k + 1) * a.V;
    int n = 0, am;
    while (true) {
        float4 z[FAST_SWEEPS];
        fast_load_row(P + (int64_t)n * a.V, a.V, z);
        am = fast_argmax(z, sh);
        if (n < a.k && a.draft_tokens[b * a.k + n] == am) ++n; else break;
    }
    if (threadIdx.x == 0) {
        if (a.n_accepted) a.n_accepted[b] = n;
        if (a.next_token) a.next_token[b] = am;
    }
}

// Small vocabularies: all k + 1 rows at once, a wavefront per row (a row after the other, each behind a
// workgroup reduction, costs 1.3 us a row and more: 16 sequences, 4 candidates, 1001 ids, 3.1 us where the first differs and
// 8.3 where all agree, 3.4 and 3.7 so).  Not where the rows behind the first mismatch are too many bytes to read for
// nothing and the register kernel takes the vocabulary: 256 sequences, 4096 ids, first mismatch at once, 8 candidates
// (38 MB) 7.5 us against 5.1, 16 (71 MB) 14.8 against 5.0.
constexpr int ROWS_MAX_V = 4096;
constexpr int64_t ROWS_MAX_IDS = 8 << 20;
__global__ void __launch_bounds__(FAST_THREADS)
accept_greedy_rows_kernel(AcceptArgs a) {
    __shared__ int am[17];
    const int b = blockIdx.x, lane = threadIdx.x & 63;
    const float* P = a.p_logits + (int64_t)b * (a.k + 1) * a.V;
    for (int r = threadIdx.x >> 6; r <= a.k; r += FAST_WAVES) {
        const float* row = P + (int64_t)r * a.V;
        float bv = -INFINITY;
        int bi = 0x7fffffff;
#pragma unroll 8
        for (int c = lane; c < a.V; c += 64) {
            const float v = row[c];
            if (v > bv) { bv = v; bi = c; }
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const float ov = __shfl_xor(bv, o, 64);
            const int oi = __shfl_xor(bi, o, 64);
            if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
        }
        if (lane == 0) am[r] = bi;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int n = 0;
        while (n < a.k && a.draft_tokens[b * a.k + n] == am[n]) ++n;
        if (a.n_accepted) a.n_accepted[b] = n;
        if (a.next_token) a.next_token[b] = am[n];
    }
}

__global__ void __launch_bounds__(FAST_THREADS)
accept_sample_kernel(AcceptArgs a) {
    __shared__ FastShared sh;
    const int b = blockIdx.x, k = a.k, V = a.V;
    const float* P = a.p_logits + (int64_t)b * (k + 1) * V;
    const float* Q = a.q_logits + (int64_t)b * k * V;
    const float it = a.inv_tau;
    int n = 0;
    float pm = 0.f, ps = 1.f, qm = 0.f, qs = 1.f;
    float4 pz[FAST_SWEEPS], qz[FAST_SWEEPS];
    // candidates are tested in order; each test needs the softmax normalisers of two rows, which stay
    // in registers for the draw that follows the first rejection
    while (true) {
        fast_load_row(P + (int64_t)n * V, V, pz);
        if (n < k) fast_load_row(Q + (int64_t)n * V, V, qz);
        fast_row_stats<false>(pz, it, sh, &pm, &ps);
        if (n == k) break;
        fast_row_stats<false>(qz, it, sh, &qm, &qs);
        if (threadIdx.x == 0) sh.stop = rejects(a, b, n, pm, ps, qm, qs);
        __syncthreads();
        const int stop = sh.stop;
        __syncthreads();
        if (stop) break;
        ++n;
    }
    const int nxt = fast_draw<false>(a, b, n, pz, qz, pm, ps, qm, qs, sh);
    if (threadIdx.x == 0) {
        if (a.n_accepted) a.n_accepted[b] = n;
        if (a.next_token) a.next_token[b] = nxt;
    }
}

// All candidates at once: a workgroup for each of the k + 1 rows of a sequence tests its candidate and, where it is rejected (or
// the row is the one behind the last candidate), draws the sequence's next token.  The outputs serve as the meeting
// point: next_token[b] holds the smallest (row << 27 | token) of those that would draw, announced without a token before
// the draw, n_accepted[b] counts the workgroups that are through, and the last one turns both into the results.  Nobody waits.
// A workgroup leaves as soon as it sees a rejection in front of it; those of the first candidates start first, so with more
// workgroups than the chip holds few rows are read for nothing.
//
// us per call, in turn / at once (32000 ids; candidates of which the given number is kept on average):
//   sequences, candidates        1, 4     16, 1    16, 4    64, 4    64, 8    100, 4   160, 4   256, 6
//   about half kept              42 / 24  30 / 27  66 / 29  69 / 46  127 / 70  77 / 59  80 / 88  117 / 161
//   nearly all                   65 / 21  30 / 23  66 / 29  75 / 46  131 / 70  78 / 57  83 / 93  128 / 175
//   nearly none                  27 / 27  29 / 28  36 / 30  45 / 39   50 / 42  53 / 47  59 / 75   70 / 99
// A draft of which nothing at all is kept is the one case that at once is slower, up to twice (in turn every sequence ends at its first
// candidate); device us, nothing kept / kept with probability 0.8 / all kept, in turn and at once:
//   32000 ids   64, 8  27, 43 / 110, 64 / 111, 66    100, 4  28, 41 / 68, 54 / 69, 49    100, 8   28, 47 / 113, 84 / 116, 88
//   512 ids     64, 8  24, 32 / 90, 46 / 90, 47      100, 4  24, 29 / 54, 38 / 53, 33    100, 16  24, 47 / 165, 87 / 164, 100
// 65537 ids (general path): 16 sequences of 4 140 / 68, 64 of 8 287 / 138, 100 of 4 168 / 125, 160 of 4 173 / 166.
// What bounds it is the exponentials of one compute unit: 4.2 us a row of 32000 ids (17 instructions each), and as much for a
// row's bytes where all units load.  (Two workgroups per unit in half the registers spill and are slower; so is a next row
// requested into LDS while the draft's is summed.)
constexpr int AHEAD_MAX_B = 100;
constexpr int PICK_BITS = 27;
constexpr uint32_t PICK_NO_TOKEN = (1u << PICK_BITS) - 1;
__global__ void accept_begin_kernel(AcceptArgs a) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b < a.B) { a.n_accepted[b] = 0; a.next_token[b] = -1; }
}
// (one thread) whether a candidate in front of row i of sequence b is known to be rejected
__device__ inline bool rejected_before(const AcceptArgs& a, int b, int i) {
    return (int)(__hip_atomic_load((uint32_t*)a.next_token + b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> PICK_BITS) < i;
}
__device__ inline void offer_pick(const AcceptArgs& a, int b, int i, uint32_t token) {
    __hip_atomic_fetch_min((uint32_t*)a.next_token + b, ((uint32_t)i << PICK_BITS) | token, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// (one thread) this workgroup is through; the last of the sequence writes the results
__device__ inline void report(const AcceptArgs& a, int b) {
    if (__hip_atomic_fetch_add(a.n_accepted + b, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) != a.k) return;
    const uint32_t v = __hip_atomic_load((uint32_t*)a.next_token + b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    a.n_accepted[b] = (int)(v >> PICK_BITS);
    a.next_token[b] = (int)(v & PICK_NO_TOKEN);
}
__global__ void __launch_bounds__(FAST_THREADS)
accept_ahead_kernel(AcceptArgs a) {
    __shared__ FastShared sh;
    const int b = blockIdx.x % a.B, i = blockIdx.x / a.B, k = a.k, V = a.V;
    if (threadIdx.x == 0) sh.stop = rejected_before(a, b, i);
    __syncthreads();
    bool go = !sh.stop;
    if (go) {
        float4 pz[FAST_SWEEPS], qz[FAST_SWEEPS];
        float pm, ps, qm = 0.f, qs = 1.f;
        fast_load_row(a.p_logits + ((int64_t)b * (k + 1) + i) * V, V, pz);
        if (i < k) fast_load_row(a.q_logits + ((int64_t)b * k + i) * V, V, qz);
        fast_row_stats<true>(pz, a.inv_tau, sh, &pm, &ps);
        if (i < k) fast_row_stats<true>(qz, a.inv_tau, sh, &qm, &qs);
        if (threadIdx.x == 0) {
            const bool draws = (i == k || rejects(a, b, i, pm, ps, qm, qs)) && !rejected_before(a, b, i);
            if (draws) offer_pick(a, b, i, PICK_NO_TOKEN);
            sh.stop = !draws;
        }
        __syncthreads();
        go = !sh.stop;
        if (go) {
            const int nxt = fast_draw<true>(a, b, i, pz, qz, pm, ps, qm, qs, sh);
            if (threadIdx.x == 0) offer_pick(a, b, i, (uint32_t)nxt);
        }
    }
    if (threadIdx.x == 0) report(a, b);
}
__global__ void __launch_bounds__(WIDE_THREADS)
accept_ahead_generic_kernel(AcceptArgs a) {
    __shared__ WideShared sh;
    const int b = blockIdx.x % a.B, i = blockIdx.x / a.B, k = a.k, V = a.V;
    if (threadIdx.x == 0) sh.stop = rejected_before(a, b, i);
    __syncthreads();
    bool go = !sh.stop;
    if (go) {
        const WideRow p(a.p_logits + ((int64_t)b * (k + 1) + i) * V, V), q(a.q_logits + ((int64_t)b * k + (i < k ? i : 0)) * V, V);
        float pm, ps, qm = 0.f, qs = 1.f;
        if (i < k) wide_row_stats<true>(p, q, a.inv_tau, sh, &pm, &ps, &qm, &qs);
        else wide_row_stats<false>(p, p, a.inv_tau, sh, &pm, &ps, nullptr, nullptr);
        if (threadIdx.x == 0) {
            const bool draws = (i == k || rejects(a, b, i, pm, ps, qm, qs)) && !rejected_before(a, b, i);
            if (draws) offer_pick(a, b, i, PICK_NO_TOKEN);
            sh.stop = !draws;
        }
        __syncthreads();
        go = !sh.stop;
        if (go) {
            const int nxt = wide_draw(a, b, i, p, q, pm, ps, qm, qs, sh);
            if (threadIdx.x == 0) offer_pick(a, b, i, (uint32_t)nxt);
        }
    }
    if (threadIdx.x == 0) report(a, b);
}

static inline bool fast_rows_ok(const float* base, int V) {
    return V % 4 == 0 && V <= FAST_MAX_V && ((uintptr_t)base & 15) == 0;
}

hipError_t launch_accept(const AcceptArgs& a, hipStream_t st) {
    if (a.B <= 0) return hipSuccess;
    const bool fast = fast_rows_ok(a.p_logits, a.V) && (!a.q_logits || fast_rows_ok(a.q_logits, a.V));
    if (a.q_logits) {
        // Candidates at once or in turn (accept_ahead_kernel has the figures).  At once a sequence takes one test and one draw, but
        // the rows behind its first rejection are read as well and a workgroup holds a compute unit: from about 100
        // sequences on, whose first candidates alone come near to filling the chip, in turn is faster again.  Rows off the register
        // path: one candidate is tested in turn (65537 ids, 16 sequences: 63 us, at once 65), and so are short rows, whose test
        // costs only V / 430 us, unless there are several candidates and sequences.
        const bool short_rows = a.V <= 2 * NARROW_MAX_V;
        const bool pays = fast               ? a.B <= AHEAD_MAX_B
                          : a.V <= NARROW_MAX_V ? a.k >= 3 && a.B >= 4 && a.B <= 256 / a.k && (int64_t)a.k * a.V >= 4 * NARROW_MAX_V
                                             : a.B <= AHEAD_MAX_B && a.k >= 2 && (!short_rows || (a.B >= 4 && (int64_t)a.k * a.V >= 4 * NARROW_MAX_V));
        const bool ahead = pays && a.n_accepted && a.next_token && a.V < (int)PICK_NO_TOKEN;
        if (ahead) {
            hipLaunchKernelGGL(accept_begin_kernel, dim3((a.B + 255) / 256), dim3(256), 0, st, a);
            if (fast) hipLaunchKernelGGL(accept_ahead_kernel, dim3(a.B * (a.k + 1)), dim3(FAST_THREADS), 0, st, a);
            else hipLaunchKernelGGL(accept_ahead_generic_kernel, dim3(a.B * (a.k + 1)), dim3(WIDE_THREADS), 0, st, a);
        } else if (fast) hipLaunchKernelGGL(accept_sample_kernel, dim3(a.B), dim3(FAST_THREADS), 0, st, a);
        else if (a.V <= NARROW_MAX_V) hipLaunchKernelGGL(accept_sample_narrow_kernel, dim3(a.B), dim3(NARROW_THREADS), 0, st, a);
        else hipLaunchKernelGGL(accept_sample_generic_kernel, dim3(a.B), dim3(WIDE_THREADS), 0, st, a);
    } else {
        const bool rows = a.V <= ROWS_MAX_V && (!fast || (int64_t)a.B * (a.k + 1) * a.V <= ROWS_MAX_IDS);
        if (rows) hipLaunchKernelGGL(accept_greedy_rows_kernel, dim3(a.B), dim3(FAST_THREADS), 0, st, a);
        else if (fast) hipLaunchKernelGGL(accept_greedy_kernel, dim3(a.B), dim3(FAST_THREADS), 0, st, a);
        else hipLaunchKernelGGL(accept_greedy_generic_kernel, dim3(a.B), dim3(WIDE_THREADS), 0, st, a);
    }
    return hipGetLastError();
}

// ---- draft token pick ---------------------------------------------------------------------------
__global__ void __launch_bounds__(WIDE_THREADS)
draft_pick_generic_kernel(const float* __restrict__ z, int64_t ld, int V, int mode, float inv_tau, uint64_t seed,
                          uint32_t round, uint32_t seq_base, int step, int32_t* __restrict__ draft_tokens, int k) {
    __shared__ WideShared sh;
    const int b = blockIdx.x;
    const WideRow row(z + (int64_t)b * ld, V);
    int pick;
    if (mode == SPEC_GREEDY) {
        pick = wide_argmax(row, sh);
    } else {
        float m, s, tot;
        wide_row_stats<false>(row, row, inv_tau, sh, &m, &s, nullptr, nullptr);
        auto w = [&](int g) { return wide_weights(row, g, m, inv_tau, 1.0f); };
        const float u = philox_uniform(seed, round, seq_base + b, (uint32_t)step, 0);
        pick = wide_inverse_cdf(w, row.n, row.off, u, sh, &tot);
    }
    if (threadIdx.x == 0) draft_tokens[b * k + step - 1] = pick;
}
__global__ void __launch_bounds__(NARROW_THREADS)
draft_pick_narrow_kernel(const float* __restrict__ z, int64_t ld, int V, int mode, float inv_tau, uint64_t seed,
                          uint32_t round, uint32_t seq_base, int step, int32_t* __restrict__ draft_tokens, int k) {
    __shared__ float shf[4];
    __shared__ int shi[5];
    int b = blockIdx.x;
    const float* row = z + (int64_t)b * ld;
    int pick;
    if (mode == SPEC_GREEDY) {
        pick = narrow_argmax(row, V, shf, shi);
    } else {
        float m, s;
        narrow_row_stats(row, V, inv_tau, shf, &m, &s);
        auto w = [&](int id) -> float { return expf((row[id] - m) * inv_tau); };
        float u = philox_uniform(seed, round, seq_base + b, (uint32_t)step, 0);
        pick = narrow_inverse_cdf(w, V, u * s, shf, shi);
    }
    if (threadIdx.x == 0) draft_tokens[b * k + step - 1] = pick;
}
// fast path (see above): the row is read once
__global__ void __launch_bounds__(FAST_THREADS)
draft_pick_kernel(const float* __restrict__ z, int64_t ld, int V, int mode, float inv_tau, uint64_t seed,
                  uint32_t round, uint32_t seq_base, int step, int32_t* __restrict__ draft_tokens, int k) {
    __shared__ FastShared sh;
    const int b = blockIdx.x;
    float4 row[FAST_SWEEPS];
    fast_load_row(z + (int64_t)b * ld, V, row);
    int pick;
    if (mode == SPEC_GREEDY) {
        pick = fast_argmax(row, sh);
    } else {
        float m, s, tot;
        fast_row_stats<true>(row, inv_tau, sh, &m, &s);        // (the row is its exponentials now)
        const float u = philox_uniform(seed, round, seq_base + b, (uint32_t)step, 0);
        pick = fast_inverse_cdf(row, u, sh, &tot);
    }
    if (threadIdx.x == 0) draft_tokens[b * k + step - 1] = pick;
}
hipError_t launch_draft_pick(const float* z, int64_t ld, int V, int B, int mode, float inv_tau,
                             uint64_t seed, uint32_t round, uint32_t seq_base, int step,
                             int32_t* draft_tokens, int k, hipStream_t st) {
    if (B <= 0) return hipSuccess;
    if (fast_rows_ok(z, V) && ld % 4 == 0)
        hipLaunchKernelGGL(draft_pick_kernel, dim3(B), dim3(FAST_THREADS), 0, st, z, ld, V, mode, inv_tau, seed,
                           round, seq_base, step, draft_tokens, k);
    else if (V <= NARROW_MAX_V)
        hipLaunchKernelGGL(draft_pick_narrow_kernel, dim3(B), dim3(NARROW_THREADS), 0, st, z, ld, V, mode, inv_tau, seed,
                           round, seq_base, step, draft_tokens, k);
    else
        hipLaunchKernelGGL(draft_pick_generic_kernel, dim3(B), dim3(WIDE_THREADS), 0, st, z, ld, V, mode, inv_tau,
                           seed, round, seq_base, step, draft_tokens, k);
    return hipGetLastError();
}

}  // namespace sv
