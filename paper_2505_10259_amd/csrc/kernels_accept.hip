// Accept/reject kernels of the verify step and the draft's token pick.
//
// Greedy rule (Section 2.2; Appendix A.1 "Generated Tokens"): keep the longest prefix of candidates
// that equal the target's own argmax, then emit the target's argmax at the first mismatch (or after
// all k).  Stochastic rule (the speculative-sampling works cited in Section 2.2): keep candidate i
// while u * q_i(c_i) < p_{i-1}(c_i); then draw from max(0, p_n - q_{n+1}) renormalised, or from p_k
// when all were kept.  All reductions over the vocabulary are wavefront reductions + one LDS hop;
// running sums for the inverse-CDF draw are taken in ascending token id (runs of 64 granules of four ids; draft picks from registers: 4096
// ids per sweep).
#include <type_traits>

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

// Softmax weights e^((z - m) / tau) = 2^(d c), d = z - m <= 0, c = log2(e) / tau in two parts, both positive so that -inf gives 0
// (weight_scale).  A weight is the library's expf with the division by tau inside the product: 2^n * exp2 of the rest, eleven instructions against
// sixteen, and weights below 2^-126 are there.  (Far below, n stays and the rest underflows.)  Error over every f32 argument, in units of half the
// last place, mean / largest: 0.51 / 1.8 at any temperature; expf of the rounded d / tau 0.51 / 1.8 at temperature 1 and, at
// 0.8, 2.4 / 33 down to e^-17, 24 / 129 below.
struct WeightScale { float hi, lo; };
__device__ inline float weight(float z, float m, const WeightScale& c) {
    const float d = z - m, h = fmaxf(d * c.hi, -200.f), n = __builtin_rintf(h);
    const float l = __builtin_fmaf(d, c.lo, __builtin_fmaf(d, c.hi, -h));
    return __builtin_amdgcn_ldexpf(__builtin_amdgcn_exp2f((h - n) + l), (int)n);
}
__device__ inline WeightScale weight_scale(float inv_tau) {
    const double c = (double)inv_tau * 1.44269504088896340736;
    float hi = (float)c;
    if ((double)hi > c) hi = __uint_as_float(__float_as_uint(hi) - 1u);       // (towards zero)
    return {hi, fmaxf((float)(c - (double)hi), 1e-45f)};
}

// =================================================================================================
// Rows of 4 ids and more at any alignment, a workgroup of T threads per row or pair of rows.  A row passes through in granules of four ids: maximum and
// normaliser in one pass (running maximum per thread), the draw in a pass for the sums of runs of 64 U granules, of which only the run that
// holds the crossing is read again.  1 / normaliser, mean error in 2^-24 at temperature 0.8 / 1, expf and one chain a thread (256 threads up to 3072
// ids, else 1024) -> here: random rows (standard deviation 3) 1001 ids 0.89 / 0.78 -> 0.89 / 0.81, 32000 ids 1.02 / 0.97 -> 0.90 / 0.82, 131073 ids
// 1.05 / 0.96 -> 0.86 / 0.74; one large logit and the rest equal, far below 32000 ids 2.7 / 2.1 -> 2.3 / 1.6, 131073 ids 10.5 / 7.3 -> 2.4 / 1.8.
// =================================================================================================
// Running maximum and sum of the weights over what a thread has seen.  With h the rounded d c and l what it lacks, a weight is
// 2^h (1 + l ln 2): the sum takes the 2^h and a second one their corrections, eight instructions and no rounding of the exponent.  (Those
// below 2^-126 of the maximum's weight count as nothing: the sum does not see them.)  What rounding takes from the sum at every step of N
// granules is kept beside it: equal weights would lose in the same direction every time.
struct MaxSum {
    float m = -INFINITY, s = 0.f, r = 0.f, lost = 0.f;
    __device__ float add(float z, float at, const WeightScale& c) {
        const float d = z - at, h = d * c.hi, e = __builtin_amdgcn_exp2f(h);
        // (far below what h lacks is no number, or as large, where the weight is 0; a not-a-number is one in e)
        r = __builtin_fmaf(e, __builtin_amdgcn_fmed3f(__builtin_fmaf(d, c.lo, __builtin_fmaf(d, c.hi, -h)), -1.f, 1.f), r);
        return e;
    }
    template <int N>
    __device__ void take(const float4 (&v)[N], const WeightScale& c) {
        static_assert(N == 1 || N == 4, "granules of a step");
        float mx = m;
#pragma unroll
        for (int q = 0; q < N; ++q) mx = fmaxf(fmaxf(fmaxf(mx, v[q].x), fmaxf(v[q].y, v[q].z)), v[q].w);
        if (mx > m) { const float f = weight(m, mx, c); s *= f; r *= f; lost *= f; m = mx; }
        // (nothing but -inf and not-a-numbers so far: the former add nothing, one of the latter makes the sum one)
        const float at = m == -INFINITY ? 0.f : m;
        float t[N];
#pragma unroll
        for (int q = 0; q < N; ++q) t[q] = (add(v[q].x, at, c) + add(v[q].y, at, c)) + (add(v[q].z, at, c) + add(v[q].w, at, c));
        const float step = N == 1 ? t[0] : (t[0] + t[1 % N]) + (t[2 % N] + t[3 % N]);
        const float now = s + step, b = now - s;              // (Knuth's sum of two and its error)
        lost += (s - (now - b)) + (step - b);
        s = now;
    }
    // the sum under the maximum of more threads, whose weight f this one's has
    __device__ float under(float f) const { return __builtin_fmaf(s, f, __builtin_fmaf(r, 0.693147181f, lost) * f); }
};

template <int T>
struct RowShared {
    float red[2][2][T / 64];
    float run[T];                 // total of every run, then the sum in front of it
    float wave_tot[T / 64];
    int pick, last, stop;
};
// granule g of a row: ids 4 g .. 4 g + 3, loaded from the row's last four ids where it does not lie inside; row_ids makes of those
// what the granule holds (-inf past the end)
__device__ inline float4 row_load(const float* row, int V, int g) {
    typedef float vec __attribute__((ext_vector_type(4), aligned(4)));
    const vec x = *(const vec*)((const char*)row + min(16u * (uint32_t)g, 4u * (uint32_t)V - 16u));
    return make_float4(x.x, x.y, x.z, x.w);
}
__device__ inline float4 row_ids(const float4& x, int V, int g) {
    const int n = V - 4 * g;
    const float I = -INFINITY;
    float4 y = make_float4(n >= 4 ? x.x : I, n >= 4 ? x.y : I, n >= 4 ? x.z : I, n >= 4 ? x.w : I);
    if (n > 0 && n < 4) y = n == 3 ? make_float4(x.y, x.z, x.w, I) : n == 2 ? make_float4(x.z, x.w, I, I) : make_float4(x.w, I, I, I);
    return y;
}
// maxima and normalisers of the rows p and (if TWO) q
template <int T, bool TWO>
__device__ inline void row_stats(const float* p, const float* q, int V, float inv_tau, RowShared<T>& sh, float* pm, float* ps, float* qm, float* qs) {
    constexpr int STEP = 4 * T;               // granules
    const int t = (int)threadIdx.x, first = __builtin_amdgcn_readfirstlane(t & ~63);
    const WeightScale c = weight_scale(inv_tau);
    MaxSum x, y;
    float4 a[2][4], b[2][4];
    // (of a wavefront: whether all its granules of the step at g0 lie inside the row, whether its j-th ones do in part)
    auto whole = [&](int g0) { return 4 * (g0 + 3 * T + first + 64) <= V; };
    auto part = [&](int g0, int j) { return 4 * (g0 + j * T + first) < V; };
    // (always all of a step's loads, so that the count of those in flight is known where their predecessors are waited for)
    auto request = [&](int buf, int g0) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            a[buf][j] = row_load(p, V, g0 + j * T + t);
            if (TWO) b[buf][j] = row_load(q, V, g0 + j * T + t);
        }
    };
    auto take = [&](int buf, int g0) {
        if (whole(g0)) {
            x.take(a[buf], c);
            if (TWO) y.take(b[buf], c);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (part(g0, j)) {
                    float4 v[1] = {row_ids(a[buf][j], V, g0 + j * T + t)};
                    x.take(v, c);
                    if (TWO) {
                        v[0] = row_ids(b[buf][j], V, g0 + j * T + t);
                        y.take(v, c);
                    }
                }
        }
    };
    request(0, 0);
    for (int g0 = 0; g0 < (V + 3) >> 2; g0 += 2 * STEP) {
        request(1, g0 + STEP);
        take(0, g0);
        request(0, g0 + 2 * STEP);
        take(1, g0 + STEP);
    }
    const int lane = t & 63, wv = t >> 6;
    auto wave = [&](const MaxSum& v, int r) {
        const float m = wave_max(v.m);
        const float s = wave_sum(v.under(v.m == -INFINITY ? 1.f : weight(v.m, m, c)));
        if (lane == 0) { sh.red[r][0][wv] = m; sh.red[r][1][wv] = s; }
    };
    auto block = [&](int r, float* mo, float* so) {
        float m = sh.red[r][0][0], s = 0.f;
#pragma unroll
        for (int w = 1; w < T / 64; ++w) m = fmaxf(m, sh.red[r][0][w]);
#pragma unroll
        for (int w = 0; w < T / 64; ++w) {
            const float mw = sh.red[r][0][w], sw = sh.red[r][1][w];
            s += mw == -INFINITY ? sw : sw * weight(mw, m, c);
        }
        *mo = m; *so = s;
    };
    __syncthreads();
    wave(x, 0);
    if (TWO) wave(y, 1);
    __syncthreads();
    block(0, pm, ps);
    if (TWO) block(1, qm, qs);
}
// sum over the lanes up to and with this one
__device__ inline float wave_prefix(float v) {
    auto up = [](float x, auto ctrl, auto rows) {
        return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(ctrl)::value, decltype(rows)::value, 0xf, false));
    };
    using All = std::integral_constant<int, 0xf>;
    v += up(v, std::integral_constant<int, 0x111>{}, All{});                                  // row_shr:1, 2, 4, 8
    v += up(v, std::integral_constant<int, 0x112>{}, All{});
    v += up(v, std::integral_constant<int, 0x114>{}, All{});
    v += up(v, std::integral_constant<int, 0x118>{}, All{});
    v += up(v, std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xa>{});     // row_bcast:15 to rows 1 and 3
    v += up(v, std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xc>{});     // row_bcast:31 to rows 2 and 3
    return v;
}
// Inverse CDF over the residual weights max(0, p - q) of two rows, or (RES false) over the target's own: the smallest id whose running sum
// (ascending ids) exceeds u * total; if rounding leaves none, the largest id of positive weight.  *total_out: the total (0: no
// positive weight; result invalid).  One pass for the sums of runs of 64 U granules; the run that holds the crossing is read again.  Both
// passes take the same weights to the bit, so that what the sums see as positive is found (and rows that are equal leave nothing).
template <int T, bool RES>
__device__ inline int row_draw(const float* p, const float* q, int V, float inv_tau, float pm, float pf, float qm, float qf, float u,
                               RowShared<T>& sh, float* total_out) {
    constexpr int W = T / 64;
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), n = (V + 3) >> 2;
    const int U = (n + 64 * T - 1) / (64 * T), runs = (n + 64 * U - 1) / (64 * U);
    const WeightScale c = weight_scale(inv_tau);
    auto weights = [&](const float4& zp, const float4& zq, int g) {
#pragma clang fp contract(off)
        auto f = [&](float z, float m) { return weight(z, m, c); };
        float4 a = zp, b = zq;
        if (4 * (g - lane) + 256 > V) {                       // (the same for all lanes)
            a = row_ids(zp, V, g);
            if (RES) b = row_ids(zq, V, g);
        }
        float4 w = make_float4(f(a.x, pm) * pf, f(a.y, pm) * pf, f(a.z, pm) * pf, f(a.w, pm) * pf);
        if (RES) w = make_float4(fmaxf(0.f, w.x - f(b.x, qm) * qf), fmaxf(0.f, w.y - f(b.y, qm) * qf),
                                 fmaxf(0.f, w.z - f(b.z, qm) * qf), fmaxf(0.f, w.w - f(b.w, qm) * qf));
        return w;
    };
    auto sum4 = [](const float4& w) { return (w.x + w.y) + (w.z + w.w); };
    // four runs of a wavefront at a time, the next granules requested ahead
    float4 zp[2][4], zq[2][4];
    float t[4] = {0.f, 0.f, 0.f, 0.f};
    auto request = [&](int buf, int r0, int i) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            zp[buf][j] = row_load(p, V, ((r0 + j * W) * U + i) * 64 + lane);
            if (RES) zq[buf][j] = row_load(q, V, ((r0 + j * W) * U + i) * 64 + lane);
        }
    };
    auto take = [&](int buf, int r0, int i) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (r0 + j * W >= runs) continue;                 // (the same for all lanes)
            t[j] += sum4(weights(zp[buf][j], RES ? zq[buf][j] : zp[buf][j], ((r0 + j * W) * U + i) * 64 + lane));
            if (i == U - 1) {
                const float v = wave_sum(t[j]);
                if (lane == 0) sh.run[r0 + j * W] = v;
                t[j] = 0.f;
            }
        }
    };
    int r0 = wv, i0 = 0;
    auto next = [&](int& r, int& i) { if (++i == U) { i = 0; r += 4 * W; } };
    request(0, r0, i0);
    if (threadIdx.x == 0) { sh.pick = 0x7fffffff; sh.last = -1; }
    while (r0 < runs) {
        int r1 = r0, i1 = i0;
        next(r1, i1);
        request(1, r1, i1);
        take(0, r0, i0);
        r0 = r1; i0 = i1;
        next(r0, i0);
        request(0, r0, i0);
        take(1, r1, i1);
    }
    __syncthreads();
    // the sum in front of every run, one per thread
    const float mine = (int)threadIdx.x < runs ? sh.run[threadIdx.x] : 0.f;
    const float incl = wave_prefix(mine);
    if (lane == 63) sh.wave_tot[wv] = incl;
    __syncthreads();
    float before = 0.f, total = 0.f;
#pragma unroll
    for (int w = 0; w < W; ++w) { if (w < wv) before += sh.wave_tot[w]; total += sh.wave_tot[w]; }
    const float target = u * total, slack = 1e-4f * total;
    const float front = before + (incl - mine);
    // the run that holds the crossing, and its neighbours within the rounding of these sums
    uint64_t near = __ballot(mine > 0.f && front <= target + slack && front + mine >= target - slack);
    int found = 0x7fffffff;
    for (; near; near &= near - 1) {
        const int l = __ffsll((unsigned long long)near) - 1, r = wv * 64 + l;
        float base = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(front), l));
        for (int i = 0; i < U; ++i) {
            const int g = (r * U + i) * 64 + lane;
            const float4 za = row_load(p, V, g), zb = RES ? row_load(q, V, g) : za;
            const float4 w = weights(za, zb, g);
            const float local = sum4(w), in = wave_prefix(local);
            float s = base + (in - local);
            const float x[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                s += x[j];
                if (x[j] > 0.f && s > target) found = min(found, 4 * g + j);
            }
            base += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(in), 63));
        }
    }
    if (found != 0x7fffffff) atomicMin(&sh.pick, found);
    __syncthreads();
    *total_out = total;
    if (sh.pick != 0x7fffffff) return sh.pick;
    int last = -1;
    for (int g = threadIdx.x; g < (n + 63) / 64 * 64; g += T) {
        const float4 za = row_load(p, V, g), zb = RES ? row_load(q, V, g) : za;
        const float4 w = weights(za, zb, g);
        const float x[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) if (x[j] > 0.f) last = 4 * g + j;
    }
    if (last >= 0) atomicMax(&sh.last, last);
    __syncthreads();
    if (sh.last < 0) *total_out = 0.f;
    return max(sh.last, 0);
}
// What the acceptance test of candidate i of sequence b needs of its rows, asked for ahead of their statistics, and the test: true = rejected
struct Candidate {
    float p = 0.f, q = 0.f, u = 0.f;
    bool valid = false;
};
__device__ inline Candidate candidate(const AcceptArgs& a, int b, int i) {
    Candidate t;
    const int c = a.draft_tokens[b * a.k + i];
    t.valid = c >= 0 && c < a.V;                      // an id outside the vocabulary is a rejected candidate
    if (t.valid) {
        t.p = a.p_logits[((int64_t)b * (a.k + 1) + i) * a.V + c];
        t.q = a.q_logits[((int64_t)b * a.k + i) * a.V + c];
    }
    t.u = a.u_accept ? a.u_accept[b * a.k + i] : philox_uniform(a.seed, a.round, a.seq_base + b, (uint32_t)(i + 1), 1);
    return t;
}
__device__ inline bool rejects(const Candidate& t, float inv_tau, float pm, float ps, float qm, float qs) {
    const float pv = expf((t.p - pm) * inv_tau) / ps, qv = expf((t.q - qm) * inv_tau) / qs;
    return !t.valid || !(t.u * qv < pv);
}

// =================================================================================================
// Vocabularies of fewer than four ids: a thread per sequence.
// =================================================================================================
__device__ inline void tiny_stats(const float* z, int V, float inv_tau, float* m, float* s) {
    *m = -INFINITY; *s = 0.f;
    for (int c = 0; c < V; ++c) *m = fmaxf(*m, z[c]);
    for (int c = 0; c < V; ++c) *s += expf((z[c] - *m) * inv_tau);
}
template <typename F>
__device__ inline int tiny_inverse_cdf(F w, int V, float u, float* total_out) {
    float total = 0.f, run = 0.f;
    int last = 0;
    for (int c = 0; c < V; ++c) total += w(c);
    *total_out = total;
    for (int c = 0; c < V; ++c) {
        const float x = w(c);
        run += x;
        if (x > 0.f && run > u * total) return c;
        if (x > 0.f) last = c;
    }
    return last;
}
__global__ void accept_sample_tiny_kernel(AcceptArgs a) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x, k = a.k, V = a.V;
    if (b >= a.B) return;
    const float* P = a.p_logits + (int64_t)b * (k + 1) * V;
    const float* Q = a.q_logits + (int64_t)b * k * V;
    const float it = a.inv_tau;
    float pm, ps, qm = 0.f, qs = 1.f, tot = 0.f;
    int n = 0, nxt = 0;
    for (;; ++n) {
        tiny_stats(P + n * V, V, it, &pm, &ps);
        if (n == k) break;
        tiny_stats(Q + n * V, V, it, &qm, &qs);
        if (rejects(candidate(a, b, n), it, pm, ps, qm, qs)) break;
    }
    const float u = a.u_resample ? a.u_resample[b * (k + 1) + n] : philox_uniform(a.seed, a.round, a.seq_base + b, (uint32_t)n, 2);
    auto wp = [&](int c) { return expf((P[n * V + c] - pm) * it) / ps; };
    if (n < k) nxt = tiny_inverse_cdf([&](int c) { return fmaxf(0.f, wp(c) - expf((Q[n * V + c] - qm) * it) / qs); }, V, u, &tot);
    if (n == k || !(tot > 0.f)) nxt = tiny_inverse_cdf(wp, V, u, &tot);       // (p == q everywhere: the target row)
    if (a.n_accepted) a.n_accepted[b] = n;
    if (a.next_token) a.next_token[b] = nxt;
}

// =================================================================================================
// Greedy rule, a workgroup per sequence, for rows of any size and alignment (the kernels for some of them follow).
// =================================================================================================
// The argmax kernels give NO_ID for a row that holds nothing above -inf (all -inf or not-a-number).  Such a row keeps no candidate and its
// token is 0, as in the sampling rule: no id outside the vocabulary is emitted, and none meets the row number of offer_pick.
constexpr int NO_ID = 0x7fffffff;
__device__ inline bool greedy_keeps(int am, int candidate) { return am != NO_ID && am == candidate; }
__device__ inline int greedy_token(int am) { return am == NO_ID ? 0 : am; }
constexpr int WIDE_THREADS = 1024, WIDE_WAVES = WIDE_THREADS / 64;
struct WideShared {
    float red[WIDE_WAVES];
    int redi[WIDE_WAVES];
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

// argmax, lowest id on ties
__device__ inline int wide_argmax(const WideRow& a, WideShared& sh) {
    float bv = -INFINITY;
    int bi = NO_ID;
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
    if ((threadIdx.x & 63) == 0) { sh.red[threadIdx.x >> 6] = bv; sh.redi[threadIdx.x >> 6] = bi; }
    __syncthreads();
    bv = sh.red[0]; bi = sh.redi[0];
#pragma unroll
    for (int w = 1; w < WIDE_WAVES; ++w)
        if (sh.red[w] > bv || (sh.red[w] == bv && sh.redi[w] < bi)) { bv = sh.red[w]; bi = sh.redi[w]; }
    return bi;
}

constexpr int NARROW_THREADS = 256, NARROW_MAX_V = 3072;       // (short rows: a quarter of the wavefronts to meet)
// argmax with lowest-index tie-break
__device__ inline int narrow_argmax(const float* __restrict__ z, int V, float* shv, int* shi) {
    float bv = -INFINITY;
    int bi = NO_ID;
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

// greedy: early exit at the first mismatch
__global__ void __launch_bounds__(WIDE_THREADS)
accept_greedy_generic_kernel(AcceptArgs a) {
    __shared__ WideShared sh;
    const int b = blockIdx.x;
    const float* P = a.p_logits + (int64_t)b * (a.k + 1) * a.V;
    int n = 0, am;
    while (true) {
        am = wide_argmax(WideRow(P + (int64_t)n * a.V, a.V), sh);
        if (n < a.k && greedy_keeps(am, a.draft_tokens[b * a.k + n])) ++n; else break;
    }
    if (threadIdx.x == 0) {
        if (a.n_accepted) a.n_accepted[b] = n;
        if (a.next_token) a.next_token[b] = greedy_token(am);
    }
}

// =================================================================================================
// Rows in registers: vocabularies of up to 32768 ids (a multiple of 4, rows 16-byte aligned), greedy rule and draft picks.  One workgroup
// of 1024 threads per sequence; a logits row is loaded once, 32 values per thread as 8 float4 (thread
// t of sweep s holds ids 4096 s + 4 t .. + 3, so running sums stay in ascending id order), and every
// reduction of that row runs on the registers.
// =================================================================================================
constexpr int FAST_THREADS = 1024, FAST_WAVES = FAST_THREADS / 64, FAST_SWEEPS = 8;
constexpr int FAST_MAX_V = FAST_THREADS * 4 * FAST_SWEEPS;

struct FastShared {
    float red[FAST_WAVES];
    int redi[FAST_WAVES];
    float tot[FAST_SWEEPS * FAST_WAVES];     // wave totals of every sweep, then their exclusive prefix
    float total;
    int pick, last;
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
// max and sum of exp((z - max) * inv_tau) of a row held in registers, which becomes those exponentials (padding is -inf: adds 0)
__device__ inline void fast_row_stats(float4 (&v)[FAST_SWEEPS], float inv_tau, FastShared& sh, float* out_max, float* out_sum) {
    float m = -INFINITY;
#pragma unroll
    for (int s = 0; s < FAST_SWEEPS; ++s) m = fmaxf(fmaxf(fmaxf(m, v[s].x), fmaxf(v[s].y, v[s].z)), v[s].w);
    m = fast_block_max(m, sh);
    float sum = 0.f;
#pragma unroll
    for (int s = 0; s < FAST_SWEEPS; ++s) {
        v[s] = make_float4(expf((v[s].x - m) * inv_tau), expf((v[s].y - m) * inv_tau), expf((v[s].z - m) * inv_tau),
                           expf((v[s].w - m) * inv_tau));
        sum += (v[s].x + v[s].y) + (v[s].z + v[s].w);
    }
    *out_max = m;
    *out_sum = fast_block_sum(sum, sh);
}
// argmax of a row held in registers, lowest id on ties
__device__ inline int fast_argmax(const float4 (&v)[FAST_SWEEPS], FastShared& sh) {
    float bv = -INFINITY;
    int bi = NO_ID;
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
        if (n < a.k && greedy_keeps(am, a.draft_tokens[b * a.k + n])) ++n; else break;
    }
    if (threadIdx.x == 0) {
        if (a.n_accepted) a.n_accepted[b] = n;
        if (a.next_token) a.next_token[b] = greedy_token(am);
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
        int bi = NO_ID;
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
        while (n < a.k && greedy_keeps(am[n], a.draft_tokens[b * a.k + n])) ++n;
        if (a.n_accepted) a.n_accepted[b] = n;
        if (a.next_token) a.next_token[b] = greedy_token(am[n]);
    }
}

// The sampling rule on rows of 4 ids and more, at any alignment.  At once: a workgroup for each of the k + 1 rows of a sequence tests its candidate
// and, where it is rejected (or the row is the one behind the last candidate), draws the sequence's next token.  The outputs serve as the
// meeting point: next_token[b] holds the smallest (row << 27 | token) of those that would draw, announced without a token before
// the draw, n_accepted[b] counts the workgroups that are through, and the last one turns both into the results.  Nobody waits.
// A workgroup leaves as soon as it sees a rejection in front of it; those of the first candidates start first, so with more
// workgroups than the chip holds few rows are read for nothing.  In turn: a workgroup per sequence.
//
// Bound by HBM where many rows are read (256 sequences of 8 candidates over 32000 ids, all kept: 557 MB, 116 us), else by the latency of a
// workgroup's few steps, so: several granules of both rows requested ahead of those being summed, in every step as many (their
// predecessors are waited for by count), two workgroups and more to a compute unit so that one's loads run under another's exponentials,
// nothing of a row kept for the draw (it reads the rows again, from the caches).  us per call (calls in a graph, on the same rows: those
// of up to 256 MB come from the last-level cache), none kept / 0.3 of the candidates / 0.8 / all, rows in registers of a
// 1024-thread workgroup or general kernels before -> 256 threads up to 8192 ids at once and 24576 in turn, 512 above:
//   ids     sequences, candidates   before                       at once                      in turn
//   512     4, 4                    24.0 / 24.0 / 23.1 / 18.0    11.9 / 12.0 / 11.0 / 9.9     7.9 / 7.9 / 15.3 / 15.4
//   512     16, 8                   25.4 / 24.8 / 24.1 / 19.1    13.4 / 12.9 / 12.1 / 10.1    8.2 / 13.1 / 23.9 / 24.2
//   1001    16, 8                   9.7 / 19.6 / 34.3 / 34.5     13.3 / 13.0 / 12.5 / 10.4    8.4 / 14.2 / 24.3 / 24.6
//   1001    64, 4                   9.9 / 19.9 / 20.9 / 20.9     14.4 / 14.1 / 13.2 / 12.4    8.4 / 14.0 / 16.0 / 16.2
//   1001    64, 8                   9.8 / 19.8 / 34.5 / 34.7     16.8 / 16.2 / 14.3 / 14.1    8.7 / 13.6 / 24.6 / 24.9
//   4001    100, 8                  40.3 / 39.9 / 50.5 / 52.5    18.2 / 18.4 / 18.6 / 16.0    10.7 / 19.2 / 33.0 / 34.9
//   9001    200, 4                  23.5 / 43.1 / 47.3 / 48.6    19.4 / 28.1 / 27.8 / 27.3    12.9 / 23.7 / 28.4 / 31.0
//   9001    200, 8                  23.5 / 65.0 / 78.2 / 80.4    20.3 / 28.7 / 35.1 / 37.6    13.1 / 34.4 / 45.1 / 49.5
//   20001   128, 8                  33.2 / 77.6 / 121 / 124      31.3 / 37.3 / 43.8 / 43.8    18.8 / 41.9 / 65.4 / 66.6
//   32000   1, 4                    27.3 / 27.1 / 27.0 / 21.8    24.2 / 24.1 / 24.2 / 17.5    20.9 / 21.0 / 21.0 / 44.3
//   32000   64, 8                   44.3 / 42.6 / 63.1 / 66.6    41.5 / 38.7 / 38.9 / 37.3    21.6 / 42.4 / 77.6 / 78.9
//   32000   128, 4                  28.7 / 63.3 / 68.4 / 71.8    39.4 / 39.8 / 42.9 / 37.8    22.6 / 45.4 / 48.8 / 50.4
//   32000   256, 4                  35.8 / 68.5 / 76.0 / 89.9    39.0 / 56.8 / 59.4 / 56.8    29.8 / 51.8 / 55.8 / 61.8
//   32000   128, 8                  28.8 / 71.2 / 111 / 127      40.0 / 46.3 / 55.7 / 55.4    22.4 / 51.7 / 79.6 / 87.0
//   32000   256, 8                  35.8 / 98.9 / 132 / 163      41.0 / 58.1 / 81.0 / 116     31.2 / 73.2 / 91.7 / 112
//   65537   16, 4                   70.0 / 68.5 / 68.2 / 39.2    40.7 / 39.8 / 39.0 / 26.0    34.7 / 71.5 / 74.8 / 75.5
//   65537   256, 4                  77.5 / 151 / 178 / 187       71.7 / 105 / 118 / 123       49.6 / 89.5 / 99.4 / 119
// In turn, then: short rows, but for few sequences of many candidates, and many sequences of up to four.  Faster than before at every rate but for short
// rows off 16 bytes of few sequences (1001 ids, 16, 8: 13.3 against 9.7 with nothing kept) and, of 128 sequences and more, 24577 to 32768 ids and more
// than four candidates (1.1 to 1.44 of it with nothing kept, 0.4 to 0.75 from 0.3 on) and 5000 to 8192 ids and 16 (1.1 to 1.27, 0.2 to 0.45).
// 256 against 512 threads at once, 9001 ids, 200 sequences of 8: 28.5 / 30.5 / 34.5 / 32 against 20.3 / 28.7 / 35.1 / 37.6; 6001 ids, 256 of 8: 24 / 27 /
// 30 / 30 against 19 / 28 / 37 / 41.  Tried and not kept: the non-temporal hint on the rows (256 of 6 over 32000 ids 66 -> 68, 100 of 4 over 32768 35.9 -> 32.5), asking
// for a rejection in front with every step (66 -> 75: the word of a sequence is in memory, and all ask for few lines of it).
constexpr int SHORT_MAX_V = 3072, IN_TURN_MAX_K = 4, IN_TURN_MIN_B = 128, IN_TURN_SHORT_MIN_B = 32, ROWS_256_AHEAD_MAX_V = 8192, ROWS_256_MAX_V = 24576;
// Greedy at once: where all rows are few enough to read (ROWS_MAX_IDS) and several may be kept, so that what is read for nothing where the first
// differs is little against the rows that come one behind the other where it does not.  us, in turn -> at once, first differs / 0.3 / 0.8 of the
// candidates agree / all: 9001 ids 16, 4 5.6 / 14.0 / 17.4 / 17.5 -> 8.8 / 8.6 / 8.6 / 8.4, 100, 8 5.7 / 14.0 / 29.1 / 31.9 -> 11.9 / 11.7 / 11.3 / 11.3;
// 32000 16, 8 5.7 / 14.5 / 30.5 / 30.7 -> 10.2 / 9.7 / 9.8 / 9.7; 65537 16, 2 8.6 / 20.1 / 20.5 / 20.6 -> 11.4 / 11.5 / 11.4 / 11.3.  In turn: 32000 16, 2
// 5.8 / 11.4 / 11.9 / 12.2 -> 9.0 / 9.0 / 9.0 / 8.8, 64, 4 5.9 / 14.5 / 19.5 / 21.3 -> 13.1 / 13.4 / 13.3 / 13.6, 64, 8 5.9 / 14.5 / 34.6 / 35.7 -> 18.2 / 18.2 / 18.4 / 18.4;
// 9001 256, 8 6.1 / 22.6 / 31.7 / 34.9 -> 18.3 / 19.3 / 19.9 / 20.5.
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
__device__ inline void announce_pick(const AcceptArgs& a, int b, int i) {
    __hip_atomic_fetch_min((uint32_t*)a.next_token + b, ((uint32_t)i << PICK_BITS) | PICK_NO_TOKEN, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// (the wait is for the value that the minimum gives back: it has been done then)
__device__ inline void offer_pick(const AcceptArgs& a, int b, int i, uint32_t token) {
    const uint32_t was = __hip_atomic_fetch_min((uint32_t*)a.next_token + b, ((uint32_t)i << PICK_BITS) | token, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("" :: "v"(was) : "memory");
}
// (one thread) this workgroup is through; the last of the sequence writes the results.  All that the workgroups of a sequence tell each
// other are these atomics, so it is enough that a workgroup's offer has been done (offer_pick waits for it) in front of its count.  (A
// release and an acquire at device scope would write back and invalidate the whole L2 every time: 20 ns of the whole chip's
// time a workgroup, 52 against 9 us for 256 sequences of 8 candidates over 512 ids.)
__device__ inline void report(const AcceptArgs& a, int b) {
    if (__hip_atomic_fetch_add(a.n_accepted + b, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != a.k) return;
    const uint32_t v = __hip_atomic_load((uint32_t*)a.next_token + b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    a.n_accepted[b] = (int)(v >> PICK_BITS);
    a.next_token[b] = (int)(v & PICK_NO_TOKEN);
}
// AHEAD: a workgroup per row, else one per sequence that tests its candidates in turn (where a caller leaves out an output)
template <int T, bool AHEAD>
__global__ void __launch_bounds__(T, 4)
accept_rows_kernel(AcceptArgs a) {
    __shared__ RowShared<T> sh;
    const int b = AHEAD ? blockIdx.x % a.B : blockIdx.x, k = a.k, V = a.V;
    int i = AHEAD ? blockIdx.x / a.B : 0;
    const float it = a.inv_tau;
    if (AHEAD) {
        if (threadIdx.x == 0) sh.stop = rejected_before(a, b, i);
        __syncthreads();
        if (sh.stop) {
            if (threadIdx.x == 0) report(a, b);
            return;
        }
    }
    const float *p, *q;
    float pm, ps, qm = 0.f, qs = 1.f;
    while (true) {
        p = a.p_logits + ((int64_t)b * (k + 1) + i) * V;
        q = a.q_logits + ((int64_t)b * k + (i < k ? i : 0)) * V;
        Candidate cand;
        if (i < k && threadIdx.x == 0) cand = candidate(a, b, i);
        if (i < k) row_stats<T, true>(p, q, V, it, sh, &pm, &ps, &qm, &qs);
        else row_stats<T, false>(p, p, V, it, sh, &pm, &ps, nullptr, nullptr);
        if (threadIdx.x == 0) {
            bool draws = i == k || rejects(cand, it, pm, ps, qm, qs);
            if (AHEAD) {
                draws = draws && !rejected_before(a, b, i);
                if (draws) announce_pick(a, b, i);
            }
            sh.stop = draws;
        }
        __syncthreads();
        if (AHEAD || sh.stop) break;
        __syncthreads();
        ++i;
    }
    if (sh.stop) {
        // the draw behind i kept candidates: from the residual of the two rows or (i == k) from the target's
        const float u = a.u_resample ? a.u_resample[b * (k + 1) + i] : philox_uniform(a.seed, a.round, a.seq_base + b, (uint32_t)i, 2);
        float tot = 0.f;
        int nxt = 0;
        if (i < k) nxt = row_draw<T, true>(p, q, V, it, pm, 1.0f / ps, qm, 1.0f / qs, u, sh, &tot);
        if (i == k || !(tot > 0.f)) nxt = row_draw<T, false>(p, p, V, it, pm, 1.0f / ps, 0.f, 0.f, u, sh, &tot);    // (p == q everywhere: the target row)
        if (threadIdx.x == 0) {
            if (AHEAD) offer_pick(a, b, i, (uint32_t)nxt);
            else {
                if (a.n_accepted) a.n_accepted[b] = i;
                if (a.next_token) a.next_token[b] = nxt;
            }
        }
    }
    if (AHEAD && threadIdx.x == 0) report(a, b);
}
// greedy: a workgroup per row; a row whose argmax is not its candidate (or the one behind the last candidate) offers the argmax
__global__ void __launch_bounds__(512)
accept_greedy_ahead_kernel(AcceptArgs a) {
    constexpr int T = 512;
    __shared__ float red[T / 64];
    __shared__ int redi[T / 64], stop;
    const int b = blockIdx.x % a.B, i = blockIdx.x / a.B, V = a.V, lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (threadIdx.x == 0) stop = rejected_before(a, b, i);
    __syncthreads();
    if (!stop) {
        const float* row = a.p_logits + ((int64_t)b * (a.k + 1) + i) * V;
        float bv = -INFINITY;
        int bi = NO_ID;
        float4 v[2][4];
        auto request = [&](int buf, int g0) {
#pragma unroll
            for (int q = 0; q < 4; ++q) v[buf][q] = row_load(row, V, g0 + q * T + (int)threadIdx.x);
        };
        auto take = [&](int buf, int g0) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int g = g0 + q * T + (int)threadIdx.x;
                const float4 z = 4 * (g - lane) + 256 <= V ? v[buf][q] : row_ids(v[buf][q], V, g);
                const float x[4] = {z.x, z.y, z.z, z.w};
#pragma unroll
                for (int j = 0; j < 4; ++j) if (x[j] > bv) { bv = x[j]; bi = 4 * g + j; }
            }
        };
        request(0, 0);
        for (int g0 = 0; g0 < (V + 3) >> 2; g0 += 8 * T) {
            request(1, g0 + 4 * T);
            take(0, g0);
            request(0, g0 + 8 * T);
            take(1, g0 + 4 * T);
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const float ov = __shfl_xor(bv, o, 64);
            const int oi = __shfl_xor(bi, o, 64);
            if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
        }
        if (lane == 0) { red[wv] = bv; redi[wv] = bi; }
        __syncthreads();
        if (threadIdx.x == 0) {
            bv = red[0]; bi = redi[0];
#pragma unroll
            for (int w = 1; w < T / 64; ++w) if (red[w] > bv || (red[w] == bv && redi[w] < bi)) { bv = red[w]; bi = redi[w]; }
            if (i == a.k || !greedy_keeps(bi, a.draft_tokens[b * a.k + i])) offer_pick(a, b, i, (uint32_t)greedy_token(bi));
        }
    }
    if (threadIdx.x == 0) report(a, b);
}
static inline bool fast_rows_ok(const float* base, int V) {
    return V % 4 == 0 && V <= FAST_MAX_V && ((uintptr_t)base & 15) == 0;
}

template <int T, bool AHEAD>
static void launch_accept_rows(const AcceptArgs& a, hipStream_t st) {
    if (AHEAD) hipLaunchKernelGGL(accept_begin_kernel, dim3((a.B + 255) / 256), dim3(256), 0, st, a);
    hipLaunchKernelGGL((accept_rows_kernel<T, AHEAD>), dim3(AHEAD ? a.B * (a.k + 1) : a.B), dim3(T), 0, st, a);
}

hipError_t launch_accept(const AcceptArgs& a, hipStream_t st) {
    if (a.B <= 0) return hipSuccess;
    const bool fast = fast_rows_ok(a.p_logits, a.V);
    const bool can = a.n_accepted && a.next_token && a.V >= 4 && a.V < (int)PICK_NO_TOKEN;      // (the outputs are the meeting point)
    const int64_t ids = (int64_t)a.B * (a.k + 1) * a.V;
    if (a.q_logits) {
        // (figures at the kernel)
        const bool turn = a.V <= SHORT_MAX_V ? a.k <= IN_TURN_MAX_K || a.B >= IN_TURN_SHORT_MIN_B : a.k <= IN_TURN_MAX_K && a.B >= IN_TURN_MIN_B;
        if (a.V < 4) hipLaunchKernelGGL(accept_sample_tiny_kernel, dim3((a.B + 63) / 64), dim3(64), 0, st, a);
        else if (can && !turn) a.V <= ROWS_256_AHEAD_MAX_V ? launch_accept_rows<256, true>(a, st) : launch_accept_rows<512, true>(a, st);
        else a.V <= ROWS_256_MAX_V ? launch_accept_rows<256, false>(a, st) : launch_accept_rows<512, false>(a, st);
    } else if (a.V <= ROWS_MAX_V && (!fast || ids <= ROWS_MAX_IDS)) {
        hipLaunchKernelGGL(accept_greedy_rows_kernel, dim3(a.B), dim3(FAST_THREADS), 0, st, a);
    } else if (can && a.k >= (a.V > FAST_MAX_V ? 2 : 3) && ids <= ROWS_MAX_IDS) {
        hipLaunchKernelGGL(accept_begin_kernel, dim3((a.B + 255) / 256), dim3(256), 0, st, a);
        hipLaunchKernelGGL(accept_greedy_ahead_kernel, dim3(a.B * (a.k + 1)), dim3(512), 0, st, a);
    } else if (fast) {
        hipLaunchKernelGGL(accept_greedy_kernel, dim3(a.B), dim3(FAST_THREADS), 0, st, a);
    } else {
        hipLaunchKernelGGL(accept_greedy_generic_kernel, dim3(a.B), dim3(WIDE_THREADS), 0, st, a);
    }
    return hipGetLastError();
}

// ---- draft token pick ---------------------------------------------------------------------------
template <int T>
__global__ void __launch_bounds__(T)
draft_sample_kernel(const float* __restrict__ z, int64_t ld, int V, float inv_tau, uint64_t seed, uint32_t round, uint32_t seq_base, int step,
                    int32_t* __restrict__ draft_tokens, int k) {
    __shared__ RowShared<T> sh;
    const int b = blockIdx.x;
    const float* row = z + (int64_t)b * ld;
    const float u = philox_uniform(seed, round, seq_base + b, (uint32_t)step, 0);
    float m, s, tot;
    int pick;
    if (V < 4) {
        tiny_stats(row, V, inv_tau, &m, &s);
        pick = tiny_inverse_cdf([&](int c) { return expf((row[c] - m) * inv_tau); }, V, u, &tot);
    } else {
        row_stats<T, false>(row, row, V, inv_tau, sh, &m, &s, nullptr, nullptr);
        pick = row_draw<T, false>(row, row, V, inv_tau, m, 1.0f, 0.f, 0.f, u, sh, &tot);
    }
    if (threadIdx.x == 0) draft_tokens[b * k + step - 1] = pick;
}
__global__ void __launch_bounds__(WIDE_THREADS)
draft_argmax_kernel(const float* __restrict__ z, int64_t ld, int V, int step, int32_t* __restrict__ draft_tokens, int k) {
    __shared__ WideShared sh;
    const int b = blockIdx.x, pick = greedy_token(wide_argmax(WideRow(z + (int64_t)b * ld, V), sh));
    if (threadIdx.x == 0) draft_tokens[b * k + step - 1] = pick;
}
__global__ void __launch_bounds__(NARROW_THREADS)
draft_argmax_narrow_kernel(const float* __restrict__ z, int64_t ld, int V, int step, int32_t* __restrict__ draft_tokens, int k) {
    __shared__ float shf[4];
    __shared__ int shi[4];
    const int b = blockIdx.x, pick = greedy_token(narrow_argmax(z + (int64_t)b * ld, V, shf, shi));
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
        pick = greedy_token(fast_argmax(row, sh));
    } else {
        float m, s, tot;
        fast_row_stats(row, inv_tau, sh, &m, &s);        // (the row is its exponentials now)
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
    else if (mode == SPEC_GREEDY && V <= NARROW_MAX_V)
        hipLaunchKernelGGL(draft_argmax_narrow_kernel, dim3(B), dim3(NARROW_THREADS), 0, st, z, ld, V, step, draft_tokens, k);
    else if (mode == SPEC_GREEDY)
        hipLaunchKernelGGL(draft_argmax_kernel, dim3(B), dim3(WIDE_THREADS), 0, st, z, ld, V, step, draft_tokens, k);
    else if (V <= ROWS_256_MAX_V)
        hipLaunchKernelGGL(draft_sample_kernel<256>, dim3(B), dim3(256), 0, st, z, ld, V, inv_tau, seed, round, seq_base, step, draft_tokens, k);
    else
        hipLaunchKernelGGL(draft_sample_kernel<512>, dim3(B), dim3(512), 0, st, z, ld, V, inv_tau, seed, round, seq_base, step, draft_tokens, k);
    return hipGetLastError();
}

}  // namespace sv
