// Element-wise / gather / normalisation / routing kernels and the plain (non-MFMA) GEMM and
// attention used for f32 models.  All are HBM- or latency-bound; they are written for 64-wide
// wavefronts with coalesced row accesses.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "common.h"

namespace sv {

typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4_t;

#define DISPATCH_DTYPE(dtype, ...)                                     \
    do {                                                               \
        if ((dtype) == SPEC_F32) { using T = float; __VA_ARGS__; }     \
        else { using T = bf16; __VA_ARGS__; }                          \
    } while (0)

// fill n 32-bit words with one value (grid-stride; used to clear or poison buffers on a stream without
// a memset node, which must stay out of captured graphs)
__global__ void fill_words_kernel(uint32_t* __restrict__ p, size_t n, uint32_t v) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = v;
}
hipError_t launch_fill_words(void* p, size_t n_words, uint32_t v, hipStream_t st) {
    if (n_words == 0) return hipSuccess;
    const size_t blocks = std::min<size_t>((n_words + 255) / 256, 4096);
    hipLaunchKernelGGL(fill_words_kernel, dim3((unsigned)blocks), dim3(256), 0, st, (uint32_t*)p, n_words, v);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// The rows of a pass in one kernel, a workgroup per row: which token at which position (RowSource), its residual
// stream x[t] = Emb[token] (or the caller's row t), and its rotary table cs[t] (positions are the same for every
// layer of a pass), computed in double so that large positions lose nothing.  As three launches
// (tokens and positions, gather, table) this was 13 to 20 us of every pass and draft step, all of it launch and
// latency; 32768 rows of 4096 were gathered by 2-byte loads at 3.4 TB/s.
// ---------------------------------------------------------------------------------------------
template <typename T>
__global__ void __launch_bounds__(256)
rows_prep_kernel(RowSource src, const T* __restrict__ rows, float* __restrict__ x, int32_t* __restrict__ row_pos,
                 float2* __restrict__ cs, int d, int vocab, int half, double theta, int vec) {
    const int t = blockIdx.x, tid = threadIdx.x;
    int pos, tok;
    src.row(t, pos, tok);
    if (tid == 0) row_pos[t] = pos;
    const T* from = rows + (int64_t)(src.embed ? (tok < 0 ? 0 : (tok >= vocab ? vocab - 1 : tok)) : t) * d;
    float* to = x + (int64_t)t * d;
    if (vec) {
        for (int c = tid * 8; c < d; c += 256 * 8) {
            alignas(16) T v[8];
            *(uint4*)v = *(const uint4*)(from + c);
            if constexpr (sizeof(T) == 4) *(uint4*)(v + 4) = *(const uint4*)(from + c + 4);
            *(float4*)(to + c) = make_float4(to_f32<T>(v[0]), to_f32<T>(v[1]), to_f32<T>(v[2]), to_f32<T>(v[3]));
            *(float4*)(to + c + 4) = make_float4(to_f32<T>(v[4]), to_f32<T>(v[5]), to_f32<T>(v[6]), to_f32<T>(v[7]));
        }
    } else {
        for (int c = tid; c < d; c += 256) to[c] = to_f32<T>(from[c]);
    }
    for (int i = tid; i < half; i += 256) {
        double inv = pow(theta, -(double)i / (double)half);      // theta^(-2i/dh)
        double a = (double)pos * inv;
        double s, c;
        sincos(a, &s, &c);
        cs[(int64_t)t * half + i] = make_float2((float)c, (float)s);
    }
}
hipError_t launch_rows_prep(const RowSource& src, const void* rows, float* x, int32_t* row_pos, float2* cs, int T_, int d,
                            int vocab, int half, float theta, int dtype, hipStream_t st) {
    if (T_ <= 0) return hipSuccess;
    const int vec = d % 8 == 0 && (((uintptr_t)rows | (uintptr_t)x) & 15) == 0;
    DISPATCH_DTYPE(dtype, hipLaunchKernelGGL(rows_prep_kernel<T>, dim3(T_), dim3(256), 0, st, src, (const T*)rows, x, row_pos,
                                             cs, d, vocab, half, (double)theta, vec));
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// (MoE combine) + RMSNorm.  One 256-thread workgroup per row.
//   if y:  x[t] += w[t,0] * y[slot[t,0]] + w[t,1] * y[slot[t,1]]      (first choice first)
//   if g:  h[t]  = x[t] * rsqrt(mean(x[t]^2) + eps) * g               (stored in the model dtype)
// ---------------------------------------------------------------------------------------------
template <typename T>
__global__ void combine_norm_kernel(float* __restrict__ x, const float* __restrict__ y,
                                    const float* __restrict__ wts, const int32_t* __restrict__ slots,
                                    const T* __restrict__ g, T* __restrict__ h, int d, float eps) {
    __shared__ float red[4];
    int t = blockIdx.x;
    float* xr = x + (int64_t)t * d;
    float ss = 0.f;
    if (y && (wts[2 * t] != 0.f || wts[2 * t + 1] != 0.f)) {       // (a row without experts has weights 0)
        float w0 = wts[2 * t], w1 = wts[2 * t + 1];
        const float* y0 = y + (int64_t)slots[2 * t] * d;
        const float* y1 = y + (int64_t)slots[2 * t + 1] * d;
        for (int c = threadIdx.x; c < d; c += blockDim.x) {
            float v = xr[c] + (w0 * y0[c] + w1 * y1[c]);
            xr[c] = v;
            ss += v * v;
        }
    } else if (g) {
        for (int c = threadIdx.x; c < d; c += blockDim.x) { float v = xr[c]; ss += v * v; }
    }
    if (!g) return;
    ss = wave_sum(ss);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
    __syncthreads();
    float tot = red[0] + red[1] + red[2] + red[3];
    float r = 1.0f / sqrtf(tot / (float)d + eps);
    T* hr = h + (int64_t)t * d;
    for (int c = threadIdx.x; c < d; c += blockDim.x) hr[c] = from_f32<T>(xr[c] * r * to_f32<T>(g[c]));
}

// the squares of 8 elements onto a sum (of none yet, if `first`), written out so that every kernel that normalises has the same bits
__device__ inline float squares8(float ss, const float (&v)[8], bool first) {
    ss = first ? fmaf(v[0], v[0], v[1] * v[1]) : fmaf(v[1], v[1], fmaf(v[0], v[0], ss));
#pragma unroll
    for (int e = 2; e < 8; ++e) ss = fmaf(v[e], v[e], ss);
    return ss;
}

// Same operation with the row held in registers (8 consecutive elements per thread and chunk, 16-byte
// loads and stores, one pass): for d % 8 == 0 and d <= 8 * 256 * COMBINE_CHUNKS; CH is the row's count of 2048-wide
// chunks.  The gains are requested with the row, not behind the reduction (round of 32 sequences, 40
// such launches of 32 and 224 rows: 3845 -> 3832 us).
constexpr int COMBINE_CHUNKS = 4;
template <typename T, int CH>
__global__ void __launch_bounds__(256)
combine_norm_vec_kernel(float* __restrict__ x, const float* __restrict__ y, const float* __restrict__ wts,
                        const int32_t* __restrict__ slots, const T* __restrict__ g, T* __restrict__ h, int d,
                        float eps) {
    __shared__ float red[4];
    const int t = blockIdx.x, tid = threadIdx.x;
    float* xr = x + (int64_t)t * d;
    float v[CH][8];
    alignas(16) T gv[CH][8];
    float ss = 0.f;
    float w0 = 0.f, w1 = 0.f;
    const float* y0 = nullptr;
    const float* y1 = nullptr;
#pragma unroll
    for (int q = 0; q < CH; ++q) {
        const int c = (q * 256 + tid) * 8;
        if (c < d) {
            const float4 a = *(const float4*)(xr + c), b = *(const float4*)(xr + c + 4);
            v[q][0] = a.x; v[q][1] = a.y; v[q][2] = a.z; v[q][3] = a.w;
            v[q][4] = b.x; v[q][5] = b.y; v[q][6] = b.z; v[q][7] = b.w;
            if (g) {
                *(uint4*)gv[q] = *(const uint4*)(g + c);
                if (sizeof(T) == 4) *(uint4*)(gv[q] + 4) = *(const uint4*)(g + c + 4);
            }
        }
    }
    if (y) {
        w0 = wts[2 * t]; w1 = wts[2 * t + 1];
        const int s0 = slots[2 * t], s1 = slots[2 * t + 1];
        if (w0 == 0.f && w1 == 0.f) y = nullptr;                   // a row without experts: nothing to add
        else { y0 = y + (int64_t)s0 * d; y1 = y + (int64_t)s1 * d; }
    }
#pragma unroll
    for (int q = 0; q < CH; ++q) {
        const int c = (q * 256 + tid) * 8;
        if (c < d) {
            if (y) {
                const float4 p0 = *(const float4*)(y0 + c), p1 = *(const float4*)(y0 + c + 4);
                const float4 q0 = *(const float4*)(y1 + c), q1 = *(const float4*)(y1 + c + 4);
                const float e0[8] = {p0.x, p0.y, p0.z, p0.w, p1.x, p1.y, p1.z, p1.w};
                const float e1[8] = {q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w};
#pragma unroll
                for (int e = 0; e < 8; ++e) v[q][e] = v[q][e] + (w0 * e0[e] + w1 * e1[e]);
                *(float4*)(xr + c) = make_float4(v[q][0], v[q][1], v[q][2], v[q][3]);
                *(float4*)(xr + c + 4) = make_float4(v[q][4], v[q][5], v[q][6], v[q][7]);
            }
            ss = squares8(ss, v[q], q == 0);
        }
    }
    if (!g) return;
    ss = wave_sum(ss);
    if ((tid & 63) == 0) red[tid >> 6] = ss;
    __syncthreads();
    const float r = 1.0f / sqrtf((red[0] + red[1] + red[2] + red[3]) / (float)d + eps);
    T* hr = h + (int64_t)t * d;
#pragma unroll
    for (int q = 0; q < CH; ++q) {
        const int c = (q * 256 + tid) * 8;
        if (c < d) {
            alignas(16) T hv[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) hv[i] = from_f32<T>(v[q][i] * r * to_f32<T>(gv[q][i]));
            if (sizeof(T) == 2) *(uint4*)(hr + c) = *(const uint4*)hv;
            else { *(uint4*)(hr + c) = *(const uint4*)hv; *(uint4*)(hr + c + 4) = *(const uint4*)(hv + 4); }
        }
    }
}

hipError_t launch_combine_norm(float* x, const float* y, const float* wts, const int32_t* slots,
                               const void* g, void* h, int T_, int d, float eps, int dtype,
                               hipStream_t st) {
    if (T_ <= 0) return hipSuccess;
    if (d % 8 == 0 && d <= 8 * 256 * COMBINE_CHUNKS) {
        DISPATCH_DTYPE(dtype, {
            auto kern = d <= 2048 ? combine_norm_vec_kernel<T, 1> : d <= 4096 ? combine_norm_vec_kernel<T, 2>
                      : d <= 6144 ? combine_norm_vec_kernel<T, 3> : combine_norm_vec_kernel<T, 4>;
            hipLaunchKernelGGL(kern, dim3(T_), dim3(256), 0, st, x, y, wts, slots, (const T*)g, (T*)h, d, eps);
        });
    } else {
        DISPATCH_DTYPE(dtype, hipLaunchKernelGGL(combine_norm_kernel<T>, dim3(T_), dim3(256), 0, st, x, y,
                                                 wts, slots, (const T*)g, (T*)h, d, eps));
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// RoPE: rotate q,k (pair (i, i+dh/2)) with the rows' table and append k,v to the sequence's KV pages.
// ---------------------------------------------------------------------------------------------
template <typename T>
__global__ void rope_kv_kernel(const float* __restrict__ qkv, const float2* __restrict__ cs,
                               const int32_t* __restrict__ row_pos,
                               const int32_t* __restrict__ page_table, T* __restrict__ q_out,
                               T* __restrict__ kv_layer, KvGeom geom, int n_new, int n_q_heads) {
    int t = blockIdx.x;
    int dh = geom.head_dim, half = dh >> 1, Hkv = geom.n_kv_heads;
    int n_heads = n_q_heads + 2 * Hkv;
    int pos = row_pos[t];
    int b = t / n_new;
    const float* row = qkv + (int64_t)t * n_heads * dh;
    int64_t page = -1;
    int slot = 0;
    if (pos >= 0) {
        int lp = pos / geom.page_tokens;
        if (lp < geom.pages_per_seq) { page = page_table[b * geom.pages_per_seq + lp]; slot = pos % geom.page_tokens; }
    }
    for (int idx = threadIdx.x; idx < n_heads * half; idx += blockDim.x) {
        int hd = idx / half, i = idx % half;
        float a = row[hd * dh + i], bb = row[hd * dh + i + half];
        if (hd < n_q_heads + Hkv) {
            float2 c = cs[t * half + i];
            float ra = a * c.x - bb * c.y, rb = bb * c.x + a * c.y;
            a = ra; bb = rb;
        }
        if (hd < n_q_heads) {
            T* dst = q_out + (int64_t)t * n_q_heads * dh + hd * dh;
            dst[i] = from_f32<T>(a); dst[i + half] = from_f32<T>(bb);
        } else if (page >= 0) {
            if (hd < n_q_heads + Hkv) {
                T* dst = kv_layer + geom.k_off(page, hd - n_q_heads, slot);
                dst[i] = from_f32<T>(a); dst[i + half] = from_f32<T>(bb);
            } else {
                int kvh = hd - n_q_heads - Hkv;
                kv_layer[geom.v_off(page, kvh, slot, i)] = from_f32<T>(a);
                kv_layer[geom.v_off(page, kvh, slot, i + half)] = from_f32<T>(bb);
            }
        }
    }
}
hipError_t launch_rope_kv(const float* qkv, const float2* cs, const int32_t* row_pos,
                          const int32_t* page_table, void* q_out, void* kv_layer, KvGeom geom, int T_,
                          int n_new, int n_q_heads, int dtype, hipStream_t st) {
    if (T_ <= 0) return hipSuccess;
    DISPATCH_DTYPE(dtype, hipLaunchKernelGGL(rope_kv_kernel<T>, dim3(T_), dim3(256), 0, st, qkv, cs,
                                             row_pos, page_table, (T*)q_out, (T*)kv_layer, geom, n_new,
                                             n_q_heads));
    return hipGetLastError();
}

// The same for a bf16 model of head_dim 128, 16-byte accesses: 16 lanes take one head of a row (dims
// 4 l .. 4 l + 3 and their rotation partners 64 above), a workgroup 16 heads.  Rotation and rounding are
// written as in the projection's fused epilogue: both ways give the same bits.
__global__ void __launch_bounds__(256)
rope_kv_bf16_kernel(const float* __restrict__ qkv, const float2* __restrict__ cs, const int32_t* __restrict__ row_pos,
                        const int32_t* __restrict__ page_table, bf16* __restrict__ q_out, bf16* __restrict__ kv_layer,
                        KvGeom geom, int n_new, int n_q_heads) {
    const int t = blockIdx.x, hd = blockIdx.y * 16 + (threadIdx.x >> 4), i = (threadIdx.x & 15) * 4;
    const int Hkv = geom.n_kv_heads, n_heads = n_q_heads + 2 * Hkv;
    if (hd >= n_heads) return;
    const int pos = row_pos[t];
    const float* src = qkv + ((int64_t)t * n_heads + hd) * 128 + i;
    f32x4_t lo = *(const f32x4_t*)src, hi = *(const f32x4_t*)(src + 64);
    const bool is_q = hd < n_q_heads, is_k = !is_q && hd < n_q_heads + Hkv;
    if (is_q || is_k) {
        const float4 c01 = *(const float4*)(cs + (int64_t)t * 64 + i), c23 = *(const float4*)(cs + (int64_t)t * 64 + i + 2);
        const float c[4] = {c01.x, c01.z, c23.x, c23.z}, sn[4] = {c01.y, c01.w, c23.y, c23.w};
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float x0 = lo[r], x1 = hi[r];
            lo[r] = x0 * c[r] - x1 * sn[r];
            hi[r] = x1 * c[r] + x0 * sn[r];
        }
    }
    const bf16x4_t l4 = __builtin_convertvector(lo, bf16x4_t), h4 = __builtin_convertvector(hi, bf16x4_t);
    bf16* dst;
    if (is_q) dst = q_out + ((int64_t)t * n_q_heads + hd) * 128 + i;
    else {
        if (pos < 0) return;
        const int lp = pos / geom.page_tokens, slot = pos % geom.page_tokens;
        if (lp >= geom.pages_per_seq) return;
        const int64_t page = page_table[(t / n_new) * geom.pages_per_seq + lp];
        if (!is_k) {
            const int kvh = hd - n_q_heads - Hkv;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                *(__bf16*)(kv_layer + geom.v_off(page, kvh, slot, i + r)) = l4[r];
                *(__bf16*)(kv_layer + geom.v_off(page, kvh, slot, 64 + i + r)) = h4[r];
            }
            return;
        }
        dst = kv_layer + geom.k_off(page, hd - n_q_heads, slot) + i;
    }
    *(bf16x4_t*)dst = l4;
    *(bf16x4_t*)(dst + 64) = h4;
}
hipError_t launch_rope_kv_bf16(const float* qkv, const float2* cs, const int32_t* row_pos, const int32_t* page_table,
                                   void* q_out, void* kv_layer, KvGeom geom, int T_, int n_new, int n_q_heads, hipStream_t st) {
    if (T_ <= 0) return hipSuccess;
    if (geom.head_dim != 128) return hipErrorInvalidValue;
    const int n_heads = n_q_heads + 2 * geom.n_kv_heads;
    hipLaunchKernelGGL(rope_kv_bf16_kernel, dim3(T_, (n_heads + 15) / 16), dim3(256), 0, st, qkv, cs, row_pos, page_table,
                       (bf16*)q_out, (bf16*)kv_layer, geom, n_new, n_q_heads);
    return hipGetLastError();
}

template <typename T>
__global__ void kv_import_kernel(const T* __restrict__ k_ctx, const T* __restrict__ v_ctx,
                                 T* __restrict__ kv_layer, const int32_t* __restrict__ page_table,
                                 KvGeom geom, int ctx_len) {
    // one workgroup per (b, kv head, position)
    int64_t id = blockIdx.x;
    int pos = (int)(id % ctx_len);
    int kvh = (int)((id / ctx_len) % geom.n_kv_heads);
    int b = (int)(id / ctx_len / geom.n_kv_heads);
    int64_t page = page_table[b * geom.pages_per_seq + pos / geom.page_tokens];
    int slot = pos % geom.page_tokens;
    const T* ks = k_ctx + id * geom.head_dim;
    const T* vs = v_ctx + id * geom.head_dim;
    T* kd = kv_layer + geom.k_off(page, kvh, slot);
    for (int c = threadIdx.x; c < geom.head_dim; c += blockDim.x) {
        kd[c] = ks[c];
        kv_layer[geom.v_off(page, kvh, slot, c)] = vs[c];
    }
}
hipError_t launch_kv_import(const void* k_ctx, const void* v_ctx, void* kv_layer,
                            const int32_t* page_table, KvGeom geom, int B, int ctx_len, int dtype,
                            hipStream_t st) {
    int64_t n = (int64_t)B * geom.n_kv_heads * ctx_len;
    if (n <= 0) return hipSuccess;
    DISPATCH_DTYPE(dtype, hipLaunchKernelGGL(kv_import_kernel<T>, dim3((unsigned)n), dim3(64), 0, st,
                                             (const T*)k_ctx, (const T*)v_ctx, (T*)kv_layer, page_table,
                                             geom, ctx_len));
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// Router: r = h Wr^T (E <= 8 logits, f32 accumulate), top-2 (lowest id wins ties), weights =
// softmax over the two chosen logits.  One wavefront per token.
// ---------------------------------------------------------------------------------------------
// Top-2 of E router logits (lowest id wins ties) and the softmax over the two chosen logits.  With
// `forced` (two expert ids of this token, a testing aid: the routing of a reference run) the two given
// experts are taken instead, if they are valid and distinct, and only the weights come from the logits.
// An inactive row (a padding row of a prefill chunk, beyond its sequence's prompt) is given no expert at
// all: ids -1 and weights 0, so that the sort leaves it out of every expert's rows.
__device__ inline void pick_top2(const float* lg, int E, const int32_t* forced, bool active, int32_t* ids, float* wts) {
    if (!active) { ids[0] = -1; ids[1] = -1; wts[0] = 0.f; wts[1] = 0.f; return; }
    // (every index a compile-time constant: a lookup lg[i0] would put the logits into scratch memory)
    int i0 = 0, i1 = -1;
    float l0 = lg[0], l1 = 0.f;
#pragma unroll
    for (int e = 1; e < 8; ++e) if (e < E && lg[e] > l0) { i0 = e; l0 = lg[e]; }
#pragma unroll
    for (int e = 0; e < 8; ++e) if (e < E && e != i0 && (i1 < 0 || lg[e] > l1)) { i1 = e; l1 = lg[e]; }
    if (forced) {
        const int f0 = forced[0], f1 = forced[1];
        if (f0 >= 0 && f0 < E && f1 >= 0 && f1 < E && f0 != f1) {
            i0 = f0; i1 = f1;
#pragma unroll
            for (int e = 0; e < 8; ++e) { if (e == i0) l0 = lg[e]; if (e == i1) l1 = lg[e]; }
        }
    }
    const float w0 = 1.0f / (1.0f + expf(l1 - l0));
    ids[0] = i0; ids[1] = i1;
    wts[0] = w0; wts[1] = 1.0f - w0;
}
template <typename T>
__global__ void router_kernel(const T* __restrict__ h, const T* __restrict__ wr,
                              int32_t* __restrict__ ids, float* __restrict__ wts, int T_, int d, int E,
                              const int32_t* __restrict__ forced, const int32_t* __restrict__ row_pos) {
    int t = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    int lane = threadIdx.x & 63;
    if (t >= T_) return;
    float acc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = 0.f;
    const T* hr = h + (int64_t)t * d;
    constexpr int VEC = 16 / sizeof(T);                 // 16-byte loads
    if (d % VEC == 0) {
        // unrolled so that the loads of four column blocks are in flight together (the kernel is
        // bound by the latency of these loads, not by their bytes)
#pragma unroll 4
        for (int c = lane * VEC; c < d; c += 64 * VEC) {
            alignas(16) T hv[VEC];
            *(uint4*)hv = *(const uint4*)(hr + c);
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (e < E) {
                    alignas(16) T wv[VEC];
                    *(uint4*)wv = *(const uint4*)(wr + (int64_t)e * d + c);
#pragma unroll
                    for (int q = 0; q < VEC; ++q) acc[e] += to_f32<T>(hv[q]) * to_f32<T>(wv[q]);
                }
        }
    } else {
        for (int c = lane; c < d; c += 64) {
            float hv = to_f32<T>(hr[c]);
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (e < E) acc[e] += hv * to_f32<T>(wr[(int64_t)e * d + c]);
        }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = wave_sum(acc[e]);
    if (lane == 0) pick_top2(acc, E, forced ? forced + 2 * t : nullptr, !row_pos || row_pos[t] >= 0, ids + 2 * t, wts + 2 * t);
}
hipError_t launch_router(const void* h, const void* wr, int32_t* ids, float* wts, int T_, int d, int E,
                         const int32_t* forced, const int32_t* row_pos, int dtype, hipStream_t st) {
    if (T_ <= 0) return hipSuccess;
    DISPATCH_DTYPE(dtype, hipLaunchKernelGGL(router_kernel<T>, dim3((T_ + 3) / 4), dim3(256), 0, st,
                                             (const T*)h, (const T*)wr, ids, wts, T_, d, E, forced, row_pos));
    return hipGetLastError();
}

// RMSNorm fused with the router (the post-attention norm of an MoE layer): one 256-thread workgroup
// per row keeps the row in registers, writes h = norm(x) * g in the model dtype and multiplies the
// rounded h by the E router rows on the way (same values the stand-alone router reads back from
// memory), then reduces the E logits over the workgroup and picks top-2 as router_kernel does.
// Needs d % 8 == 0 and d <= 8 * 256 * NORM_ROUTE_CHUNKS; CH is the row's count of 2048-wide chunks.  What bounds it is
// latency, so a bf16 router's rows and the gains are requested with the row itself, in front of the reduction
// that they would otherwise wait behind (AHEAD).  Of rows of four chunks that takes 212 registers, two workgroups a compute unit, and pays
// while they are few: 8192 wide, 8 experts, us behind the reduction / with the row: 320 rows 17.0 / 11.2, 640 19.4 / 18.4, 768 19.7 / 19.0,
// 1024 22.7 / 22.9, 1152 22.4 / 27.3, 2304 41.6 / 46.2, 4096 57.4 / 70.4.  6144 wide, 2304 rows 34.4 / 30.0.
constexpr int NORM_ROUTE_CHUNKS = 4, NORM_ROUTE_AHEAD_ROWS = 768;
template <typename T, int CH, bool AHEAD>
__global__ void __launch_bounds__(256)
norm_route_kernel(const float* __restrict__ x, const T* __restrict__ g, T* __restrict__ h,
                  const T* __restrict__ wr, int32_t* __restrict__ ids, float* __restrict__ wts, int d, int E,
                  float eps, const int32_t* __restrict__ forced, const int32_t* __restrict__ row_pos) {
    static_assert(!AHEAD || sizeof(T) == 2, "a router's row as 16-byte words");
    constexpr bool GAINS_AHEAD = AHEAD || sizeof(T) == 4;
    __shared__ float red[4];
    __shared__ float part[4][8];
    const int t = blockIdx.x, tid = threadIdx.x;
    const float* xr = x + (int64_t)t * d;
    auto load8 = [&](const T* p, T* to) {
        *(uint4*)to = *(const uint4*)p;
        if (sizeof(T) == 4) *(uint4*)(to + 4) = *(const uint4*)(p + 4);
    };
    float v[CH][8];
    alignas(16) T gv[CH][8];
    uint4 wv[AHEAD ? CH : 1][8];                      // (whole words: as elements they would take a register each)
#pragma unroll
    for (int q = 0; q < CH; ++q) {
        const int c = (q * 256 + tid) * 8;
        if (c < d) {
            const float4 a = *(const float4*)(xr + c), b = *(const float4*)(xr + c + 4);
            v[q][0] = a.x; v[q][1] = a.y; v[q][2] = a.z; v[q][3] = a.w;
            v[q][4] = b.x; v[q][5] = b.y; v[q][6] = b.z; v[q][7] = b.w;
        }
    }
#pragma unroll
    for (int q = 0; q < CH; ++q) {
        const int c = (q * 256 + tid) * 8;
        if (c < d) {
            if (GAINS_AHEAD) load8(g + c, gv[q]);
            if constexpr (AHEAD) {
#pragma unroll
                for (int e = 0; e < 8; ++e) if (e < E) wv[q][e] = *(const uint4*)(wr + (int64_t)e * d + c);
            }
        }
    }
    float ss = 0.f;
#pragma unroll
    for (int q = 0; q < CH; ++q) {
        if ((q * 256 + tid) * 8 < d) ss = squares8(ss, v[q], q == 0);
    }
    ss = wave_sum(ss);
    if ((tid & 63) == 0) red[tid >> 6] = ss;
    __syncthreads();
    const float r = 1.0f / sqrtf((red[0] + red[1] + red[2] + red[3]) / (float)d + eps);
    float acc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = 0.f;
    T* hr = h + (int64_t)t * d;
#pragma unroll
    for (int q = 0; q < CH; ++q) {
        const int c = (q * 256 + tid) * 8;
        if (c < d) {
            alignas(16) T hv[8];
            float hf[8];
            if (!GAINS_AHEAD) load8(g + c, gv[q]);
#pragma unroll
            for (int i = 0; i < 8; ++i) { hv[i] = from_f32<T>(v[q][i] * r * to_f32<T>(gv[q][i])); hf[i] = to_f32<T>(hv[i]); }
            if (sizeof(T) == 2) *(uint4*)(hr + c) = *(const uint4*)hv;
            else { *(uint4*)(hr + c) = *(const uint4*)hv; *(uint4*)(hr + c + 4) = *(const uint4*)(hv + 4); }
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (e < E) {
                    float w[8];
                    if constexpr (AHEAD) {
                        const uint32_t u[4] = {wv[q][e].x, wv[q][e].y, wv[q][e].z, wv[q][e].w};
#pragma unroll
                        for (int i = 0; i < 8; ++i) w[i] = __uint_as_float(i & 1 ? u[i >> 1] & 0xffff0000u : u[i >> 1] << 16);
                    } else {
                        alignas(16) T we[8];
                        load8(wr + (int64_t)e * d + c, we);
#pragma unroll
                        for (int i = 0; i < 8; ++i) w[i] = to_f32<T>(we[i]);
                    }
#pragma unroll
                    for (int i = 0; i < 8; ++i) acc[e] += hf[i] * w[i];
                }
        }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = wave_sum(acc[e]);
    if ((tid & 63) == 0) {
#pragma unroll
        for (int e = 0; e < 8; ++e) part[tid >> 6][e] = acc[e];
    }
    __syncthreads();
    if (tid == 0) {
        float lg[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) lg[e] = (part[0][e] + part[1][e]) + (part[2][e] + part[3][e]);
        pick_top2(lg, E, forced ? forced + 2 * t : nullptr, !row_pos || row_pos[t] >= 0, ids + 2 * t, wts + 2 * t);
    }
}
bool norm_route_supported(int d, int E) { return d % 8 == 0 && d <= 8 * 256 * NORM_ROUTE_CHUNKS && E >= 2 && E <= 8; }
hipError_t launch_norm_route(const float* x, const void* g, void* h, const void* wr, int32_t* ids, float* wts,
                             int T_, int d, int E, float eps, const int32_t* forced, const int32_t* row_pos, int dtype,
                             hipStream_t st) {
    if (T_ <= 0) return hipSuccess;
    DISPATCH_DTYPE(dtype, {
        constexpr bool B = sizeof(T) == 2;
        auto kern = d <= 2048 ? norm_route_kernel<T, 1, B> : d <= 4096 ? norm_route_kernel<T, 2, B> : d <= 6144 ? norm_route_kernel<T, 3, B>
                  : T_ <= NORM_ROUTE_AHEAD_ROWS ? norm_route_kernel<T, 4, B> : norm_route_kernel<T, 4, false>;
        hipLaunchKernelGGL(kern, dim3(T_), dim3(256), 0, st, x, (const T*)g, (T*)h, (const T*)wr, ids, wts, d, E, eps, forced, row_pos);
    });
    return hipGetLastError();
}

// Stable counting sort of the 2T (token, choice) pairs by expert id, one 1024-thread workgroup.  Pairs
// of rows without experts (id < 0: inactive rows) are left out: offsets[E] is the number of routed pairs.
// Every wavefront takes a contiguous range of the pairs, 64 at a time: a ballot per expert counts them, and in a second
// pass ranks them (lane order is pair order, so the sort is stable).  A scan of per-thread counts over LDS took
// 7.4 us for 640 pairs and 75 us for 65536 (a thread's pairs were neighbours in memory).
__global__ void __launch_bounds__(1024)
moe_sort_kernel(const int32_t* __restrict__ ids, int32_t* __restrict__ offsets,
                int32_t* __restrict__ perm, int32_t* __restrict__ slots, int n_pairs, int E) {
    __shared__ int cnt[16][8];          // pairs of expert e in wavefront w's range, then its first row
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int seg = ((n_pairs + 1023) / 1024) * 64, p0 = w * seg, p1 = min(p0 + seg, n_pairs);
    int run[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) run[q] = 0;
#pragma unroll 4
    for (int p = p0; p < p1; p += 64) {
        const int e = p + lane < p1 ? ids[p + lane] : -1;
#pragma unroll
        for (int q = 0; q < 8; ++q) run[q] += __popcll(__ballot(e == q));
    }
    if (lane == 0) {
#pragma unroll
        for (int q = 0; q < 8; ++q) cnt[w][q] = run[q];
    }
    __syncthreads();
    if (w == 0) {                       // lane q (and its copies): exclusive sums over the experts, then over the wavefronts
        const int q = lane & 7;
        int c[16], total = 0;
#pragma unroll
        for (int v = 0; v < 16; ++v) { c[v] = cnt[v][q]; total += c[v]; }
        int incl = total;
#pragma unroll
        for (int o = 1; o < 8; o <<= 1) {
            const int up = __shfl_up(incl, o, 8);
            if (q >= o) incl += up;
        }
        int base = incl - total;
        if (lane < 8) {
            if (q < E) offsets[q] = base;
            if (q == E - 1) offsets[E] = incl;
#pragma unroll
            for (int v = 0; v < 16; ++v) { cnt[v][q] = base; base += c[v]; }
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 8; ++q) run[q] = cnt[w][q];
    const unsigned long long before = (1ull << lane) - 1;
#pragma unroll 2
    for (int p = p0; p < p1; p += 64) {
        const bool in = p + lane < p1;
        const int e = in ? ids[p + lane] : -1;
        int row = 0;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const unsigned long long m = __ballot(e == q);
            if (e == q) row = run[q] + __popcll(m & before);
            run[q] += __popcll(m);
        }
        if (in) {
            if (e >= 0) perm[row] = (p + lane) >> 1;
            slots[p + lane] = row;
        }
    }
}
hipError_t launch_moe_sort(const int32_t* ids, int32_t* offsets, int32_t* perm, int32_t* slots, int T_,
                           int E, hipStream_t st) {
    hipLaunchKernelGGL(moe_sort_kernel, dim3(1), dim3(1024), 0, st, ids, offsets, perm, slots, 2 * T_, E);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// Plain tiled GEMM (any dtype, any size): 64x64 output tile, 256 threads, 4x4 outputs each.
// Used for f32 models; bf16 models use the MFMA kernels.
// What bounds it is the wait for a step of 16 k, so the next step's elements are requested before this one is multiplied
// (registers: 120 with SwiGLU, four wavefronts a SIMD).  f32 layer of 80 / 576 rows, us, requested when needed / a step ahead:
// 1024 wide 292 / 243 and 1346 / 965, 2048 wide 832 / 664 and 3604 / 2700.
// ---------------------------------------------------------------------------------------------
// f32 sums: four segments of the contraction, each a chain of fused multiply-adds over ascending k, added in ascending order,
// so that four wavefronts can share an output (gemm_f32_kernel) and every f32 kernel gives the same bits.  (bf16 here: one chain.)
__host__ __device__ inline int f32_segment(int K) { return (K + 63) / 64 * 16; }
template <typename T, bool SWIGLU, bool PANELS>
__global__ void __launch_bounds__(256)
gemm_simple_kernel(GemmArgs a) {
    constexpr int BM = 64, BN = 64, BK = 16;
    constexpr bool SEGS = std::is_same<T, float>::value;
    __shared__ float As[BK][BM + 1];
    __shared__ float Ws[BK][BN + 1];
    __shared__ float W3s[SWIGLU ? BK : 1][BN + 1];
    int row_begin = 0, row_end = a.M, group = 0;
    int tile_m = blockIdx.y;
    if (a.group_offsets) {
        int acc_tiles = 0;
        bool found = false;
        for (int g = 0; g < a.n_groups; ++g) {
            int b0 = a.group_offsets[g], b1 = a.group_offsets[g + 1];
            int nt = (b1 - b0 + BM - 1) / BM;
            if (!found && tile_m < acc_tiles + nt) {
                group = g; row_begin = b0 + (tile_m - acc_tiles) * BM; row_end = b1; found = true;
            }
            acc_tiles += nt;
        }
        if (!found) return;
    } else {
        row_begin = tile_m * BM;
        if (row_begin >= a.M) return;
    }
    const T* A = (const T*)a.A;
    const T* W = (const T*)a.W + (int64_t)group * a.w_group_stride;
    const T* W3 = SWIGLU ? (const T*)a.W3 + (int64_t)group * a.w_group_stride : nullptr;
    int col0 = blockIdx.x * BN;
    int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
    float acc[4][4], acc3[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) { acc[i][j] = 0.f; acc3[i][j] = 0.f; }
    float tot[4][4] = {}, tot3[4][4] = {};            // (SEGS: the segments behind the running one)
    // loader mapping: thread loads (row = tid/4, k = (tid%4)*4 .. +3)
    int lr = tid >> 2, lk = (tid & 3) * 4;
    int arow = row_begin + lr;
    int64_t asrc = -1;
    if (arow < row_end) asrc = a.a_rows ? a.a_rows[arow] : arow;
    int wrow = col0 + lr;
    float ra[4], rw[4], rw3[4];
    auto request = [&](int k0) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int kk = k0 + lk + q;
            const bool wv = wrow < a.N && kk < a.K;
            ra[q] = (asrc >= 0 && kk < a.K) ? to_f32<T>(A[asrc * a.lda + kk]) : 0.f;
            rw[q] = wv ? to_f32<T>(W[weight_elem(wrow, kk, a.K, PANELS ? a.w_panel : 0)]) : 0.f;
            if (SWIGLU) rw3[q] = wv ? to_f32<T>(W3[weight_elem(wrow, kk, a.K, PANELS ? a.w_panel : 0)]) : 0.f;
        }
    };
    request(0);
    const int seg = SEGS ? f32_segment(a.K) : a.K;
    for (int k_beg = 0; k_beg < a.K; k_beg += seg) {
    const int k_end = min(k_beg + seg, a.K);
    for (int k0 = k_beg; k0 < k_end; k0 += BK) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            As[lk + q][lr] = ra[q];
            Ws[lk + q][lr] = rw[q];
            if (SWIGLU) W3s[lk + q][lr] = rw3[q];
        }
        __syncthreads();
        request(k0 + BK);
#pragma unroll
        for (int kk = 0; kk < BK; ++kk) {
            float av[4], wv[4], w3v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) av[i] = As[kk][ty * 4 + i];
#pragma unroll
            for (int j = 0; j < 4; ++j) { wv[j] = Ws[kk][tx * 4 + j]; if (SWIGLU) w3v[j] = W3s[kk][tx * 4 + j]; }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    acc[i][j] += av[i] * wv[j];
                    if (SWIGLU) acc3[i][j] += av[i] * w3v[j];
                }
        }
        __syncthreads();
    }
    if (SEGS && k_end < a.K) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                tot[i][j] += acc[i][j]; acc[i][j] = 0.f;
                if (SWIGLU) { tot3[i][j] += acc3[i][j]; acc3[i][j] = 0.f; }
            }
    }
    }
    if (SEGS) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) { acc[i][j] = tot[i][j] + acc[i][j]; acc3[i][j] = tot3[i][j] + acc3[i][j]; }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        int r = row_begin + ty * 4 + i;
        if (r >= row_end) continue;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            int c = col0 + tx * 4 + j;
            if (c >= a.N) continue;
            int64_t o = (int64_t)r * a.ldc + c;
            float v = acc[i][j];
            if (SWIGLU) {
                float s = v / (1.0f + expf(-v));
                ((T*)a.C)[o] = from_f32<T>(s * acc3[i][j]);
            } else if (a.epilogue == EPI_ADD_F32) ((float*)a.C)[o] += v;
            else ((float*)a.C)[o] = v;
        }
    }
}

// The same product for problems that 64x64 tiles would run on a handful of compute units, where the matrix cores do not take them
// (bf16 in the plain-kernel mode or onto outputs off 16 bytes, f32 rows not of whole 16 bytes: gemm_f32_kernel takes the others): 8x32
// tiles, one output per thread, the contraction in steps of 256 whose elements are requested a step ahead.  What bounds such a product is
// latency: 35-48 us per launch as 16-wide steps on one to sixteen workgroups (8 rows, 256 to 1024 columns,
// K = 256 to 1024), 5-11 us so.  Weights may be panels (a bf16 layer of 5 rows, d = 4096, whose output is off 16 bytes: 225 us, and
// 1207 where panels left it to the 64x64 tiles).  Every output is the same sum as there.
constexpr int F32_TILE = 16, F32_PIECES = 16;               // rows and columns of a tile; pieces of 16 k requested at once
constexpr int F32_NORM_K = 16 * F32_PIECES, F32_ROPE_K = 2048;      // longest rows that are normalised and rotated inside (see gemm_small_fuses)
// Tiles (of one weight matrix) up to which four wavefronts share one, K over 256: 0.42 to 0.91 of one wavefront's time up to 512
// tiles, 1.01 to 1.16 of it from 1008 to 2016.
constexpr int F32_SEGMENT_TILES = 512;
constexpr int SMALL_BM = 8, SMALL_BN = 32, SMALL_BK = 256, SMALL_LK = SMALL_BK / 128;
template <typename T>
__device__ inline float4 load4_guarded(const T* __restrict__ p, int left, bool vec) {     // zeros past the `left` elements of the row
    float v[4] = {0.f, 0.f, 0.f, 0.f};
    if (vec && left >= 4) {
        alignas(4 * sizeof(T)) T e[4];
        if constexpr (sizeof(T) == 2) *(uint2*)e = *(const uint2*)p;
        else *(uint4*)e = *(const uint4*)p;
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = to_f32<T>(e[q]);
    } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) if (q < left) v[q] = to_f32<T>(p[q]);
    }
    return make_float4(v[0], v[1], v[2], v[3]);
}
template <typename T, bool SWIGLU, bool PANELS>
__global__ void __launch_bounds__(256)
gemm_small_kernel(GemmArgs a, int vec) {
    constexpr int PITCH = SMALL_BK + 4, WQ = SMALL_BN / 8;      // weight rows per thread and 128 columns of a step
    __shared__ __attribute__((aligned(16))) float As[SMALL_BM][PITCH];
    __shared__ __attribute__((aligned(16))) float Ws[SWIGLU ? 2 : 1][SMALL_BN][PITCH];
    int row_begin = blockIdx.y * SMALL_BM, row_end = a.M, group = 0;
    if (a.group_offsets) {
        int tiles = 0;
        bool found = false;
        for (int g = 0; g < a.n_groups; ++g) {
            const int b0 = a.group_offsets[g], b1 = a.group_offsets[g + 1], nt = (b1 - b0 + SMALL_BM - 1) / SMALL_BM;
            if (!found && (int)blockIdx.y < tiles + nt) {
                group = g; row_begin = b0 + ((int)blockIdx.y - tiles) * SMALL_BM; row_end = b1; found = true;
            }
            tiles += nt;
        }
        if (!found) return;
    }
    const T* A = (const T*)a.A;
    const T* W[2] = {(const T*)a.W + (int64_t)group * a.w_group_stride,
                     SWIGLU ? (const T*)a.W3 + (int64_t)group * a.w_group_stride : nullptr};
    const int col0 = blockIdx.x * SMALL_BN, tid = threadIdx.x;
    // loader: thread takes 4 elements at k = 4 (tid % 32) + 128 j of activation row tid / 32 and of weight rows
    // tid / 32 + 8 q
    const int lk = (tid & 31) * 4, lr = tid >> 5;
    const bool a_on = row_begin + lr < row_end;
    const T* arow = A + (a_on ? (int64_t)(a.a_rows ? a.a_rows[row_begin + lr] : row_begin + lr) * a.lda : 0);
    float4 ra[SMALL_LK], rw[SWIGLU ? 2 : 1][WQ][SMALL_LK];
    auto request = [&](int k0) {
        const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int j = 0; j < SMALL_LK; ++j) {
            const int k = k0 + lk + 128 * j;
            ra[j] = a_on ? load4_guarded<T>(arow + k, a.K - k, vec) : z;
#pragma unroll
            for (int m = 0; m < (SWIGLU ? 2 : 1); ++m)
#pragma unroll
                for (int q = 0; q < WQ; ++q) {
                    const int n = col0 + lr + 8 * q;
                    rw[m][q][j] = n < a.N ? load4_guarded<T>(W[m] + weight_elem(n, k, a.K, PANELS ? a.w_panel : 0), a.K - k, vec) : z;
                }
        }
    };
    const int n_in = tid & 31, m_in = tid >> 5;
    constexpr bool SEGS = std::is_same<T, float>::value;
    float acc = 0.f, acc3 = 0.f, tot = 0.f, tot3 = 0.f;
    const int seg = f32_segment(a.K);
    int fold = seg;
    request(0);
    for (int k0 = 0; k0 < a.K; k0 += SMALL_BK) {
        __syncthreads();
#pragma unroll
        for (int j = 0; j < SMALL_LK; ++j) {
            *(float4*)&As[lr][lk + 128 * j] = ra[j];
#pragma unroll
            for (int m = 0; m < (SWIGLU ? 2 : 1); ++m)
#pragma unroll
                for (int q = 0; q < WQ; ++q) *(float4*)&Ws[m][lr + 8 * q][lk + 128 * j] = rw[m][q][j];
        }
        __syncthreads();
        if (k0 + SMALL_BK < a.K) request(k0 + SMALL_BK);
        auto four = [&](int k) __attribute__((always_inline)) {
            const float4 x = *(const float4*)&As[m_in][k], w = *(const float4*)&Ws[0][n_in][k];
            acc = fmaf(x.x, w.x, acc); acc = fmaf(x.y, w.y, acc); acc = fmaf(x.z, w.z, acc); acc = fmaf(x.w, w.w, acc);
            if (SWIGLU) {
                const float4 u = *(const float4*)&Ws[SWIGLU ? 1 : 0][n_in][k];
                acc3 = fmaf(x.x, u.x, acc3); acc3 = fmaf(x.y, u.y, acc3); acc3 = fmaf(x.z, u.z, acc3); acc3 = fmaf(x.w, u.w, acc3);
            }
        };
        auto behind = [&](int k) {                           // a segment's sum is whole behind its last k
            if (SEGS && k0 + k == fold) {
                fold += seg;
                tot += acc; acc = 0.f;
                if (SWIGLU) { tot3 += acc3; acc3 = 0.f; }
            }
        };
        if (!SEGS || seg % SMALL_BK == 0) {
#pragma unroll 8
            for (int k = 0; k < SMALL_BK; k += 4) four(k);
            behind(SMALL_BK);
        } else if (seg % 64 == 0) {
            for (int k1 = 0; k1 < SMALL_BK; k1 += 64) {
#pragma unroll
                for (int k = 0; k < 64; k += 4) four(k1 + k);
                behind(k1 + 64);
            }
        } else {
#pragma unroll 2
            for (int k1 = 0; k1 < SMALL_BK; k1 += 16) {
#pragma unroll
                for (int k = 0; k < 16; k += 4) four(k1 + k);
                behind(k1 + 16);
            }
        }
    }
    if (SEGS) { acc = tot + acc; acc3 = tot3 + acc3; }
    const int r = row_begin + m_in, c = col0 + n_in;
    if (r >= row_end || c >= a.N) return;
    const int64_t o = (int64_t)r * a.ldc + c;
    if (SWIGLU) ((T*)a.C)[o] = from_f32<T>(acc / (1.0f + expf(-acc)) * acc3);
    else if (a.epilogue == EPI_ADD_F32) ((float*)a.C)[o] += acc;
    else ((float*)a.C)[o] = acc;
}

// f32 products of few tiles on the matrix cores: a tile is 16 rows x 16 columns (of each of two weight matrices one).  What bounds such a product is
// latency (a round of the 256-wide two-layer model is 29 of them, 4 to 20 rows): round trips to memory and the chain of matrix
// instructions (16 cycles for four k).  So every operand piece goes straight from memory to registers, up to 256 k in flight at once,
// and the four segments of a sum go to four wavefronts, which meet once, in LDS.  A lane's four
// consecutive k are turned (permlane swaps) so that v_mfma_f32_16x16x4_f32 takes them in ascending order: it is four
// chained fused multiply-adds, so every output has the bits of the VALU kernels' sums, whatever the row count chooses.
// Where the tiles alone fill the chip four wavefronts only add traffic and one makes all segments (SEGS = 1).
// Round of four sequences and four candidates: 433 us with 8x32 VALU tiles, 376 with one wavefront a tile, 329 here (the error of its
// probabilities against 64 bits: 2.6e-7 with one chain a sum, 1.6e-7 with four).
// A product alone, us, one wavefront and one chain / here, from 229 sizes of 1 to 512 rows (0.42 to 1.04 of the time, mean 0.70):
//   K = 256    256 columns, 4 rows 4.4 / 3.4, 128 rows 4.7 / 3.7     8064 columns, 4 rows 5.7 / 4.6, 64 rows 12.0 / 10.9
//   K = 1024  1024 columns, 1 row 10.7 / 6.4                         8064 columns, 4 rows 14.8 / 10.3
//   K = 2048   256 columns, 16 rows 21.0 / 12.5                      4096 columns, 20 rows 25.0 / 20.0
//   K = 8192   256 columns, 4 rows 71.4 / 31.9
// (SEGS = 1 holds 8 pieces at once: 16 took 219 registers and up to 1.17 of the time, 19.9 -> 23.3 for 64 rows, 8064 columns, K = 512.)
//
// NORM: the rows are the residual stream and the product takes rmsnorm(row) * norm_g, with the row's squares summed in the
// order of combine_norm_vec_kernel (same bits); EPI_ROPE_KV: a wavefront makes 16 rotary pairs (the second weight row of a
// pair is where SwiGLU has the up row), rotates and appends as rope_kv_kernel does.  4 rows, K = 256, us: norm 2.6,
// QKV 4.6 and a rotary kernel as launches of their own, 8.4 as one; gate/up 6.6 behind its norm, 7.3 with it.
__device__ inline void turn4(f32x4_t& v) {        // element e of lane group q (16 lanes each) <-> element q of group e
    auto swap = [](float& x, float& y, auto by32) {
        auto r = decltype(by32)::value ? __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false)
                                       : __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
        x = __uint_as_float(r[0]);
        y = __uint_as_float(r[1]);
    };
    float e0 = v[0], e1 = v[1], e2 = v[2], e3 = v[3];
    swap(e0, e2, std::true_type()); swap(e1, e3, std::true_type());
    swap(e0, e1, std::false_type()); swap(e2, e3, std::false_type());
    v = f32x4_t{e0, e1, e2, e3};
}
template <typename F, int... I>
__device__ __forceinline__ void static_for_p_impl(F&& f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, typename F>
__device__ __forceinline__ void static_for_p(F&& f) { static_for_p_impl(f, std::make_integer_sequence<int, N>{}); }
template <int EPI, bool NORM, int P, int SEGS>
__global__ void __launch_bounds__((EPI == EPI_SWIGLU_T || EPI == EPI_ROPE_KV ? 128 : 64) * SEGS)
gemm_f32_kernel(GemmArgs a) {
    constexpr bool SWIGLU = EPI == EPI_SWIGLU_T, ROPE = EPI == EPI_ROPE_KV, DUAL = SWIGLU || ROPE;
    constexpr int TILE = F32_TILE;
    constexpr int NE = DUAL ? 2 : 4;                             // outputs that a lane finishes
    __shared__ f32x4_t part[DUAL ? 2 : 1][SEGS][64];
    __shared__ __attribute__((aligned(16))) float squares[NORM ? TILE : 1][NORM ? 2 * F32_PIECES + 4 : 1];
    int row_begin = blockIdx.y * TILE, row_end = a.M, group = 0;
    if (a.group_offsets) {
        int tiles = 0;
        bool found = false;
        for (int g = 0; g < a.n_groups; ++g) {
            const int b0 = a.group_offsets[g], b1 = a.group_offsets[g + 1], nt = (b1 - b0 + TILE - 1) / TILE;
            if (!found && (int)blockIdx.y < tiles + nt) {
                group = g; row_begin = b0 + ((int)blockIdx.y - tiles) * TILE; row_end = b1; found = true;
            }
            tiles += nt;
        }
        if (!found) return;
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, w = DUAL ? wave & 1 : 0, s = DUAL ? wave >> 1 : wave;
    const int fr = lane & 15, kq = (lane >> 4) * 4;
    const int seg = f32_segment(a.K);
    const int k_beg = SEGS > 1 ? min(s * seg, a.K) : 0, k_end = SEGS > 1 ? min(k_beg + seg, a.K) : a.K;     // this wavefront's segment, or all
    const int col0 = blockIdx.x * TILE;
    // ROPE: columns are rotary pairs, `half` of them a head
    const int half = ROPE ? a.rope.geom.head_dim >> 1 : 0, n_cols = ROPE ? a.N >> 1 : a.N;
    // operand rows of this lane (rows and columns past the last one repeat it and are not stored)
    const int ar = min(row_begin + fr, row_end - 1), n = min(col0 + fr, n_cols - 1);
    // the outputs that this lane finishes, row r and columns c..c+NE-1, and what that needs from memory, requested in front
    // of the operands (loads land in order)
    const int r = row_begin + fr, c = col0 + kq + w * NE;
    float old[NE] = {};
    float2 cs[NE];
    int pos = -1, page = 0;
    if (EPI == EPI_STORE_F32 && a.epilogue == EPI_ADD_F32) {
#pragma unroll
        for (int e = 0; e < NE; ++e) old[e] = ((const float*)a.C)[(int64_t)ar * a.ldc + min(c + e, n_cols - 1)];
    }
    if (ROPE) {
        pos = a.rope.row_pos[ar];
#pragma unroll
        for (int e = 0; e < NE; ++e) cs[e] = a.rope.cs[(int64_t)ar * half + (c + e) % half];
    }
    const float* arow = (const float*)a.A + (int64_t)(a.a_rows ? a.a_rows[ar] : ar) * a.lda;
    const float* wrow = (SWIGLU && w ? (const float*)a.W3 : (const float*)a.W) + (int64_t)group * a.w_group_stride +
                        (int64_t)(ROPE ? n / half * 2 * half + n % half + w * half : n) * a.K;
    // Chunks of 16 P: a whole one takes one address per operand and neither clamps nor branches (with them the dozen
    // instructions more per piece outweigh its four MFMAs: 3 % of a round of four sequences).
    f32x4_t fa[P], fw[P], fg[P];
    const float *pa = arow + kq, *pw = wrow + kq, *pg = (const float*)a.norm_g + kq;
    auto request = [&](auto whole_c, int k0, int p) __attribute__((always_inline)) {
        const f32x4_t z = {0.f, 0.f, 0.f, 0.f};
        const bool in = decltype(whole_c)::value || k0 + 16 * p + kq < k_end;        // pieces past the end become zeros
        f32x4_t x = z, g = z, wv = z;
        if (in) {
            x = *(const f32x4_t*)(pa + k0 + 16 * p);
            if (NORM) g = *(const f32x4_t*)(pg + k0 + 16 * p);
            wv = *(const f32x4_t*)(pw + k0 + 16 * p);
        }
        fa[p] = x; fw[p] = wv;
        if (NORM) fg[p] = g;
    };
    using Yes = std::true_type;
    using No = std::false_type;
    if (k_end - k_beg >= 16 * P) static_for_p<P>([&](auto p_c) __attribute__((always_inline)) { request(Yes(), k_beg, decltype(p_c)::value); });
    else static_for_p<P>([&](auto p_c) __attribute__((always_inline)) { request(No(), k_beg, decltype(p_c)::value); });
    if (ROPE) {
        const int lp = pos / a.rope.geom.page_tokens;
        if (pos < 0 || lp >= a.rope.geom.pages_per_seq) pos = -1;
        page = a.rope.page_table[(int64_t)(ar / a.rope.n_new) * a.rope.geom.pages_per_seq + (pos < 0 ? 0 : lp)];
    }
    const f32x4_t z = {0.f, 0.f, 0.f, 0.f};
    float rs = 1.f;
    if constexpr (NORM) {
        // A slot is 8 consecutive elements (a thread of the norm kernel), its squares one chain that the even lane groups begin and the
        // odd ones finish (see squares8); the row's at most 32 slots are half a wavefront there, summed as its shuffles do: slots 16
        // apart, then 8, ... 1.
        static_assert(!NORM || 4 * P == F32_PIECES, "a row's pieces lie in the four wavefronts' first chunks");
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const f32x4_t& x = fa[p];                             // (zeros past the segment)
            float t = fmaf(x[0], x[0], x[1] * x[1]);
            t = fmaf(x[3], x[3], fmaf(x[2], x[2], t));
            t = __shfl_xor(t, 16, WAVE);
            t = fmaf(x[3], x[3], fmaf(x[2], x[2], fmaf(x[1], x[1], fmaf(x[0], x[0], t))));
            const int slot = (k_beg + 16 * p) / 8 + (lane >> 5);
            if (w == 0 && (lane & 16) && slot < 2 * F32_PIECES && k_beg + 16 * p < k_end) squares[fr][slot] = t;
        }
        if (threadIdx.x < TILE) {                                 // slots past the row
            for (int q = (a.K + 15) / 16 * 2; q < 2 * F32_PIECES; ++q) squares[threadIdx.x][q] = 0.f;
        }
        __syncthreads();
        float v[2 * F32_PIECES];
#pragma unroll
        for (int q = 0; q < 2 * F32_PIECES; q += 4) {
            const f32x4_t x = *(const f32x4_t*)&squares[fr][q];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[q + e] = x[e];
        }
#pragma unroll
        for (int o = F32_PIECES; o > 0; o >>= 1)
#pragma unroll
            for (int q = 0; q < o; ++q) v[q] += v[q + o];
        rs = 1.0f / sqrtf(v[0] / (float)a.K + a.norm_eps);
    }
    f32x4_t acc = z, tot = z;
    int fold = seg;
    // the chunk in the registers, with the requests of the next one (NEXT: 0 none, 1 whole, 2 the rest) as they fall free
    auto chunk = [&](auto next_c, int k0) __attribute__((always_inline)) {
        constexpr int NEXT = decltype(next_c)::value;
        static_for_p<P>([&](auto p_c) __attribute__((always_inline)) {
            constexpr int p = decltype(p_c)::value;
            if (NEXT == 0 && k0 + 16 * p >= k_end) return;
            if (SEGS == 1 && k0 + 16 * p == fold) {
                fold += seg;
                tot += acc;
                acc = z;
            }
            f32x4_t av = fa[p], wv = fw[p];
            if (NORM) {
#pragma unroll
                for (int e = 0; e < 4; ++e) av[e] = av[e] * rs * fg[p][e];
            }
            turn4(av);
            turn4(wv);
            if constexpr (NEXT == 1) request(Yes(), k0 + 16 * P, p);
            else if constexpr (NEXT == 2) request(No(), k0 + 16 * P, p);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[e], av[e], acc, 0, 0, 0);
        });
    };
    int k0 = k_beg;
    for (; k0 + 32 * P <= k_end; k0 += 16 * P) chunk(std::integral_constant<int, 1>(), k0);
    if (k0 + 16 * P < k_end) { chunk(std::integral_constant<int, 2>(), k0); k0 += 16 * P; }
    chunk(std::integral_constant<int, 0>(), k0);
    if (SEGS == 1) acc = tot + acc;
    float v0[NE], v1[NE];
    if constexpr (SEGS > 1 || DUAL) {
        part[w][s][lane] = acc;
        __syncthreads();
        if (s != 0) return;                               // the first segment's wavefronts add them (DUAL: each finishes half of the columns)
        auto sum = [&](int m, int e) {
            float v = part[m][0][lane][e];
#pragma unroll
            for (int q = 1; q < SEGS; ++q) v += part[m][q][lane][e];
            return v;
        };
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            v0[e] = sum(0, DUAL ? w * NE + e : e);
            if constexpr (DUAL) v1[e] = sum(1, w * NE + e);
        }
    } else {
#pragma unroll
        for (int e = 0; e < NE; ++e) v0[e] = acc[e];
    }
    if (r >= row_end) return;
#pragma unroll
    for (int e = 0; e < NE; ++e) {
        if (c + e >= n_cols) break;
        if constexpr (ROPE) {
            const RopeKvArgs& rp = a.rope;
            const int hd = (c + e) / half, i = (c + e) % half, Hq = rp.n_q_heads, Hkv = rp.geom.n_kv_heads;
            float lo = v0[e], hi = v1[e];
            if (hd < Hq + Hkv) {
                const float ra = lo * cs[e].x - hi * cs[e].y, rb = hi * cs[e].x + lo * cs[e].y;
                lo = ra; hi = rb;
            }
            float* kv = (float*)rp.kv_layer;
            if (hd < Hq) {
                float* dst = (float*)rp.q_out + ((int64_t)r * Hq + hd) * 2 * half;
                dst[i] = lo; dst[i + half] = hi;
            } else if (pos >= 0) {
                const int slot = pos % rp.geom.page_tokens;
                if (hd < Hq + Hkv) {
                    float* dst = kv + rp.geom.k_off(page, hd - Hq, slot);
                    dst[i] = lo; dst[i + half] = hi;
                } else {
                    kv[rp.geom.v_off(page, hd - Hq - Hkv, slot, i)] = lo;
                    kv[rp.geom.v_off(page, hd - Hq - Hkv, slot, i + half)] = hi;
                }
            }
        } else {
            float* C = (float*)a.C + (int64_t)r * a.ldc + c + e;
            if constexpr (SWIGLU) *C = v0[e] / (1.0f + expf(-v0[e])) * v1[e];
            else *C = a.epilogue == EPI_ADD_F32 ? old[e] + v0[e] : v0[e];
        }
    }
}

// 64x64 tiles on fewer than half the compute units: small tiles (4 to 8 times the reads of a weight, from L2)
static bool small_tiles(const GemmArgs& a) {
    const int rows = a.group_offsets ? a.m_upper : a.M;
    return (int64_t)((rows + 63) / 64) * ((a.N + 63) / 64) < 128;
}
// Rotation inside pays at every size measured (a launch less): layer of 20 rows, us, as a launch of its own / inside, K = 512 62.9 / 60.9,
// 1024 105 / 101, 2048 535 / 536, of one row 515 / 508.  The norm inside pays only where a row's squares come from the pieces that
// the product holds anyway, up to 256 k: every column tile sums them again, and behind that each further chunk is
// a round trip to memory in front of the product.  Layer of 1 / 20 / 80 rows, norm as a launch / inside (from 512 on with those trips;
// measured with one wavefront a tile, and with four the trips weigh more):
//   K = 128   32.2 / 35.4 / 36.0                          29.9 / 32.6 / 33.1
//   K = 256   39.9 / 44.5 / 48.0                          38.2 / 42.0 / 46.1
//   K = 512   54.0 / 60.9 / 73.0                          57.3 / 63.1 / 83.3
//   K = 768   72.8 / 83.0 / 106                           84.2 / 92.6 / 128
//   K = 1024  87.9 / 101 / 292                            103 / 116 / 300
//   K = 2048  508 / 536 / 831                             529 / 550 / 842
// Verify of a four-layer model, 1024 wide, 1 and 20 rows: 476 -> 415 and 521 -> 453 us with the line here and not at 2048.
bool gemm_small_fuses(int M, int N, int K, int dtype) {
    GemmArgs a{};
    a.M = M; a.N = N;
    return dtype == SPEC_F32 && K % 8 == 0 && K <= F32_ROPE_K && small_tiles(a);
}
bool gemm_small_norms(int K) { return K <= F32_NORM_K; }

hipError_t launch_gemm_simple(const GemmArgs& a, int dtype, hipStream_t st, bool plain) {
    int rows = a.group_offsets ? a.m_upper : a.M;
    if (rows <= 0 || a.N <= 0) return hipSuccess;
    const bool swiglu = a.epilogue == EPI_SWIGLU_T;
    const bool rope = a.epilogue == EPI_ROPE_KV;
    if (small_tiles(a)) {
        const size_t es = dtype == SPEC_F32 ? 4 : 2;
        const uintptr_t base = (uintptr_t)a.A | (uintptr_t)a.W | (swiglu ? (uintptr_t)a.W3 : 0) | (uintptr_t)(a.w_group_stride * es) | (uintptr_t)a.norm_g;
        const int vec = base % (4 * es) == 0 && a.lda % 4 == 0 && a.K % 4 == 0;
        if ((rope || a.norm_g) && (dtype != SPEC_F32 || !vec || a.group_offsets || plain)) return hipErrorInvalidValue;
        if (rope && a.N % a.rope.geom.head_dim != 0) return hipErrorInvalidValue;
        if (a.norm_g && (a.K % 8 != 0 || a.K > F32_NORM_K || a.epilogue == EPI_ADD_F32)) return hipErrorInvalidValue;
        if (dtype == SPEC_F32 && vec && !plain) {
            const int cols = rope ? a.N / 2 : a.N;
            dim3 grid((cols + F32_TILE - 1) / F32_TILE, (rows + F32_TILE - 1) / F32_TILE + (a.group_offsets ? a.n_groups : 0));
            // (EPI_STORE_F32 stores or adds as a.epilogue says)
            // A wavefront per segment and tile, with all pieces of a row of up to 256 k in flight; one for all segments where the tiles alone
            // fill the chip (figures at F32_SEGMENT_TILES).
            const bool all = a.K > 256 && (int64_t)grid.x * grid.y * (rope || swiglu ? 2 : 1) > F32_SEGMENT_TILES;
            auto pick = [&](auto p_c, auto segs_c) {
                constexpr int P = decltype(p_c)::value, SEGS = decltype(segs_c)::value;
                return rope ? gemm_f32_kernel<EPI_ROPE_KV, false, P, SEGS> : swiglu ? gemm_f32_kernel<EPI_SWIGLU_T, false, P, SEGS>
                                                                                   : gemm_f32_kernel<EPI_STORE_F32, false, P, SEGS>;
            };
            using C1 = std::integral_constant<int, 1>;
            using C4 = std::integral_constant<int, 4>;
            using CP = std::integral_constant<int, F32_PIECES>;
            auto kern = a.norm_g ? (rope ? gemm_f32_kernel<EPI_ROPE_KV, true, 4, 4> : swiglu ? gemm_f32_kernel<EPI_SWIGLU_T, true, 4, 4>
                                                                                              : gemm_f32_kernel<EPI_STORE_F32, true, 4, 4>)
                        : a.K <= 256 ? pick(C4(), C4()) : all ? pick(std::integral_constant<int, F32_PIECES / 2>(), C1()) : pick(CP(), C4());
            hipLaunchKernelGGL(kern, grid, dim3((rope || swiglu ? 128 : 64) * (all ? 1 : 4)), 0, st, a);
            return hipGetLastError();
        }
        dim3 sgrid((a.N + SMALL_BN - 1) / SMALL_BN, (rows + SMALL_BM - 1) / SMALL_BM + (a.group_offsets ? a.n_groups : 0));
        DISPATCH_DTYPE(dtype, {
            if (a.w_panel) {
                if constexpr (sizeof(T) == 2) {
                    if (swiglu) hipLaunchKernelGGL((gemm_small_kernel<T, true, true>), sgrid, dim3(256), 0, st, a, vec);
                    else hipLaunchKernelGGL((gemm_small_kernel<T, false, true>), sgrid, dim3(256), 0, st, a, vec);
                } else return hipErrorInvalidValue;
            } else if (swiglu) hipLaunchKernelGGL((gemm_small_kernel<T, true, false>), sgrid, dim3(256), 0, st, a, vec);
            else hipLaunchKernelGGL((gemm_small_kernel<T, false, false>), sgrid, dim3(256), 0, st, a, vec);
        });
        return hipGetLastError();
    }
    if (rope || a.norm_g) return hipErrorInvalidValue;
    int tiles_m = (rows + 63) / 64 + (a.group_offsets ? a.n_groups : 0);
    dim3 grid((a.N + 63) / 64, tiles_m);
    bool sw = a.epilogue == EPI_SWIGLU_T;
    DISPATCH_DTYPE(dtype, {
        if (a.w_panel) {
            if constexpr (sizeof(T) == 2) {
                if (sw) hipLaunchKernelGGL((gemm_simple_kernel<T, true, true>), grid, dim3(256), 0, st, a);
                else hipLaunchKernelGGL((gemm_simple_kernel<T, false, true>), grid, dim3(256), 0, st, a);
            } else return hipErrorInvalidValue;
        } else if (sw) hipLaunchKernelGGL((gemm_simple_kernel<T, true, false>), grid, dim3(256), 0, st, a);
        else hipLaunchKernelGGL((gemm_simple_kernel<T, false, false>), grid, dim3(256), 0, st, a);
    });
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// Rows -> panels of a weight matrix, in place (see common.h): one workgroup holds a panel, at most 256 KB, in registers
// between its reads and its writes.
// ---------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(1024)
weight_panels_kernel(uint4* __restrict__ W, int K, int log2) {
    constexpr int CHUNKS = 8 * PANEL_MAX_K / 8 / 1024;
    const int n = (K >> 3) << log2;                      // 16-byte chunks of a panel
    uint4* panel = W + (int64_t)blockIdx.x * n;
    uint4 v[CHUNKS];
#pragma unroll
    for (int q = 0; q < CHUNKS; ++q) {
        const int i = q * 1024 + (int)threadIdx.x;       // chunk i % 8 of row (i / 8) % R of slab i / (8 R)
        if (i < n) v[q] = panel[((i >> 3) & ((1 << log2) - 1)) * (K >> 3) + ((i >> (3 + log2)) << 3) + (i & 7)];
    }
    __syncthreads();                                     // (every read of the panel has landed before the first write)
#pragma unroll
    for (int q = 0; q < CHUNKS; ++q) {
        const int i = q * 1024 + (int)threadIdx.x;
        if (i < n) panel[i] = v[q];
    }
}
hipError_t launch_weight_panels(void* W, int64_t N, int64_t K, int log2, hipStream_t st) {
    if (N <= 0) return hipSuccess;
    if (log2 <= 0 || log2 != weight_panel_log2(N, K) || ((uintptr_t)W & 15)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(weight_panels_kernel, dim3((unsigned)(N >> log2)), dim3(1024), 0, st, (uint4*)W, (int)K, log2);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// Plain paged attention: one wavefront per (row, query head); keys in chunks of 64 with an online
// softmax; lanes own keys for the scores and output dimensions for the value sum.
// ---------------------------------------------------------------------------------------------
template <typename T>
__global__ void __launch_bounds__(64)
attention_simple_kernel(AttnArgs a) {
    __shared__ float qs[256];
    int t = blockIdx.x / a.n_q_heads, hq = blockIdx.x % a.n_q_heads;
    int lane = threadIdx.x;
    int dh = a.geom.head_dim;
    int g = a.n_q_heads / a.geom.n_kv_heads, kvh = hq / g;
    int b = t / a.n_new;
    int pos = a.row_pos[t];
    T* out = (T*)a.out + (int64_t)t * a.n_q_heads * dh + hq * dh;
    if (pos < 0) {
        for (int c = lane; c < dh; c += 64) out[c] = from_f32<T>(0.f);
        return;
    }
    const T* q = (const T*)a.q + (int64_t)t * a.n_q_heads * dh + hq * dh;
    for (int c = lane; c < dh; c += 64) qs[c] = to_f32<T>(q[c]);
    __syncthreads();
    const T* kv = (const T*)a.kv_layer;
    const int32_t* pt = a.page_table + b * a.geom.pages_per_seq;
    int n_keys = pos + 1;
    float m = -INFINITY, l = 0.f;
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    for (int c0 = 0; c0 < n_keys; c0 += 64) {
        int key = c0 + lane;
        float s = -INFINITY;
        const int page_l = key < n_keys ? pt[key / a.geom.page_tokens] : 0;       // page of this lane's key
        if (key < n_keys) {
            int64_t page = page_l;
            const T* kr = kv + a.geom.k_off(page, kvh, key % a.geom.page_tokens);
            float dot = 0.f;
            if (dh % 16 == 0) {       // 16 elements requested at a time; the sum runs over ascending dims as below
                for (int c = 0; c < dh; c += 16) {
                    alignas(16) T kv16[16];
#pragma unroll
                    for (int q = 0; q < (int)(16 * sizeof(T)) / 16; ++q) ((uint4*)kv16)[q] = ((const uint4*)(kr + c))[q];
#pragma unroll
                    for (int q = 0; q < 16; ++q) dot = fmaf(qs[c + q], to_f32<T>(kv16[q]), dot);
                }
            } else {
                for (int c = 0; c < dh; ++c) dot += qs[c] * to_f32<T>(kr[c]);
            }
            s = dot * a.scale;
        }
        float m_new = fmaxf(m, wave_max(s));
        float p = key < n_keys ? expf(s - m_new) : 0.f;
        float corr = expf(m - m_new);       // m = -inf on the first chunk -> 0
        l = l * corr + wave_sum(p);
#pragma unroll
        for (int dd = 0; dd < 4; ++dd) acc[dd] *= corr;
        // values are stored transposed, so four consecutive positions of a dimension are one 16- or 8-byte piece
        // (pages and sub-blocks are multiples of 16 tokens); positions past the last key have weight 0
        int nk = min(64, n_keys - c0);
#pragma unroll
        for (int dd = 0; dd < 4; ++dd) {
            const int c = min(lane + 64 * dd, dh - 1);           // (lanes past the last dimension store nothing)
            if (64 * dd >= dh) break;
#pragma unroll
            for (int j0 = 0; j0 < 64; j0 += 16) {                // 16 positions requested at a time
                if (j0 >= nk) break;
                alignas(16) T v[4][4];
#pragma unroll
                for (int g4 = 0; g4 < 4; ++g4) {
                    const int j = min(j0 + 4 * g4, (nk - 1) & ~3);
                    const int64_t page = __shfl(page_l, j, 64);
                    const T* vp = kv + a.geom.v_off(page, kvh, (c0 + j) % a.geom.page_tokens, c);
                    if constexpr (sizeof(T) == 2) *(uint2*)v[g4] = *(const uint2*)vp;
                    else *(uint4*)v[g4] = *(const uint4*)vp;
                }
#pragma unroll
                for (int q = 0; q < 16; ++q) {
                    const float pj = __shfl(p, j0 + q, 64);
                    if (j0 + q < nk) acc[dd] = fmaf(pj, to_f32<T>(v[q >> 2][q & 3]), acc[dd]);
                }
            }
        }
        m = m_new;
    }
    float inv = 1.0f / l;
#pragma unroll
    for (int dd = 0; dd < 4; ++dd) {
        int c = lane + 64 * dd;
        if (c < dh) out[c] = from_f32<T>(acc[dd] * inv);
    }
}
// The same for an f32 model of head_dim 64 or 128, every key and value piece of a chunk requested before its first score (a
// value's address does not wait for the softmax): the general kernel asks for 16 elements at a time, eight or
// more round trips a chunk, and latency is all that bounds a launch of few workgroups.  Same order of operations, same bits.
// 16 workgroups, 33 to 100 keys 8.9 -> 6.8 us.  The pieces take 255 registers (64 dims) or 413 (128): two wavefronts or one a SIMD
// where the general kernel has three, so with more workgroups than that occupancy counts for more.  us, 4 query heads, general kernel / this one:
//   workgroups                256          512          640          768          1024         1280          3072
//   64 dims, 100 keys      14.1 / 12.6  15.0 / 13.4  16.2 / 15.0  16.0 / 15.4  17.4 / 16.9  19.2 / 20.7   29.7 / 34.6
//            1000 keys     85.0 / 74.8  90.0 / 78.6  94.5 / 94.7  96.1 / 95.9   101 / 107    115 / 118     255 / 274
//   128 dims, 100 keys     21.8 / 15.6  24.2 / 18.9  26.2 / 22.8  25.0 / 25.8  29.4 / 30.3  31.1 / 47.2   54.4 / 75.2
//            1000 keys      156 / 100    165 / 125    184 / 159    175 / 169    212 / 206    242 / 321     528 / 530
// (16 query heads the same within 4 %; prefills of 4 x 257 and 16 x 1000 rows 47 / 48 and 1830 / 2056, 128 dims 85 / 98 and 3764 / 4282.)
constexpr int F32_ATTN_GRID_64 = 768, F32_ATTN_GRID_128 = 640;
template <int DH>
__global__ void __launch_bounds__(64)
attention_f32_kernel(AttnArgs a) {
    constexpr int NK = DH / 4, ND = DH / 64;
    __shared__ float qs[DH];
    const int t = blockIdx.x / a.n_q_heads, hq = blockIdx.x % a.n_q_heads, lane = threadIdx.x;
    const int kvh = hq / (a.n_q_heads / a.geom.n_kv_heads), b = t / a.n_new;
    const int64_t row = ((int64_t)t * a.n_q_heads + hq) * DH;
    const float* q = (const float*)a.q + row;
    float* out = (float*)a.out + row;
    float qv[ND];
#pragma unroll
    for (int d = 0; d < ND; ++d) qv[d] = q[lane + 64 * d];
    const int pos = a.row_pos[t], n_keys = pos + 1;
    const float* kv = (const float*)a.kv_layer;
    const int32_t* pt = a.page_table + (int64_t)b * a.geom.pages_per_seq;
    const int pages = a.geom.page_tokens;
    int page_l = pt[min(lane / pages, a.geom.pages_per_seq - 1)];      // page of this lane's key of the first chunk
    if (pos < 0) {
#pragma unroll
        for (int d = 0; d < ND; ++d) out[lane + 64 * d] = 0.f;
        return;
    }
#pragma unroll
    for (int d = 0; d < ND; ++d) qs[lane + 64 * d] = qv[d];
    __syncthreads();
    float m = -INFINITY, l = 0.f, acc[ND] = {};
    for (int c0 = 0; c0 < n_keys; c0 += 64) {
        const int key = c0 + lane, nk = min(64, n_keys - c0), last = (nk - 1) & ~3;
        // (lanes past the last key repeat it; their weight is 0)
        const int kc = min(key, n_keys - 1);
        page_l = c0 > 0 ? pt[kc / pages] : __shfl(page_l, min(lane, nk - 1), 64);
        const float4* kr = (const float4*)(kv + a.geom.k_off(page_l, kvh, kc % pages));
        float4 kk[NK], vv[ND][16];
#pragma unroll
        for (int c = 0; c < NK; ++c) kk[c] = kr[c];
#pragma unroll
        for (int g = 0; g < 16; ++g) {
            const int j = min(4 * g, last);
            const int64_t page = __shfl(page_l, j, 64);
#pragma unroll
            for (int d = 0; d < ND; ++d)
                if (4 * g < nk) vv[d][g] = *(const float4*)(kv + a.geom.v_off(page, kvh, (c0 + j) % pages, lane + 64 * d));
        }
        float dot = 0.f;
#pragma unroll
        for (int c = 0; c < NK; ++c) {
            const float4 qq = *(const float4*)&qs[4 * c];
            dot = fmaf(qq.x, kk[c].x, dot); dot = fmaf(qq.y, kk[c].y, dot); dot = fmaf(qq.z, kk[c].z, dot); dot = fmaf(qq.w, kk[c].w, dot);
        }
        const float s = key < n_keys ? dot * a.scale : -INFINITY;
        const float m_new = fmaxf(m, wave_max(s));
        const float p = key < n_keys ? expf(s - m_new) : 0.f;
        const float corr = expf(m - m_new);       // m = -inf on the first chunk -> 0
        l = l * corr + wave_sum(p);
#pragma unroll
        for (int d = 0; d < ND; ++d) acc[d] *= corr;
#pragma unroll
        for (int g = 0; g < 16; ++g) {
            if (4 * g >= nk) break;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float pj = __shfl(p, 4 * g + e, 64);
#pragma unroll
                for (int d = 0; d < ND; ++d) {
                    const float ve = e == 0 ? vv[d][g].x : e == 1 ? vv[d][g].y : e == 2 ? vv[d][g].z : vv[d][g].w;
                    if (4 * g + e < nk) acc[d] = fmaf(pj, ve, acc[d]);
                }
            }
        }
        m = m_new;
    }
    const float inv = 1.0f / l;
#pragma unroll
    for (int d = 0; d < ND; ++d) out[lane + 64 * d] = acc[d] * inv;
}

hipError_t launch_attention_simple(const AttnArgs& a, int dtype, hipStream_t st, bool plain) {
    int T_ = a.B * a.n_new;
    if (T_ <= 0) return hipSuccess;
    // (values are read in pieces of four positions: pages of whole fours; 16-byte rows)
    const int chunked = a.geom.head_dim == 64 ? F32_ATTN_GRID_64 : a.geom.head_dim == 128 ? F32_ATTN_GRID_128 : 0;
    if (!plain && dtype == SPEC_F32 && (int64_t)T_ * a.n_q_heads <= chunked && a.geom.page_tokens % 4 == 0 && !((uintptr_t)a.kv_layer & 15)) {
        if (a.geom.head_dim == 64) hipLaunchKernelGGL(attention_f32_kernel<64>, dim3(T_ * a.n_q_heads), dim3(64), 0, st, a);
        else hipLaunchKernelGGL(attention_f32_kernel<128>, dim3(T_ * a.n_q_heads), dim3(64), 0, st, a);
        return hipGetLastError();
    }
    DISPATCH_DTYPE(dtype, hipLaunchKernelGGL(attention_simple_kernel<T>, dim3(T_ * a.n_q_heads), dim3(64),
                                             0, st, a));
    return hipGetLastError();
}

}  // namespace sv
