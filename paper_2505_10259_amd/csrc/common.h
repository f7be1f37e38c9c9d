// Internal declarations shared by the HIP sources of the specverify library (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/specverify.h"

namespace sv {

// ---- bf16 storage type ------------------------------------------------------------------
struct bf16 {
    uint16_t bits;
};

__host__ __device__ inline float bf16_to_f32(bf16 v) {
    union { uint32_t u; float f; } c;
    c.u = (uint32_t)v.bits << 16;
    return c.f;
}
// round to nearest even; NaN stays NaN
__host__ __device__ inline bf16 f32_to_bf16(float f) {
    union { uint32_t u; float f; } c;
    c.f = f;
    uint32_t u = c.u;
    bf16 r;
    if ((u & 0x7fffffffu) > 0x7f800000u) { r.bits = (uint16_t)((u >> 16) | 0x40u); return r; }
    u += 0x7fffu + ((u >> 16) & 1u);
    r.bits = (uint16_t)(u >> 16);
    return r;
}

template <typename T> __host__ __device__ inline float to_f32(T v);
template <> __host__ __device__ inline float to_f32<float>(float v) { return v; }
template <> __host__ __device__ inline float to_f32<bf16>(bf16 v) { return bf16_to_f32(v); }
template <typename T> __host__ __device__ inline T from_f32(float v);
template <> __host__ __device__ inline float from_f32<float>(float v) { return v; }
template <> __host__ __device__ inline bf16 from_f32<bf16>(float v) { return f32_to_bf16(v); }

constexpr int WAVE = 64;

// Sum and maximum over a wavefront, in every lane: pairs of lanes 32, 16, 8, 4, 2 and 1 apart (the order of a butterfly of shuffles, the
// same bits), without the trip through the LDS crossbar that a shuffle is (0.04 us each, six behind one another).
template <typename F>
__device__ inline float wave_reduce(float v, F f) {
    auto bits = [](float x) { return __float_as_uint(x); };
    auto w = __builtin_amdgcn_permlane32_swap(bits(v), bits(v), false, false);
    v = f(__uint_as_float(w[0]), __uint_as_float(w[1]));
    w = __builtin_amdgcn_permlane16_swap(bits(v), bits(v), false, false);
    v = f(__uint_as_float(w[0]), __uint_as_float(w[1]));
    v = f(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x128, 0xf, 0xf, false)));     // row_ror:8
    v = f(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x124, 0xf, 0xf, false)));     // row_ror:4
    v = f(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4e, 0xf, 0xf, false)));      // quad_perm 2,3,0,1
    return f(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xb1, 0xf, 0xf, false)));   // quad_perm 1,0,3,2
}
__device__ inline float wave_sum(float v) { return wave_reduce(v, [](float a, float b) { return a + b; }); }
__device__ inline float wave_max(float v) { return wave_reduce(v, [](float a, float b) { return fmaxf(a, b); }); }

// ---- KV page pool geometry -----------------------------------------------------------------
// One pool per (model, sub-batch).  A (layer, page, kv_head) block holds the page's tokens in
// sub-blocks of 32 (see sub_tokens); each sub-block is its keys followed by its values:
//   keys   [slot][dim]   -- a key row is contiguous (the contraction dimension of q.k)
//   values [dim][slot]   -- TRANSPOSED, so that consecutive positions of one dimension are
//                           contiguous (the contraction dimension of p.v): both MFMA operands of
//                           the attention kernel are then 16-byte pieces of memory rows.
// A sequence owns pages_per_seq logical pages listed in its page-table row.
struct KvGeom {
    int n_kv_heads, head_dim, page_tokens, pages_per_seq;
    int64_t n_pages;        // physical pages per layer
    __host__ __device__ int64_t layer_elems() const {
        return n_pages * (int64_t)n_kv_heads * 2 * page_tokens * head_dim;
    }
    __host__ __device__ int64_t block(int64_t page, int kvh) const {
        return (page * n_kv_heads + kvh) * 2 * (int64_t)page_tokens * head_dim;
    }
    // Inside a (page, kv head) block the tokens are cut into sub-blocks of 32 (the attention kernel's
    // key tile; the whole page if its size is not a multiple of 32), and each sub-block holds its keys
    // [slot][dim] followed by its values transposed [dim][slot]: one key tile of K and V is then one
    // contiguous run of 2 * 32 * head_dim elements in HBM.
    __host__ __device__ int sub_tokens() const { return page_tokens % 32 == 0 ? 32 : page_tokens; }
    __host__ __device__ int64_t sub_block(int64_t page, int kvh, int slot) const {
        return block(page, kvh) + (int64_t)(slot / sub_tokens()) * 2 * sub_tokens() * head_dim;
    }
    __host__ __device__ int64_t k_off(int64_t page, int kvh, int slot) const {
        return sub_block(page, kvh, slot) + (int64_t)(slot % sub_tokens()) * head_dim;
    }
    __host__ __device__ int64_t v_off(int64_t page, int kvh, int slot, int dim) const {
        return sub_block(page, kvh, slot) + (int64_t)sub_tokens() * head_dim + (int64_t)dim * sub_tokens() +
               slot % sub_tokens();
    }
};

// ---- GEMM problem description -------------------------------------------------------------
// C[M,N] (+)= A[M,K] * W[N,K]^T ; all row-major; optional row gather on A; optional grouping:
// rows are split into groups by `group_offsets` (device, [n_groups+1]) and group g uses weights
// W + g * w_group_stride (elements).
enum GemmEpilogue {
    EPI_STORE_F32 = 0,   // C float = acc
    EPI_ADD_F32 = 1,     // C float += acc           (residual accumulate; one writer per element)
    EPI_SWIGLU_T = 2,    // C (model dtype)[M, N] = silu(A W^T) * (A W3^T)   (W3 = second weight)
    EPI_ROPE_KV = 3      // QKV projection (bf16 MFMA kernel with head_dim 128, small f32 products): columns are
                         // [q heads | k heads | v heads]; q and k are rotated (pair (i, i + head_dim/2)) with the
                         // row's cos/sin table, q goes to rope.q_out, k and v to the row's KV page slot
};

struct RopeKvArgs {               // EPI_ROPE_KV: what rope_kv_kernel takes, minus the f32 qkv buffer
    const float2* cs;             // [M, head_dim / 2] (cos, sin) per row
    const int32_t* row_pos;       // [M] absolute position of each row (< 0: row inactive)
    const int32_t* page_table;    // [B, pages_per_seq]
    void* q_out;                  // [M, n_q_heads * head_dim] model dtype
    void* kv_layer;               // KV pool of this layer
    KvGeom geom;
    int n_new, n_q_heads;
};

struct GemmArgs {
    const void* A; int64_t lda;
    const int32_t* a_rows;          // nullable: A row of output row m is a_rows[m]
    const void* W; const void* W3;  // [N,K] each, ld = K
    void* C; int64_t ldc;
    int M, N, K;
    int epilogue;
    const int32_t* group_offsets;   // nullable
    int n_groups;
    int64_t w_group_stride;         // elements between consecutive groups' W (and W3)
    int w_panel;                    // log2 of the rows of a weight panel (see weight_panel_log2); 0: plain rows
    int m_upper;                    // grouped: upper bound on total rows (grid sizing)
    int m_expected;                 // grouped: expected rows per group if known (tile-height choice), else 0
    RopeKvArgs rope;                // EPI_ROPE_KV only
    const void* norm_g;             // nullable (small f32 products): A holds f32 rows x, the product takes rmsnorm(x) * norm_g
    float norm_eps;
    int force_max_rows, force_cols; // tests: tile height limit (multiple of 32, <= 256) and weight columns per tile (256, 128, 64 or 32,
                                    // SwiGLU 256 or 128); 0 = the launcher's choice
};

// ---- weight panels ---------------------------------------------------------------------------
// Resident bf16 matrices [N, K] are kept as panels of R = 2^log2 rows, each panel cut into slabs of 64 columns:
// [N/R][K/64][R][64].  A panel covers the same bytes as its rows, so the layout inside a blob does not move.  The GEMM's
// slab loads then take R x 128 B runs of HBM where plain rows give 128 B pieces a row pitch apart.  Panels of 8 are one 1 KB load
// of a wavefront; measured on grouped products with real blobs, us as plain rows / panels of 4 / of 8 / of 16 / of 32:
//   gate/up  K = 4096   80 rows an expert 328 / 293 / 303 / 325 / 322    224 rows 418 / 380 / 404 / 426 / 420
//            K = 6144   20 rows 484 / 486 / 466 / 479 / 482              224 rows 728 / 690 / 675 / 698 / 690
//   down     K = 14336  20 rows 155 / 141 / 138 / 138 / 140              80 rows 175 / 159 / 156 / 157 / 158
//            K = 16384  20 rows 305 / 270 / 263 / 260 / 263              224 rows 380 / 346 / 353 / 355 / 359
// so panels of 4 up to K = 4096 and of 8 above (with 224 rows of K = 16384 the 4 would be 2 % better).  Single matrices of other widths, time as
// panels over time as rows, 1 to 8192 rows: K = 256 to 1024 0.98-1.02 (one of 4.5 us 1.08), 2048 and 3072 0.95-1.02, 4096 0.86-1.03, 5120 0.92-0.98, 6144
// 0.84-1.02, 8192 0.94-1.02, 14336 0.94-1.03, 16384 0.82-1.02; from 2304 rows on the matrix cores bound it and the layout counts
// for nothing.  (Rotating the slabs of a panel by its position gave nothing.)
constexpr int PANEL_MAX_K = 16384;     // a panel is turned in the registers of one workgroup
__host__ __device__ inline int weight_panel_log2(int64_t N, int64_t K) {
    if (K % 64 != 0 || K > PANEL_MAX_K || N % 8 != 0) return 0;
    return K <= 4096 ? 2 : 3;
}
// element (n, k) of a matrix of row length K
__host__ __device__ inline int64_t weight_elem(int64_t n, int64_t k, int64_t K, int log2) {
    if (log2 == 0) return n * K + k;
    return (((n >> log2) * (K >> 6) + (k >> 6)) << (log2 + 6)) + ((n & ((1 << log2) - 1)) << 6) + (k & 63);
}
// rows -> panels, in place (bf16; 16-byte aligned; log2 from weight_panel_log2, not 0)
hipError_t launch_weight_panels(void* W, int64_t N, int64_t K, int log2, hipStream_t st);

// launchers (kernels_*.hip) -------------------------------------------------------------------
// plain: f32 products stay off the matrix cores (the plain-kernel mode; same bits)
hipError_t launch_gemm_simple(const GemmArgs& a, int dtype, hipStream_t st, bool plain = false);
hipError_t launch_gemm_mfma_bf16(const GemmArgs& a, hipStream_t st);   // gemm_mfma.hip
bool qkv_unfused_pays(int M, int N, int K);
// whether an f32 product of this size takes the small tiles and is to rotate (EPI_ROPE_KV), and whether it is to normalise its rows (norm_g) too
bool gemm_small_fuses(int M, int N, int K, int dtype);
bool gemm_small_norms(int K);

struct AttnArgs {
    const void* q;            // [T, Hq*dh] model dtype
    void* out;                // [T, Hq*dh] model dtype
    const void* kv_layer;     // pool base of this layer
    const int32_t* page_table;// [B, pages_per_seq]
    const int32_t* row_pos;   // [T] absolute position of each row (<0: row inactive)
    KvGeom geom;
    int B, n_new, n_q_heads;
    float scale;
};
// plain: the general kernel at any size (the plain-kernel mode; same bits)
hipError_t launch_attention_simple(const AttnArgs& a, int dtype, hipStream_t st, bool plain = false);
hipError_t launch_attention_mfma_bf16(const AttnArgs& a, hipStream_t st);   // attn_mfma.hip

hipError_t launch_fill_words(void* p, size_t n_words, uint32_t value, hipStream_t st);
// x[t] += w[t,0]*y[slot[t,0]] + w[t,1]*y[slot[t,1]]  (if y), then h[t] = rmsnorm(x[t]) * g (if g)
hipError_t launch_combine_norm(float* x, const float* y, const float* wts, const int32_t* slots,
                               const void* g, void* h, int T, int d, float eps, int dtype,
                               hipStream_t st);
// RMSNorm + router in one kernel (see kernels_basic.hip); norm_route_supported tells whether it applies
bool norm_route_supported(int d, int E);
// `forced` (nullable): [T, 2] expert ids to use instead of the top-2 (weights still from the logits);
// `row_pos` (nullable): rows with a negative position are inactive and get no experts (ids -1, weights 0)
hipError_t launch_norm_route(const float* x, const void* g, void* h, const void* wr, int32_t* ids, float* wts,
                             int T, int d, int E, float eps, const int32_t* forced, const int32_t* row_pos, int dtype,
                             hipStream_t st);
hipError_t launch_rope_kv(const float* qkv, const float2* cs, const int32_t* row_pos,
                          const int32_t* page_table, void* q_out, void* kv_layer, KvGeom geom,
                          int T, int n_new, int n_q_heads, int dtype, hipStream_t st);
// bf16, head_dim 128 (the MFMA path's buffer): the arithmetic of EPI_ROPE_KV on f32 projections
hipError_t launch_rope_kv_bf16(const float* qkv, const float2* cs, const int32_t* row_pos, const int32_t* page_table,
                               void* q_out, void* kv_layer, KvGeom geom, int T, int n_new, int n_q_heads, hipStream_t st);
hipError_t launch_router(const void* h, const void* wr, int32_t* ids, float* wts, int T, int d,
                         int E, const int32_t* forced, const int32_t* row_pos, int dtype, hipStream_t st);
// counting sort of the 2T (token, choice) pairs by expert: offsets[E+1], perm[2T] (sorted row ->
// token), slots[T,2] (token choice -> sorted row)
hipError_t launch_moe_sort(const int32_t* ids, int32_t* offsets, int32_t* perm, int32_t* slots,
                           int T, int E, hipStream_t st);
hipError_t launch_kv_import(const void* k_ctx, const void* v_ctx, void* kv_layer,
                            const int32_t* page_table, KvGeom geom, int B, int ctx_len, int dtype,
                            hipStream_t st);

// sequence-state kernels (kernels_state.hip)
struct SeqState {
    int32_t* tokens;     // [B, tok_cap] committed tokens (prompt included)
    int32_t* len;        // [B] committed length
    int32_t* n_new;      // [B] new tokens so far
    int32_t* max_new;    // [B]
    int tok_cap;
};
// Token and position of every row of a pass
struct RowSource {
    SeqState s;
    int kind;                                   // ROWS_*
    int embed;                                  // 1: the rows are embeddings of the tokens, 0: given by the caller
    const int32_t* draft_tokens; int k, step;   // candidates [B, k]; step of a draft pass (1-based)
    const int32_t* seq_of; const int32_t* pos0; int Q;   // prefill: blocks of Q rows
    enum { ROWS_VERIFY, ROWS_DRAFT, ROWS_PREFILL };
    __device__ void row(int t, int& pos, int& tok) const {
        if (kind == ROWS_VERIFY) {
            // rows of sequence b: [last committed token, candidate 1..k] at positions len-1 .. len-1+k
            // (Section 2.2: all candidates are scored by the target in one forward pass)
            const int b = t / (k + 1), i = t % (k + 1), len = s.len[b];
            pos = len - 1 + i;
            tok = !embed ? 0 : i == 0 ? s.tokens[(int64_t)b * s.tok_cap + len - 1] : draft_tokens[b * k + i - 1];
        } else if (kind == ROWS_DRAFT) {
            // Step 1 feeds TWO rows per sequence, the tokens at positions len-2 and len-1: after a round in which every
            // candidate was kept the draft cache lacks position len-2, otherwise that entry is recomputed to the
            // same value, so the cache always covers [0, len-1) before candidate 1 is produced.  Step i >= 2
            // feeds candidate i-1 at position len-2+i.
            if (step == 1) {
                const int b = t >> 1, len = s.len[b], at = len - 2 + (t & 1);
                pos = at >= 0 ? at : -1;
                tok = at >= 0 ? s.tokens[(int64_t)b * s.tok_cap + at] : 0;
            } else {
                pos = s.len[t] - 2 + step;
                tok = draft_tokens[t * k + step - 2];
            }
        } else {
            // block v carries positions pos0[v] .. pos0[v]+Q-1 of sequence seq_of[v]; only positions before the last
            // prompt token are active (the last token is fed by the first verify pass)
            const int v = t / Q, b = seq_of[v], at = pos0[v] + t % Q;
            const bool on = at < s.len[b] - 1;
            pos = on ? at : -1;
            tok = on ? s.tokens[(int64_t)b * s.tok_cap + at] : 0;
        }
    }
};
// rows: the embedding table, or the caller's rows (model dtype); fills x [T, d], row_pos [T] and cs [T, half]
hipError_t launch_rows_prep(const RowSource& src, const void* rows, float* x, int32_t* row_pos, float2* cs, int T, int d,
                            int vocab, int half, float theta, int dtype, hipStream_t st);
hipError_t launch_commit(SeqState s, const int32_t* draft_tokens, int k, const int32_t* n_acc,
                         const int32_t* next_tok, int64_t* hist, int64_t* committed, int B,
                         hipStream_t st);

// accept / sampling kernels (kernels_accept.hip)
struct AcceptArgs {
    const float* p_logits;   // [B, k+1, V]
    const float* q_logits;   // [B, k, V] or null (greedy)
    const int32_t* draft_tokens;  // [B, k]
    const float* u_accept;   // [B, k] or null -> philox
    const float* u_resample; // [B, k+1] or null -> philox
    float inv_tau;
    uint64_t seed; uint32_t round, seq_base;
    int B, k, V;
    int32_t* n_accepted; int32_t* next_token;
};
hipError_t launch_accept(const AcceptArgs& a, hipStream_t st);
// draft token choice from logits rows z[b] (row stride ld): greedy argmax or inverse-CDF sample
hipError_t launch_draft_pick(const float* z, int64_t ld, int V, int B, int mode, float inv_tau,
                             uint64_t seed, uint32_t round, uint32_t seq_base, int step /*1-based*/,
                             int32_t* draft_tokens, int k, hipStream_t st);
hipError_t launch_philox_uniforms(uint64_t seed, uint32_t round, uint32_t seq_base, int B, int k,
                                  float* out, hipStream_t st);

}  // namespace sv
