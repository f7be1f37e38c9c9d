// Sequence-state kernel: accepted tokens are committed to the sequences kept in HBM (the rows of each pass are built
// from them in rows_prep_kernel), so that the host never has to read results back inside the draft/verify loop.
#include "common.h"

namespace sv {

// Commit: append candidates 1..n and the target's token, clipped to the sequence's remaining quota
// (a round emits between 1 and k+1 tokens, Appendix A.1 "Generated Tokens").  The KV caches need no
// work: entries beyond the new length are simply overwritten by the next pass.
__global__ void commit_kernel(SeqState s, const int32_t* __restrict__ d, int k,
                              const int32_t* __restrict__ n_acc, const int32_t* __restrict__ next_tok,
                              unsigned long long* __restrict__ hist,
                              unsigned long long* __restrict__ committed, int B) {
    int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B) return;
    int remaining = s.max_new[b] - s.n_new[b];
    if (remaining <= 0) return;
    const int n = min(max(n_acc[b], 0), k);        // (what is read and counted below has room for k)
    int c = min(n + 1, remaining);
    int len = s.len[b];
    int32_t* toks = s.tokens + (int64_t)b * s.tok_cap;
    for (int j = 0; j < c; ++j) toks[len + j] = j < n ? d[b * k + j] : next_tok[b];
    s.len[b] = len + c;
    s.n_new[b] += c;
    atomicAdd(&hist[n], 1ull);
    atomicAdd(committed, (unsigned long long)c);
}
hipError_t launch_commit(SeqState s, const int32_t* draft_tokens, int k, const int32_t* n_acc,
                         const int32_t* next_tok, int64_t* hist, int64_t* committed, int B,
                         hipStream_t st) {
    if (B <= 0) return hipSuccess;
    hipLaunchKernelGGL(commit_kernel, dim3((B + 255) / 256), dim3(256), 0, st, s, draft_tokens, k, n_acc,
                       next_tok, (unsigned long long*)hist, (unsigned long long*)committed, B);
    return hipGetLastError();
}

}  // namespace sv
