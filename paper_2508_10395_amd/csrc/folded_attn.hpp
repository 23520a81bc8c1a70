// Host interface of the folded attention kernels (folded_attn.hip).
#pragma once
#include "folded_common.hpp"

namespace xq {

struct FoldProblem {
    int Hq, Hkv;                         // heads
    int dense;                           // bf16 rows
    int bits, group, nibbles;            // of the walk (8-bit caches: 4, 128, 1)
    int n_slabs_k, n_slabs_v, ng_v;      // slabs of 128 walked channels on either side, groups of the values' side
    int block;                           // per-channel cache: tokens per block (else 0); its walk has groups of 128
    int digits;                          // queries in base-32 digits (set by the plan)
    size_t query_bytes;                  // what the entry point's workspace query says for this call
};

hipError_t allow_large_lds(const void* kernel, int lds_bytes);
bool unpack_table_for(int bits, UnpackTable* t);

int fold_splits(int nb, int nrb, int n_slabs_v, int max_len, int per_cu);               // token splits of the weighted sums
size_t fold_workspace_bytes(const FoldProblem& f, int B, int max_len);
bool fold_fits(const FoldProblem& f, int B, int max_len, size_t bytes);
hipError_t run_folded_attn(const FoldProblem& f, const uint16_t* q, const FoldSource& kx, const FoldSource& vx, const FoldWeights& kw,
                           const FoldWeights& vw, int B, const BatchI32& len, int max_len, float softmax_scale, float* out, void* ws,
                           size_t ws_bytes, hipStream_t s, const FoldSource* window = nullptr);   // window: of a per-channel cache

}  // namespace xq
