// A whole window of decode steps at once: attention (chunk.hip, called by fk_decode_window) and attention with the feature
// state (chunk_feat.hip, called by fk_decode_window_feat).
#pragma once
#include "fk_common.h"

namespace fk {

struct ChunkParams {
    const void *q_seq, *k_seq, *v_seq;  // [T][batch][heads][head_dim]
    void *K, *V;                        // the cache
    int32_t *pos, *len;
    const int32_t* pos_seq;             // [T][batch]
    void* out_seq;
    float scale_log2e;
    int batch, n_kv, g, cap, T, rows;
    int qtiles;                         // workgroups per row
    uint32_t* row_cnt;                  // [rows] arrival counters, zero between launches
    // feature variant
    float2* stat;                       // [rows][T * g] (maximum, 1 / normaliser) of every query
    float* feat;                        // [rows][6][cap][GP]
    int chunk_pos, chunk_len;           // position of the window's first step in its chunk
};

// bf16 caches (with features: head_dim 128); the arguments have been checked by the caller
fk_status chunk_window(const fk_cache_desc* d, const ChunkParams& P, hipStream_t st);
fk_status chunk_window_feat(const ChunkParams& P, int max_len /* at the last step; sizes the launch */, hipStream_t st);

}  // namespace fk
