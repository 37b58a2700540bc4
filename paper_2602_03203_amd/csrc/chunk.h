// Attention of a whole window of decode steps at once (chunk.hip), called by fk_decode_window.
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
};

// bf16 caches; the arguments have been checked by the caller
fk_status chunk_window(const fk_cache_desc* d, const ChunkParams& P, hipStream_t st);

}  // namespace fk
