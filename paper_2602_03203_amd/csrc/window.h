// A whole window of decode steps at once (window.hip): attention, called by fk_decode_window, and attention with the feature
// state, called by fk_decode_window_feat.  And how a single step cuts a row into splits (attn.hip), which the windows follow.
#pragma once
#include "fk_common.h"

namespace fk {

// ---- splits of a row in a single step ----------------------------------------------------------------------------
struct AttnShape {
    int rows, head_dim;
    bool bf16, cold;   // cold: FK_CACHE_COLD
};

struct AttnPlan {
    int split_len;  // keys per split (multiple of the wave tile)
    int nsplit;     // splits per row
    bool rotate;    // workgroups start at different tiles of their splits
};

// Splits per row that the workspace has records for, an upper bound on the plan's for any max_len.  The bf16 D = 128 kernel
// saturates the memory system from 128 workgroups of eight wavefronts when the cache sits in the Infinity Cache, so rows are
// split only when there are fewer rows than that (no split = no cross-workgroup merge at the end of the launch); a cold cache
// comes from HBM, whose latency takes every CU to cover: up to 256 workgroups.
__host__ __device__ inline int attn_max_splits(const AttnShape& a) {
    if (a.bf16 && a.head_dim == 128 && a.cold) {
        const int want = 256 / a.rows;
        return want < 1 ? 1 : want;
    }
    const int target = (a.bf16 && a.head_dim == 128) ? 128 : 512;
    const int want = (target + a.rows - 1) / a.rows;
    return want < 1 ? 1 : want;
}

__host__ __device__ inline AttnPlan attn_plan(const AttnShape& a, int max_len) {
    const int tile = 32, rows = a.rows;
    int want = attn_max_splits(a);
    // A split is worth its share of the merge (1 to 1.5 us, and 0.1 us for every record beyond sixteen) when it fills its wavefronts.
    // bf16: eight wavefronts take 256 keys a round, about 1.1 us; fp32: four take 64 (D = 128: 32).  Measured per step, us:
    //   8 rows, D = 64:  1500 keys  47 splits 12.8, 8: 6.9, 4: 7.5, 1: 12.7;  300 keys  10: 6.7, 1: 6.1;  8192 keys  64: 15.4, 32: 11.1, 16: 10.1
    //   D = 128:  8 rows of 2048  16: 8.3, 8: 7.8;  8 rows of 300  10: 7.3, 1: 6.5;  1 row of 16000  125: 17.3, 32: 10.9, 16: 13.0
    //   D = 64, 128 rows of 2048  4: 15.0, 2: 14.7, 1: 18.4;  32 rows of 2048  16: 10.2, 8: 8.2, 4: 9.0 (so 256 workgroups there)
    //   fp32, 16 rows:  D = 128, 300 keys  10: 9.2, 5: 8.2;  D = 64, 500 keys  16: 9.1, 8: 7.0;  2 rows of 144  5: 5.7, 3: 5.8
    int most;
    if (a.bf16) {
        // (long rows keep the finer cut: as fast for equal lengths, 64 rows of 8000 23.6 against 23.0 us, and it evens out ragged ones,
        // 288 rows of up to 21676: 176 against 182 us)
        if (a.head_dim == 64 && max_len < 4096 && want > (255 + rows) / rows) want = (255 + rows) / rows;
        most = max_len <= 512 ? 1 : (max_len + 255) / 256;
        if (most > 16) most = max_len / 512 > 16 ? max_len / 512 : 16;
        // A cold cache's latency takes more workgroups to cover, as long as the merge fetches the records in one go, eight at a time: 8 rows
        // of 500 pairs 8.1 -> 6.7 us, of 1000 7.8 -> 7.1, of 1500 8.0 -> 7.7; 32 rows of 565 8.7 -> 8.4; beyond eight 8 rows of 2000 take
        // 18.2 (15.4).  Not below one round of the wavefronts: 8 rows of 256 6.5 -> 5.6 us unsplit, 64 rows 7.6 -> 6.2.
        if (a.head_dim == 128 && a.cold && max_len > 256) {
            const int fine = (max_len + 95) / 96;
            if (want <= 8) most = fine;
            else if (most < 8) most = fine < 8 ? fine : 8;
        }
    } else {
        most = max_len <= 1024 ? 8 : (max_len + 127) / 128;   // (the merge fetches eight records at a time)
        if (most > (max_len + tile - 1) / tile) most = (max_len + tile - 1) / tile;
    }
    if (want > most) want = most;
    int split_len = (max_len + want - 1) / want;
    split_len = (split_len + tile - 1) / tile * tile;
    // (Rounding the splits down to whole rounds of the workgroup, with the rest of the row as a short split of its
    // own, was measured and dropped: more workgroups than CUs end up two to a CU while other CUs idle, 85 -> 112 us
    // at 64 rows of 16448 keys.)
    AttnPlan p;
    p.split_len = split_len;
    p.nsplit = (max_len + split_len - 1) / split_len;
    if (p.nsplit < 1) p.nsplit = 1;
    // Start every workgroup at another tile of its split when the splits are long and the cache comes from HBM:
    // workgroups that walk rows a near power of two apart in step crowd the same memory channels (measured on
    // 512 MB per launch, 4128 keys per split: 5.2 TB/s in step, 6.3 TB/s rotated); short splits lose 2 % to it.
    p.rotate = p.nsplit > 1 && split_len >= 2048;
    return p;
}

// where a tile walk starts (rotate): tile 0 of the walk is this tile of the split
__host__ __device__ inline int attn_rotation(int row, int split, int ntiles) {
    return (int)(((unsigned)row * 37u + (unsigned)split * 11u) % (unsigned)ntiles);
}

// Which key of a tile of 32 is row (column) n of K in half nt of q.K^T.  Slot u of lane group `quad` of P.V, one 16x16x32 product, is key
// quad * 8 + u: with the logits transposed, as in the windows, a lane then holds the logits of exactly these keys, and its
// probabilities are an operand as they are.  head_dim 128: a lane's two logits are neighbours and go to LDS in one store.  head_dim 64, where
// the operand comes straight from the cache, whose rows should not be every second one (128 rows of 2112 pairs 14.8 us, so 15.3): key, key + 4.
template <int D> __host__ __device__ constexpr int attn_qk_key(int nt, int n) { return D == 128 ? 2 * n + nt : n / 4 * 8 + nt * 4 + n % 4; }
// ... and where the keys of a tile lie in LDS, so that the rows of a half follow each other
template <int D> __host__ __device__ constexpr int attn_qk_row(int key) { return D == 128 ? key % 2 * 16 + key / 2 : key / 4 % 2 * 16 + key / 8 * 4 + key % 4; }

// A logit in base 2, rounded before anything is subtracted from it (no fma with the maximum): the largest key's exponent is then 0 whatever
// the logits' size - the rounding of its product, half a unit in the last place, is beyond +-128 from 2^32 on - and a weight is the same
// in the normaliser and in the feature planes.
__device__ __forceinline__ float attn_logit(float c, float scale) {
#pragma clang fp contract(off)
    return c * scale;
}

// bf16 pairs with an infinity or a NaN among them
__device__ __forceinline__ bool pair_not_finite(uint32_t w) { return (w & 0x7f80u) == 0x7f80u || (w & 0x7f800000u) == 0x7f800000u; }

// head_dim 64, probabilities as three bf16 terms: the merged products of the terms; an infinity or a NaN of the first stays what it is
__device__ __forceinline__ float add_terms(float first, float second, float third) {
    return (__float_as_uint(first) & 0x7f800000u) == 0x7f800000u ? first : first + (second + third);
}

// ---- windows -----------------------------------------------------------------------------------------------------
struct WindowParams {
    const void *q_seq, *k_seq, *v_seq;  // [T][batch][heads][head_dim]
    void *K, *V;                        // the cache
    int32_t *pos, *len;
    const int32_t* pos_seq;             // [T][batch]
    void* out_seq;
    float scale_log2e;
    int batch, n_kv, g, cap, T, rows;
    uint32_t* row_cnt;                  // [rows] arrival counters, zero between launches
    AttnShape shape;                    // without features: the single steps' splits, ...
    int max_len_first;                  // ... which also follow from this
    // feature variant
    float2* stat;                       // [rows][T * g] (maximum, 1 / normaliser) of every query
    float* feat;                        // [rows][6][cap][GP]
    int chunk_pos, chunk_len;           // position of the window's first step in its chunk
};

// bf16 caches (with features: head_dim 128); the arguments have been checked by the caller
fk_status window_attn(const WindowParams& P, bool split /* some step's rows are split */, hipStream_t st);
fk_status window_feat(const WindowParams& P, int max_len /* at the last step; sizes the launch */, hipStream_t st);

}  // namespace fk
