// fk_decode_attn / fk_decode_step: split-K flash-decode attention over the retained set
// (Appendix A, "Problem Setup": o_hat = sum_{i in S} softmax_S(s)_i v_i), optionally fused with
// the append of the step's new pair (Section 3.1) so that one decode step is ONE launch.
//
// Work decomposition.  A row (sequence, KV head) is cut into `nsplit` splits of `split_len`
// keys; one workgroup handles one split for all g query heads of the group, so K and V are
// fetched from HBM once per group.  Inside a workgroup every wavefront walks its own tiles of
// the split and keeps an online softmax (running maximum m, running sum l, un-normalised
// accumulator acc); the wavefronts are merged through LDS and the splits of a row through a
// small record in the workspace, the last workgroup of the row to arrive doing the final
// log-sum-exp merge and the store of `out` (no second launch).  Short rows, and rows of which there are
// enough to fill the chip (attn_plan says where), are not split and the launch has no cross-workgroup traffic.
//
// bf16, D = 128.  K and V tiles of 32 keys are fetched with fully coalesced 128-bit loads (a row is
// 16 lanes x 16 bytes, four rows per wavefront instruction).  The K tile is staged in LDS (padded
// rows) and read back in the MFMA operand layout (one key per lane, 8 consecutive channels), so
// q.K^T is a 16x16x32 MFMA chain with A = the group's query rows zero padded to 16.  The softmax
// runs on the MFMA result layout (one key per lane, 4 heads per lane).  The probabilities, rounded
// to bf16 (the same rounded values feed the normaliser), go through LDS into the A operand of the
// second contraction; its B operand is the V tile, transposed 8x8 inside each lane's registers
// (byte permutes, no cross-lane traffic), so P.V is MFMA too and the accumulator lives in the
// MFMA result layout.  The vector ALUs only do the softmax.
// bf16, D = 64.  The same with shorter rows: the K operand is loaded directly (a row is four lanes x 16 bytes per k-step), V
// 8 bytes a lane, and the probabilities go in as three bf16 terms (all 24 bits of them), normalised by their
// fp32 sum.  P.V as fp32 FMA, every key group its own accumulator and 64 of them to merge per workgroup, took 18.9 us at
// 128 rows of 2048 pairs and 8.7 us at 8 rows of 300; this takes 14.6 and 6.2.
// fp32.  q.K^T as fp32 FMA plus a DPP row reduction, P.V as fp32 FMA.
//
// fk_decode_step_feat (FEAT variant, Appendix B.1).  One workgroup per row.  The scaled base-2 logits
// are stored to a per-row scratch as they are formed; after the wavefront merge, with the final maximum
// and normaliser known, a second pass turns them into attention weights and adds them to the open
// planes of the row's feature state.
#include "window.h"
#include <mutex>

namespace fk {

static constexpr float kNegBig = -1.0e30f;  // "no key seen yet"; exp2(kNegBig - m) == 0

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
union B128 {
    uint4 u;
    bf16x8_t v;
};

// Cross-workgroup traffic (split records, arrival counters) uses agent-scope relaxed atomics:
// they compile to loads / stores that bypass the per-XCD caches (sc1), which costs nothing next
// to a device-wide fence (that one writes back and invalidates a whole L2).
__device__ __forceinline__ void st_agent(float* p, float v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float ld_agent(const float* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// all of this wave's earlier global stores have been acknowledged (vmcnt(0); expcnt, lgkmcnt untouched)
__device__ __forceinline__ void wait_stores_done() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0x0F70);
}

// 16-byte load of streamed cache data.  NT marks it non-temporal: a cache that is larger than the Infinity Cache
// (256 MB) is re-read from HBM every step anyway, and lines that are not kept in the caches make room faster
// (+8 .. 11 % bandwidth measured at 0.5 .. 4 GB); below that size the plain load is the faster one.
template <bool NT>
__device__ __forceinline__ uint4 ld_stream(const uint4* p) {
    if constexpr (NT) {
        typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
        const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
        return make_uint4(v.x, v.y, v.z, v.w);
    } else {
        return *p;
    }
}
template <bool NT>
__device__ __forceinline__ uint2 ld_stream(const uint2* p) {
    if constexpr (NT) {
        typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
        const u32x2 v = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(p));
        return make_uint2(v.x, v.y);
    } else {
        return *p;
    }
}
static constexpr size_t kStreamNtBytes = (size_t)352 << 20;  // K + V bytes of a launch from which NT loads are used

// i-th dword of a 16-byte register quad; i is a compile-time constant after unrolling
__device__ __forceinline__ uint32_t dword_of(const uint4& v, int i) { return i == 0 ? v.x : (i == 1 ? v.y : (i == 2 ? v.z : v.w)); }

template <int CTRL>
__device__ __forceinline__ float dpp_max_step(float v) { return fmaxf(v, dpp_f<CTRL>(v)); }
__device__ __forceinline__ float row16_max(float v) {
    v = dpp_max_step<DPP_QUAD_XOR1>(v);
    v = dpp_max_step<DPP_QUAD_XOR2>(v);
    v = dpp_max_step<DPP_ROW_HALF_MIRROR>(v);
    v = dpp_max_step<DPP_ROW_MIRROR>(v);
    return v;
}

// over the KG key groups of a wavefront (fp32): lanes that differ in bit 5, and with four groups in bit 4
template <int KG> __device__ __forceinline__ float lanes_sum(float v) {
    v = add_halves(v, v);
    return KG == 4 ? add_rows(v, v) : v;
}
template <int KG> __device__ __forceinline__ float lanes_max(float v) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
    if (KG == 4) {
        auto x = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = fmaxf(__uint_as_float(x[0]), __uint_as_float(x[1]));
    }
    return v;
}

// ---- geometry ------------------------------------------------------------------------------
// HEADS: fp32, a workgroup for every query head (attn_by_head)
template <typename T, int D, int G, bool HEADS = false> struct AttnCfg {
    static constexpr bool MFMA = sizeof(T) == 2;
    static constexpr bool PVM = MFMA;                       // P.V on MFMA as well
    static constexpr bool SPLIT_P = PVM && D == 64;         // probabilities as three bf16 terms, together all 24 bits of them
    static constexpr int CH = D * (int)sizeof(T) / 16;      // 16-byte chunks per row = lanes per key (P.V layout)
    static constexpr int KG = kWave / CH;                   // key groups per wave in the P.V layout
    static constexpr int WAVES = PVM ? 8 : HEADS ? 16 : 4;
    static constexpr int THREADS = WAVES * kWave;
    static constexpr int KT = MFMA ? 32 : KG * 4;           // keys per wave iteration
    static constexpr int VU = KT / KG;                      // V (and fp32 K) loads per lane per iteration
    static constexpr int EPL = Vec16<T>::N;                 // channels per lane
    static constexpr int GP = G <= 4 ? 4 : 8;               // heads padded to the MFMA result rows in use
    static constexpr int NG = PVM || HEADS ? WAVES : WAVES * KG;     // partial accumulators per workgroup
    static constexpr int PS = KT + 8;                       // PVM: bf16 row stride of the P tile in LDS
    static constexpr int KRS = 272;                         // D = 128: padded byte stride of a K row in LDS
    // dynamic LDS (floats unless noted):
    //   PVM:   m [NG][G] | l [NG][G] | w [NG][G] | M [8] | P tiles [WAVES][PROWS][PS] bf16 | D = 128:
    //          K tiles [WAVES][KT][KRS] bytes (a wavefront's partial accumulator [G][D] reuses its own K tile once its loop is
    //          over), 73 KB at G = 4: two workgroups fit the 160 KB of a CU; D = 64: the partial accumulators, term by term
    //   fp32:  acc [NG][G][D] | m [NG][G] | l [NG][G] | w [NG][G] | M [8]
    static constexpr int ACC_STRIDE = PVM && D == 128 ? KT * KRS / 4 : (SPLIT_P ? 3 : 1) * G * D;  // floats between the partial accumulators
    static constexpr size_t HEAD_FLOATS = 3 * (size_t)NG * G + 8;   // m, l, w, M
    static constexpr int PROWS = SPLIT_P ? 3 * GP : GP;               // PVM: rows of a P tile, term by term
    static constexpr size_t PB_BYTES = (size_t)WAVES * PROWS * PS * 2;  // PVM: the bf16 P tiles
    static constexpr size_t LDS_BYTES =
        PVM ? sizeof(float) * (HEAD_FLOATS + (size_t)WAVES * ACC_STRIDE) + PB_BYTES
            : sizeof(float) * ((size_t)NG * G * D + HEAD_FLOATS);
    // attention-feature variant: lx [NG][G] exact normaliser partials | invL [8], behind everything else
    static constexpr size_t LDS_BYTES_FEAT = LDS_BYTES + sizeof(float) * ((size_t)NG * G + 8);
    static constexpr size_t LX_OFFSET = LDS_BYTES / sizeof(float);  // float index of lx in the dynamic LDS
};

static AttnShape attn_shape(const fk_cache_desc* d) {
    return {d->batch * d->n_kv_heads, d->head_dim, d->dtype == FK_BF16, (d->flags & FK_CACHE_COLD) != 0};
}

// workspace: [row arrival counters: rows u32] padded to 256 B | records
static size_t attn_counter_bytes(const fk_cache_desc* d) {
    const size_t n = (size_t)d->batch * d->n_kv_heads;
    return (n * sizeof(uint32_t) + 255) / 256 * 256;
}

struct AttnParams {
    const void* q;
    void* K;
    void* V;
    int32_t* pos;
    int32_t* len;
    const void* k_new;  // null: no append
    const void* v_new;
    const int32_t* pos_new;
    float scale_log2e;
    int n_kv, cap, split_len, nsplit;
    int rotate;          // bf16: workgroups start at different tiles of their splits
    int by_length;       // bf16, streamed cache, unsplit rows: workgroup i takes the i-th longest row
    float* rec;          // [rows][nsplit][G][D + 2]
    uint32_t* row_cnt;   // [rows], zero between launches
    void* out;
    // attention features (Appendix B.1), only read by the feature variant of the kernel
    float* feat;      // [rows][6][cap][GP]
    float* logit;     // [rows][cap][GP] scratch: base-2 logits of this step
    int chunk_pos, chunk_len;
};

// planes of the feature state: sums of this chunk's attention weights over the last 8 / 16 / 32
// queries and over the whole chunk, then the sums carried over the earlier chunks (plain, 0.9-decayed)
enum { FEAT_W8 = 0, FEAT_W16, FEAT_W32, FEAT_WL, FEAT_CUM, FEAT_DEC, FEAT_PLANES };

__device__ __forceinline__ void feat_add(float4* dst, const float4 p) {
    const float4 v = *dst;
    *dst = make_float4(v.x + p.x, v.y + p.y, v.z + p.z, v.w + p.w);
}

__device__ __forceinline__ float4 keep_if(bool c, const float4 p) {
    return make_float4(c ? p.x : 0.f, c ? p.y : 0.f, c ? p.z : 0.f, c ? p.w : 0.f);
}

// The row at place `rank` of the rows from the longest to the shortest: lengths in 256 classes (equal within a 256th of the
// longest), rows of a class in their order; lengths that differ by less than an eighth keep the order they have.  LDS words:
// lengths [rows] | class counts [256] | maximum, minimum, result.  Every thread calls;
// all workgroups of a launch see the same lengths (they change after the last one has finished).
template <int THREADS>
__device__ __forceinline__ int row_by_length(const int32_t* len, int rows, int cap, int rank, int* lds) {
    int *s_len = lds, *s_cnt = lds + rows, *s_max = s_cnt + 256, *s_min = s_max + 1, *s_row = s_min + 1;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    if (tid < 256) s_cnt[tid] = 0;
    if (tid == 0) {
        *s_max = 1;
        *s_min = cap;
    }
    __syncthreads();
    int lo = cap, hi = 1;
    for (int r = tid; r < rows; r += THREADS) {
        const int n = min(max(len[r], 0), cap);
        s_len[r] = n;
        lo = min(lo, n);
        hi = max(hi, n);
    }
    if (lo < *s_min) atomicMin(s_min, lo);
    if (hi > *s_max) atomicMax(s_max, hi);
    __syncthreads();
    lo = *s_min;
    hi = *s_max;
    if (hi - lo < hi / 8) {
        __syncthreads();
        return rank;
    }
    const float per_class = 255.9f / (float)*s_max;
    auto cls = [&](int n) { return 255 - (int)((float)n * per_class); };   // the longest first
    for (int r = tid; r < rows; r += THREADS) atomicAdd(&s_cnt[cls(s_len[r])], 1);
    __syncthreads();
    if (tid < kWave) {   // one wavefront, four classes a lane
        int c[4], tot = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) tot += c[j] = s_cnt[4 * lane + j];
        int incl = tot;
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const int o = __shfl_up(incl, off);
            if (lane >= off) incl += o;
        }
        int run = incl - tot, mine = -1, left = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (run <= rank && rank < run + c[j]) {   // one lane
                mine = 4 * lane + j;
                left = rank - run;
            }
            run += c[j];
        }
        const int src = __ffsll((long long)__ballot(mine >= 0)) - 1;
        const int k = __builtin_amdgcn_readlane(mine, src);
        left = __builtin_amdgcn_readlane(left, src);
        for (int base = 0; base < rows; base += kWave) {   // the left-th row of class k
            const int r = base + lane;
            unsigned long long m = __ballot(r < rows && cls(s_len[min(r, rows - 1)]) == k);
            const int n = __popcll(m);
            if (left < n) {
                for (; left > 0; --left) m &= m - 1;
                if (lane == 0) *s_row = base + __ffsll((long long)m) - 1;
                break;
            }
            left -= n;
        }
    }
    __syncthreads();
    const int row = *s_row;
    __syncthreads();   // the LDS is the caller's again
    return row;
}

// Up to three heads of head_dim 128 are told to leave room for two workgroups on a CU: by themselves they take 130 (two heads) to 134 registers,
// told 128 (512 rows of 300 pairs: one head 16.7 and 14.9 us, two 15.6 and 13.9, three 18.1 and 15.7; the same streamed, two 14.4 and 12.4).
// Four take 128 untold.  None of them spills.
template <typename T, int D, int G, bool FEAT> constexpr bool attn_two() { return sizeof(T) == 2 && D == 128 && G <= 3 && !FEAT; }

template <typename T, int D, int G, bool FEAT, bool NT, bool HEADS = false>
__global__ __launch_bounds__((AttnCfg<T, D, G, HEADS>::THREADS), (attn_two<T, D, G, FEAT>() ? 4 : AttnCfg<T, D, G, HEADS>::WAVES / 4)) void attn_kernel(const AttnParams P) {
    using C = AttnCfg<T, D, G, HEADS>;
    constexpr int CH = C::CH, KG = C::KG, WAVES = C::WAVES, KT = C::KT, VU = C::VU, EPL = C::EPL, GP = C::GP, NG = C::NG;
    extern __shared__ __attribute__((aligned(16))) float smem[];
    constexpr bool CAN_ORDER = C::PVM && NT && !FEAT;
    int row = HEADS ? blockIdx.x : blockIdx.y;   // (HEADS: so that the workgroups of a row sit on one XCD where the rows are a multiple of eight)
    if constexpr (CAN_ORDER) {
        if (P.by_length) row = row_by_length<C::THREADS>(P.len, gridDim.y, P.cap, row, reinterpret_cast<int*>(smem));
    }
    const int split = HEADS ? 0 : blockIdx.x, head = HEADS ? blockIdx.y : 0, heads = HEADS ? gridDim.y : G;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;

    // PVM: head | P tiles | K tiles, the partial accumulators live in the K tiles; fp32: acc | head
    float* s_m = C::PVM ? smem : smem + (size_t)NG * G * D;  // [NG][G]
    float* s_l = s_m + NG * G;                 // [NG][G]
    float* s_w = s_l + NG * G;                 // [NG][G] merge weights 2^(m_g - M)
    float* s_M = s_w + NG * G;                 // [8] merged maximum per head
    float* s_p = s_M + 8;                      // PVM: the bf16 P tiles
    unsigned char* s_kt = reinterpret_cast<unsigned char*>(s_p) + C::PB_BYTES;  // PVM: K tiles [WAVES][KT][KRS]
    float* s_acc = C::PVM ? reinterpret_cast<float*>(s_kt) : smem;  // partial g2 at s_acc + g2 * ACC_STRIDE, [G][D]
    __shared__ int s_last;

    const bool appending = P.k_new != nullptr;
    const int n_old = min(max(P.len[row], 0), P.cap);
    const bool do_append = appending && n_old < P.cap;
    const int n = n_old + (do_append ? 1 : 0);
    // if the caller's max_len was too small the last split runs on to the row's end (slower, still right)
    const bool one_split = n <= P.split_len || P.nsplit == 1;   // (no division before the loads: they wait for what is worked out here)
    T* out = reinterpret_cast<T*>(P.out) + ((size_t)row * heads + head) * D;
    uint32_t arrived = 0;   // HEADS, thread 0

    // Every workgroup of the row calls finish() once, as its last action.  With one workgroup per
    // row it just publishes the new length.  With several, all of them (also those whose split lies
    // beyond the row's end) report to the row's arrival counter; the last one to arrive merges the
    // splits, out = sum_s acc_s 2^(m_s - m*) / sum_s l_s 2^(m_s - m*), and only then bumps len[row],
    // which every workgroup of the row has read by that time.
    auto finish = [&](bool wrote_record) {
        if constexpr (CAN_ORDER) {
            if (P.by_length) {   // other workgroups still look the lengths up: the last one to finish appends for all rows
                if (!appending) return;
                __syncthreads();
                if (tid == 0) {
                    s_last = __hip_atomic_fetch_add(&P.row_cnt[0], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.y - 1;
                    if (s_last) __hip_atomic_store(&P.row_cnt[0], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                __syncthreads();
                if (s_last)
                    for (int r = tid; r < (int)gridDim.y; r += C::THREADS) {
                        const int len = min(max(P.len[r], 0), P.cap);
                        if (len < P.cap) P.len[r] = len + 1;
                    }
                return;
            }
        }
        if constexpr (HEADS) {   // the last workgroup of the row: the others have read its length
            if (do_append && tid == 0 && arrived == gridDim.y - 1) {
                if (gridDim.y > 1) __hip_atomic_store(&P.row_cnt[row], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                P.len[row] = n;
            }
            return;
        }
        if (gridDim.x == 1) {
            if (do_append && tid == 0) P.len[row] = n;
            return;
        }
        if (!appending && one_split) return;  // same decision in every workgroup of the row
        const int used = min((n + P.split_len - 1) / P.split_len, P.nsplit);   // splits in use
        if (wrote_record) wait_stores_done();
        __syncthreads();
        if (tid == 0) {
            const uint32_t prev = __hip_atomic_fetch_add(&P.row_cnt[row], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s_last = prev == gridDim.x - 1;
            if (s_last) __hip_atomic_store(&P.row_cnt[row], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
        if (!s_last) return;
        if (used > 1) {
            // log-sum-exp merge of the splits' records, eight records' loads in flight per thread
            const float* r0 = P.rec + (size_t)row * P.nsplit * G * (D + 2);
            const size_t stride = (size_t)G * (D + 2);
            for (int idx = tid; idx < G * D; idx += C::THREADS) {
                const int h = idx / D, d = idx % D;
                const float* r = r0 + (size_t)h * (D + 2);
                float M = kNegBig, a = 0.f, ls = 0.f;
                for (int s0 = 0; s0 < used; s0 += 8) {
                    float mv[8], lv[8], av[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const float* rs = r + (size_t)min(s0 + u, used - 1) * stride;
                        mv[u] = ld_agent(rs + D);
                        lv[u] = ld_agent(rs + D + 1);
                        av[u] = ld_agent(rs + d);
                    }
                    float cm = M;
#pragma unroll
                    for (int u = 0; u < 8; ++u)
                        if (s0 + u < used) cm = fmaxf(cm, mv[u]);
                    const float c0 = exp2f(M - cm);
                    a *= c0;
                    ls *= c0;
                    M = cm;
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        if (s0 + u < used) {
                            const float cw = exp2f(mv[u] - M);
                            a = fmaf(av[u], cw, a);
                            ls = fmaf(lv[u], cw, ls);
                        }
                    }
                }
                store_out(out + idx, a / ls);
            }
        }
        if (do_append && tid == 0) P.len[row] = n;
    };

    if (n == 0) {
        if (split == 0)
            for (int i = tid; i < G * D; i += C::THREADS) store_out(out + i, 0.f);
        finish(false);
        return;
    }
    const int start = split * P.split_len;
    if (start >= n) {
        finish(false);
        return;
    }
    const int end = split == P.nsplit - 1 ? n : min(n, start + P.split_len);

    T* Kr = reinterpret_cast<T*>(P.K) + (size_t)row * P.cap * D;
    T* Vr = reinterpret_cast<T*>(P.V) + (size_t)row * P.cap * D;
    // The workgroup whose split holds the slot of the new pair stores it into the cache.  The bf16
    // D = 128 path never waits for that store: lanes that need the new row read it from k_new / v_new.
    const bool owns_new = do_append && n_old >= start && n_old < end;
    const uint4* knew_row = reinterpret_cast<const uint4*>(reinterpret_cast<const T*>(P.k_new) + (size_t)row * D);
    const uint4* vnew_row = reinterpret_cast<const uint4*>(reinterpret_cast<const T*>(P.v_new) + (size_t)row * D);
    if (owns_new && head == 0) {
        if (tid < CH) {
            reinterpret_cast<uint4*>(Kr + (size_t)n_old * D)[tid] = knew_row[tid];
        } else if (tid < 2 * CH) {
            reinterpret_cast<uint4*>(Vr + (size_t)n_old * D)[tid - CH] = vnew_row[tid - CH];
        } else if (tid == 2 * CH) {
            P.pos[(size_t)row * P.cap + n_old] = P.pos_new[row / P.n_kv];
        }
        if constexpr (!C::PVM && !HEADS) __syncthreads();  // this fp32 path reads the row back from the cache
    }
    const int new_slot = owns_new ? n_old : -1;
    const uint4* Krow = reinterpret_cast<const uint4*>(Kr);
    const uint4* Vrow = reinterpret_cast<const uint4*>(Vr);
    const T* qrow = reinterpret_cast<const T*>(P.q) + ((size_t)row * heads + head) * D;

    const int dl = lane % CH;   // 16-byte chunk of the row (P.V layout)
    const int kgv = lane / CH;  // key group (P.V layout)
    float acc[G][EPL];
#pragma unroll
    for (int h = 0; h < G; ++h)
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[h][e] = 0.f;

    if constexpr (C::PVM) {
        constexpr int PS = C::PS, KRS = C::KRS;
        const int n16 = lane & 15, quad = lane >> 4;
        constexpr int KEY1 = attn_qk_key<D>(1, 0);
        constexpr int KS = D / 32;          // k-steps of q.K^T
        constexpr int ET = D / 16;          // channel tiles of P.V
        constexpr int HR = G < 4 ? G : 4;   // of a lane's four result rows, those that can belong to a head
        uint16_t* my_pb = reinterpret_cast<uint16_t*>(s_p) + (size_t)wave * C::PROWS * PS;   // [PROWS][PS] bf16
        unsigned char* my_k = s_kt + (size_t)wave * KT * KRS;   // D = 128
        auto put_pair = [&](uint16_t* p, int key0, uint32_t w) {   // probabilities of the lane's two keys
            if constexpr (KEY1 == 1) {
                *reinterpret_cast<uint32_t*>(p + key0) = w;
            } else {
                p[key0] = (uint16_t)w;
                p[key0 + KEY1] = (uint16_t)(w >> 16);
            }
        };
        B128 qa[KS];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const int h = C::SPLIT_P ? n16 % GP : n16;   // SPLIT_P: the heads once for every term (below)
            if (h < G) qa[ks].u = *reinterpret_cast<const uint4*>(qrow + (size_t)h * D + ks * 32 + quad * 8);
            else qa[ks].u = make_uint4(0, 0, 0, 0);
        }
        const float scale = P.scale_log2e;
        // l: the normaliser, of unrounded weights where P.V has all their bits (SPLIT_P), otherwise a column of ones more in P.V, a 129th, the same
        // rounded weights; lx: sum of the unrounded weights (feature variant).  Against sums by vector instructions, us: four heads, 2 rows of
        // 144 pairs 5.34 and 5.20, 128 of 2048 23.1 and 22.9; one head, which has a quarter of the additions and pays for the registers, 8 of 144 4.21
        // and 4.14, 128 of 2048 alike, 512 of 300 14.26 and 14.20; two alike; three 8 of 144 4.86 and 4.94, 128 of 300 6.32 and 6.26.  Windows, which give
        // the same bits: one head 4 %, three 6 to 7 (128 rows of 2048, 128 steps 51.9 and 49.8, 136 and 127).
        float m_run[4], l_run[4], lx_run[4];
        f32x4_t ol = (f32x4_t){0.f, 0.f, 0.f, 0.f};
        B128 ones;
        ones.u = make_uint4(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            m_run[i] = kNegBig;
            l_run[i] = 0.f;
            lx_run[i] = 0.f;
        }
        float* lg_row = FEAT ? P.logit + (size_t)row * P.cap * GP : nullptr;
        f32x4_t o[ET];  // o[e][i] = out[head quad*4 + i][channel n16*ET + e], un-normalised
        // SPLIT_P: the three terms of a probability are rows of their own in the same product: heads 0 .. GP - 1 times (first, second, third
        // term), GP = 4 twelve of the sixteen rows, GP = 8 two products.  The logits and the softmax are formed in every row (the query
        // rows are repeated), so the sums of a term are rescaled like any others; they are added at the end, in the merge.  (A second product
        // onto the rows of the second terms would leave 0 * inf in the others.)  Sums of their own also keep infinite values what they
        // are: a later term may be 0 or negative.
        constexpr bool THIRD = C::SPLIT_P && GP == 8;   // the third terms in a product of their own
        f32x4_t o3[THIRD ? ET : 1];
#pragma unroll
        for (int e = 0; e < ET; ++e) {
            o[e] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
            if constexpr (THIRD) o3[e] = o[e];
        }

        // Tiles are dealt round robin to the wavefronts; with P.rotate the deal starts from a tile that differs
        // from workgroup to workgroup (the online softmax does not care about the order).
        const int ntiles = (end - start + KT - 1) / KT;
        const int rot = P.rotate ? attn_rotation(row, split, ntiles) : 0;
        auto base_of = [&](int t) { return start + (t + rot < ntiles ? t + rot : t + rot - ntiles) * KT; };
        // Feature steps run one workgroup a row: with one head, whose softmax is short, the next tile's loads are issued a tile ahead (32
        // rows of 8192 pairs 62 -> 55 us; with more heads the registers cost more than that: four heads +10 %, eight +30 % at 512 rows).
        constexpr bool AHEAD = FEAT && D == 64 && G == 1;
        // The order of a tile's loads, head_dim 64: K's first halves, its second halves, V (one head, 128 rows of 2112 pairs 14.1 us; the halves of
        // a row together 14.8).  Feature steps: the halves of a row together (four heads, 32 rows of 4000 pairs 36.3 us, otherwise 37.7), and a
        // tile ahead V before K (32 rows of 4000 pairs 31.2 us, otherwise 32.5).
        auto fetch64 = [&](int base, B128 (&kd)[2][2], uint2 (&v)[8]) {
            auto load_k = [&]() {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int nt = FEAT ? i / 2 : i % 2, ks = FEAT ? i % 2 : i / 2;
                    const int kc = min(base + attn_qk_key<D>(nt, n16), end - 1);
                    kd[nt][ks].u = ld_stream<NT>((kc == new_slot ? knew_row : Krow + (size_t)kc * CH) + ks * 4 + quad);
                }
            };
            if constexpr (!AHEAD) load_k();
#pragma unroll
            for (int u = 0; u < 8; ++u) {  // lane (quad, n16): key base + quad*8 + u, channels n16*4 .. +4
                const int kc = min(base + quad * 8 + u, end - 1);
                v[u] = ld_stream<NT>(reinterpret_cast<const uint2*>(kc == new_slot ? vnew_row : Vrow + (size_t)kc * CH) + n16);
            }
            if constexpr (AHEAD) load_k();
        };
        B128 kd_next[2][2];
        uint2 v_next[8];
        if constexpr (AHEAD) {
            if (wave < ntiles) fetch64(base_of(wave), kd_next, v_next);
        }
        for (int t = wave; t < ntiles; t += WAVES) {
            const int base = base_of(t);
            uint4 vr[8];  // D = 64: x, y only
            B128 kd[2][2];  // D = 64: K operand
            if constexpr (D == 64) {
                uint2 v2[8];
                if constexpr (AHEAD) {
#pragma unroll
                    for (int u = 0; u < 8; ++u) v2[u] = v_next[u];
#pragma unroll
                    for (int u = 0; u < 4; ++u) kd[u / 2][u % 2].u = kd_next[u / 2][u % 2].u;
                    if (t + WAVES < ntiles) fetch64(base_of(t + WAVES), kd_next, v_next);
                } else {
                    fetch64(base, kd, v2);
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    vr[u].x = v2[u].x;
                    vr[u].y = v2[u].y;
                }
            } else {
                uint4 kr[8];  // lane (quad, n16): key base + quad*8 + u, 16-byte chunk n16
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int kc = min(base + quad * 8 + u, end - 1);
                    kr[u] = ld_stream<NT>((kc == new_slot ? knew_row : Krow + (size_t)kc * CH) + n16);
                }
                // (One head: with the normaliser's registers the compiler sent the last two rows of K off when the first were there.  32 streamed rows of
                // 1171 pairs 8.42 us a step, so 8.19; out of the caches 12 of 12077 15.3 and 15.1, 8 of 2000 5.95 and 6.0.  Two heads, streamed, 8 of
                // 1624 7.17 and 7.10; out of the caches 128 of 2048 22.55 and 22.7.  Three heads spill.)
                if constexpr ((G == 1 || (NT && G == 2)) && attn_two<T, D, G, FEAT>()) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int kc = min(base + quad * 8 + u, end - 1);
                    vr[u] = ld_stream<NT>((kc == new_slot ? vnew_row : Vrow + (size_t)kc * CH) + n16);
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) *reinterpret_cast<uint4*>(my_k + (quad * 4 + attn_qk_row<D>(u)) * KRS + n16 * 16) = kr[u];
            }
            __builtin_amdgcn_wave_barrier();
            // B operand of q.K^T: lane = key attn_qk_key(nt, n16), channels ks*32 + quad*8 .. +8
            f32x4_t c[2];
#pragma unroll
            for (int nt = 0; nt < 2; ++nt) {
                c[nt] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    B128 kb;
                    if constexpr (D == 64) kb = kd[nt][ks];
                    else kb.u = *reinterpret_cast<const uint4*>(my_k + (nt * 16 + n16) * KRS + (ks * 4 + quad) * 16);
                    c[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qa[ks].v, kb.v, c[nt], 0, 0, 0);
                }
            }
            if constexpr (attn_two<T, D, G, FEAT>()) {
                // K's operands two reads ahead of the products, which the compiler gives up where registers are short: three heads, 128 rows of 300
                // pairs 6.44 us a step, so 6.25, of 2048 23.1 and 22.8; two, 128 of 2048 22.7 and 22.5; one, 128 of 300 5.61 and 5.51.
                __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);   // LDS reads
#pragma unroll
                for (int i = 0; i < 2 * KS - 2; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);   // a product
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                }
                __builtin_amdgcn_sched_group_barrier(0x8, 2, 0);
            }
            int any_lane = threadIdx.x;
            if constexpr (attn_two<T, D, G, FEAT>()) asm volatile("" : "+v"(any_lane));   // (opaque: the key would stay in a register)
            const int key0 = attn_qk_key<D>(0, any_lane & 15);   // the lane's logits: keys key0 and key0 + KEY1 of the tile
            bool changed = false;
            float corr[4];
            uint32_t pw[4], p3[4];   // bf16 pairs: keys key0 and key0 + KEY1
            if constexpr (FEAT) {  // keep the step's logits: the second pass turns them into attention weights
                if (quad * 4 < GP) {
                    if (base + key0 < end)
                        *reinterpret_cast<float4*>(lg_row + (size_t)(base + key0) * GP + quad * 4) =
                            make_float4(attn_logit(c[0][0], scale), attn_logit(c[0][1], scale), attn_logit(c[0][2], scale), attn_logit(c[0][3], scale));
                    if (base + key0 + KEY1 < end)
                        *reinterpret_cast<float4*>(lg_row + (size_t)(base + key0 + KEY1) * GP + quad * 4) =
                            make_float4(attn_logit(c[1][0], scale), attn_logit(c[1][1], scale), attn_logit(c[1][2], scale), attn_logit(c[1][3], scale));
                }
            }
#pragma unroll
            for (int i = 0; i < HR; ++i) {
                const float s0 = (base + key0 < end) ? attn_logit(c[0][i], scale) : -INFINITY;
                const float s1 = (base + key0 + KEY1 < end) ? attn_logit(c[1][i], scale) : -INFINITY;
                const float mn = fmaxf(m_run[i], row16_max(fmaxf(s0, s1)));
                changed |= mn > m_run[i];
                corr[i] = exp2f(m_run[i] - mn);
                // probabilities rounded to bf16; the SAME rounded values go into l, so the weights stay normalised
                const float e0 = exp2f(s0 - mn), e1 = exp2f(s1 - mn);
                const uint32_t w = pack_bf16(e0, e1);
                pw[i] = w;
                if constexpr (C::SPLIT_P) {   // each term of what the ones before leave; GP = 4: row quad q holds term q, GP = 8: q / 2
                    const float r0 = e0 - bf16_lo(w), r1 = e1 - bf16_hi(w);
                    const uint32_t w2 = pack_bf16(r0, r1);
                    p3[i] = pack_bf16(r0 - bf16_lo(w2), r1 - bf16_hi(w2));
                    const int term = quad * 4 / GP;
                    pw[i] = term == 0 ? w : w2;
                    if constexpr (!THIRD) pw[i] = term < 2 ? pw[i] : p3[i];
                    l_run[i] = l_run[i] * corr[i] + e0 + e1;
                } else {
                    if constexpr (FEAT) lx_run[i] = lx_run[i] * corr[i] + e0 + e1;
                }
                m_run[i] = mn;
            }
            if (quad * 4 < C::PROWS) {
#pragma unroll
                for (int i = 0; i < HR; ++i) {
                    put_pair(my_pb + (quad * 4 + i) * PS, key0, pw[i]);
                    if constexpr (THIRD) {
                        if (quad < 2) put_pair(my_pb + (16 + quad * 4 + i) * PS, key0, p3[i]);
                    }
                }
            }
            if (__any(changed)) {  // the running maximum moved: rescale what has been accumulated
#pragma unroll
                for (int e = 0; e < ET; ++e)
#pragma unroll
                    for (int i = 0; i < HR; ++i) {
                        o[e][i] *= corr[i];
                        if constexpr (THIRD) o3[e][i] *= corr[i];
                    }
                if constexpr (!C::SPLIT_P) {
#pragma unroll
                    for (int i = 0; i < HR; ++i) ol[i] *= corr[i];
                }
            }
            if (base + KT > end) {
                // The lanes past the end hold copies of the last pair, whose weight 0 there must not meet an infinity or a NaN.  Where it has
                // one (the last quad's last register is a copy: all channels are looked at) the copies become zeros; zeroing them
                // always takes 0.15 to 0.3 us of a step.
                int tail = threadIdx.x;   // (opaque: addresses shared with the loads would stay in registers, 134 of them instead of 126)
                asm volatile("" : "+v"(tail));
                tail = (tail & (kWave - 1)) >> 4;   // quad
                bool bad = pair_not_finite(vr[7].x) || pair_not_finite(vr[7].y);
                if constexpr (D == 128) bad = bad || pair_not_finite(vr[7].z) || pair_not_finite(vr[7].w);
                if (__any(bad && tail == 3)) {
#pragma unroll
                    for (int u = 0; u < 8; ++u)
                        if (base + tail * 8 + u >= end) vr[u] = make_uint4(0, 0, 0, 0);
                }
            }
            __builtin_amdgcn_wave_barrier();
            // A operand of P.V: P[row n16][k-slots quad*8 .. +8]; k-slot u of group quad is key base + quad*8 + u
            B128 pa, pr;
            pa.u = pr.u = make_uint4(0, 0, 0, 0);
            if (n16 < C::PROWS && n16 % 4 < HR) pa.u = *reinterpret_cast<const uint4*>(my_pb + n16 * PS + quad * 8);
            if constexpr (THIRD) {
                if (n16 < GP) pr.u = *reinterpret_cast<const uint4*>(my_pb + (16 + n16) * PS + quad * 8);
            }
            if constexpr (!C::SPLIT_P) ol = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pa.v, ones.v, ol, 0, 0, 0);
            // B operand: tile e = channel n16*ET + e over this lane's 8 k-slots (8 x ET transpose in registers)
#pragma unroll
            for (int e = 0; e < ET; ++e) {
                const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;
                B128 vb;
                vb.u.x = __builtin_amdgcn_perm(dword_of(vr[1], e >> 1), dword_of(vr[0], e >> 1), sel);
                vb.u.y = __builtin_amdgcn_perm(dword_of(vr[3], e >> 1), dword_of(vr[2], e >> 1), sel);
                vb.u.z = __builtin_amdgcn_perm(dword_of(vr[5], e >> 1), dword_of(vr[4], e >> 1), sel);
                vb.u.w = __builtin_amdgcn_perm(dword_of(vr[7], e >> 1), dword_of(vr[6], e >> 1), sel);
                o[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pa.v, vb.v, o[e], 0, 0, 0);
                if constexpr (THIRD) o3[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pr.v, vb.v, o3[e], 0, 0, 0);
            }
            __builtin_amdgcn_wave_barrier();
        }
        // A wavefront without a tile still has its queries' loads open.  Left open, the compiler (one head of head_dim 128) waits for every store
        // of wave 0 before the records are read, the arrival counter's reset among them: 8 rows of 2000 pairs 5.9 us, so 5.7; 32 of 900 6.2 and 5.9.
        __builtin_amdgcn_s_waitcnt(0x0F70);
        // publish one partial per wave
#pragma unroll
        for (int i = 0; i < HR; ++i) {
            const int h = quad * 4 + i;
            const float ls = C::SPLIT_P ? group_sum<16>(l_run[i]) : ol[i];
            const int ht = C::SPLIT_P ? h % GP : h, term = C::SPLIT_P ? h / GP : 0;   // SPLIT_P: row h holds term `term` of head ht
            float* dst = s_acc + (size_t)wave * C::ACC_STRIDE + (size_t)(term * G + ht) * D + n16 * ET;  // D = 128: own K tile, its loop is over
            if (ht < G && h < C::PROWS) {
#pragma unroll
                for (int e = 0; e < ET; e += 4) *reinterpret_cast<float4*>(dst + e) = make_float4(o[e][i], o[e + 1][i], o[e + 2][i], o[e + 3][i]);
            }
            if constexpr (THIRD) {
                if (h < G) *reinterpret_cast<float4*>(dst + 2 * G * D) = make_float4(o3[0][i], o3[1][i], o3[2][i], o3[3][i]);
            }
            if (h < G && n16 == 0) {
                s_m[wave * G + h] = m_run[i];
                s_l[wave * G + h] = ls;
            }
            if constexpr (FEAT && !C::SPLIT_P) {
                const float lxs = group_sum<16>(lx_run[i]);
                if (h < G && n16 == 0) smem[C::LX_OFFSET + wave * G + h] = lxs;
            }
        }
    } else {
        // fp32: every key group (CH lanes) keeps its own online softmax over the keys it sees
        float qf[G][EPL];
#pragma unroll
        for (int h = 0; h < G; ++h) {
            Vec16<T>::unpack(*reinterpret_cast<const uint4*>(qrow + (size_t)h * D + dl * EPL), qf[h]);
#pragma unroll
            for (int e = 0; e < EPL; ++e) qf[h][e] *= P.scale_log2e;
        }
        float m[G], l[G];
#pragma unroll
        for (int h = 0; h < G; ++h) {
            m[h] = kNegBig;
            l[h] = 0.f;
        }
        for (int base = start + wave * KT; base < end; base += WAVES * KT) {
            uint4 kr[VU], vr[VU];
            int key[VU];
#pragma unroll
            for (int u = 0; u < VU; ++u) {
                key[u] = base + u * KG + kgv;
                const int kc = min(key[u], end - 1);
                kr[u] = (HEADS && kc == new_slot ? knew_row : Krow + (size_t)kc * CH)[dl];
            }
#pragma unroll
            for (int u = 0; u < VU; ++u) {
                const int kc = min(key[u], end - 1);
                vr[u] = (HEADS && kc == new_slot ? vnew_row : Vrow + (size_t)kc * CH)[dl];
            }
            float s[VU][G];
#pragma unroll
            for (int u = 0; u < VU; ++u) {
                float kf[EPL];
                Vec16<T>::unpack(kr[u], kf);
#pragma unroll
                for (int h = 0; h < G; ++h) {
                    float d = 0.f;
#pragma unroll
                    for (int e = 0; e < EPL; ++e) d = fmaf(qf[h][e], kf[e], d);
                    d = group_sum<CH>(d);
                    s[u][h] = key[u] < end ? d : kNegBig;
                }
                if constexpr (FEAT) {
                    if (dl == 0 && key[u] < end) {  // heads beyond the group hold zeros
                        float* lg = P.logit + ((size_t)row * P.cap + key[u]) * GP;
#pragma unroll
                        for (int h4 = 0; h4 < GP; h4 += 4)
                            *reinterpret_cast<float4*>(lg + h4) =
                                make_float4(h4 + 0 < G ? s[u][h4 + 0 < G ? h4 + 0 : 0] : 0.f, h4 + 1 < G ? s[u][h4 + 1 < G ? h4 + 1 : 0] : 0.f,
                                            h4 + 2 < G ? s[u][h4 + 2 < G ? h4 + 2 : 0] : 0.f, h4 + 3 < G ? s[u][h4 + 3 < G ? h4 + 3 : 0] : 0.f);
                    }
                }
            }
            float p[VU][G];
#pragma unroll
            for (int h = 0; h < G; ++h) {
                float mn = m[h];
#pragma unroll
                for (int u = 0; u < VU; ++u) mn = fmaxf(mn, s[u][h]);
                const float corr = exp2f(m[h] - mn);
                float ps = 0.f;
#pragma unroll
                for (int u = 0; u < VU; ++u) {
                    p[u][h] = key[u] < end ? exp2f(s[u][h] - mn) : 0.f;
                    ps += p[u][h];
                }
                l[h] = l[h] * corr + ps;
                m[h] = mn;
#pragma unroll
                for (int e = 0; e < EPL; ++e) acc[h][e] *= corr;
            }
            if (base + KT > end) {   // past the end: zeros, as above
#pragma unroll
                for (int u = 0; u < VU; ++u)
                    if (key[u] >= end) vr[u] = make_uint4(0, 0, 0, 0);
            }
#pragma unroll
            for (int u = 0; u < VU; ++u) {
                float vf[EPL];
                Vec16<T>::unpack(vr[u], vf);
#pragma unroll
                for (int h = 0; h < G; ++h)
#pragma unroll
                    for (int e = 0; e < EPL; ++e) acc[h][e] = fmaf(p[u][h], vf[e], acc[h][e]);
            }
        }
        if constexpr (HEADS) {
            // The wavefront's key groups become one partial: two halves of the wavefront, with D = 64 two rows of 16 lanes in each.  A swap puts
            // one value's parts beside the other's, so the sums of a pair take one addition: a lane ends with G * EPL / KG of them.
#pragma unroll
            for (int h = 0; h < G; ++h) {
                const float mn = lanes_max<KG>(m[h]), w = exp2f(m[h] - mn);
                l[h] = lanes_sum<KG>(l[h] * w);
#pragma unroll
                for (int e = 0; e < EPL; ++e) acc[h][e] *= w;
                if (lane == 0) {
                    s_m[wave * G + h] = mn;
                    s_l[wave * G + h] = l[h];
                }
                float* dst = s_acc + (size_t)wave * C::ACC_STRIDE + (size_t)h * D + dl * EPL;
                const float a = add_halves(acc[h][0], acc[h][1]), b = add_halves(acc[h][2], acc[h][3]);   // upper lanes: of channels 1 and 3
                if constexpr (KG == 2) {
                    dst[lane / 32] = a;
                    dst[2 + lane / 32] = b;
                } else {
                    dst[lane / 16 % 2 * 2 + lane / 32] = add_rows(a, b);
                }
            }
        } else {
            if (dl == 0) {
#pragma unroll
                for (int h = 0; h < G; ++h) {
                    s_m[(wave * KG + kgv) * G + h] = m[h];
                    s_l[(wave * KG + kgv) * G + h] = l[h];
                }
            }
            float* dst = s_acc + (size_t)(wave * KG + kgv) * C::ACC_STRIDE + dl * EPL;
#pragma unroll
            for (int h = 0; h < G; ++h)
#pragma unroll
                for (int e4 = 0; e4 < EPL; e4 += 4)
                    *reinterpret_cast<float4*>(dst + (size_t)h * D + e4) =
                        make_float4(acc[h][e4], acc[h][e4 + 1], acc[h][e4 + 2], acc[h][e4 + 3]);
        }
    }

    // ---- merge the partials of the workgroup -----------------------------------------------------
    __syncthreads();
    // (all wavefronts have the row's length; looked at when the result is out)
    if (HEADS && do_append && gridDim.y > 1 && tid == 0) arrived = __hip_atomic_fetch_add(&P.row_cnt[row], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (int t = tid; t < NG * G; t += C::THREADS) {  // weight of every partial: 2^(m_g - M)
        const int h = t % G;
        float mn = kNegBig;
#pragma unroll 8
        for (int g2 = 0; g2 < NG; ++g2) mn = fmaxf(mn, s_m[g2 * G + h]);
        s_w[t] = exp2f(s_m[t] - mn);
        if (t < G) s_M[t] = mn;
    }
    __syncthreads();
    float* rec = P.rec + ((size_t)row * P.nsplit + split) * G * (D + 2);
    for (int idx = tid; idx < G * D; idx += C::THREADS) {
        const int h = idx / D, d = idx % D;
        const float mn = s_M[h];
        float a = 0.f, ls = 0.f;
        if constexpr (C::SPLIT_P) {
            float a2 = 0.f, a3 = 0.f;
#pragma unroll 8
            for (int g2 = 0; g2 < NG; ++g2) {
                const float *p = s_acc + (size_t)g2 * C::ACC_STRIDE + (size_t)h * D + d, w = s_w[g2 * G + h];
                a = fmaf(p[0], w, a);
                a2 = fmaf(p[G * D], w, a2);
                a3 = fmaf(p[2 * G * D], w, a3);
            }
            a = add_terms(a, a2, a3);
        } else {
#pragma unroll 8
            for (int g2 = 0; g2 < NG; ++g2) a = fmaf(s_acc[(size_t)g2 * C::ACC_STRIDE + (size_t)h * D + d], s_w[g2 * G + h], a);
        }
        if (d == 0 || one_split) {
#pragma unroll 8
            for (int g2 = 0; g2 < NG; ++g2) ls = fmaf(s_l[g2 * G + h], s_w[g2 * G + h], ls);
        }
        if (one_split) {
            store_out(out + idx, a / ls);
        } else {
            st_agent(rec + (size_t)h * (D + 2) + d, a);
            if (d == 0) {
                st_agent(rec + (size_t)h * (D + 2) + D, mn);
                st_agent(rec + (size_t)h * (D + 2) + D + 1, ls);
            }
        }
    }
    if constexpr (FEAT) {
        // Second pass (one workgroup per row): weight of key i for head h = 2^(s_i - M_h) / L_h with the
        // merged maximum M_h and the exact (unrounded) normaliser L_h.  Every live slot gains its weight
        // in the chunk plane and in the windows that reach back to this step; the slot appended at this
        // step starts all six planes afresh.
        // exact normaliser partials: the bf16 D = 128 path keeps them apart from the rounded ones it uses for P.V
        const float* s_lx = C::PVM && !C::SPLIT_P ? smem + C::LX_OFFSET : s_l;
        float* s_invL = smem + C::LX_OFFSET + NG * G;
        if (tid < G) {
            float ls = 0.f;
#pragma unroll 8
            for (int g2 = 0; g2 < NG; ++g2) ls = fmaf(s_lx[g2 * G + tid], s_w[g2 * G + tid], ls);
            s_invL[tid] = 1.0f / ls;
        }
        __syncthreads();  // also: the logits stored above by other waves of this workgroup are visible
        const float* lg_row = P.logit + (size_t)row * P.cap * GP;
        float* frow = P.feat + (size_t)row * FEAT_PLANES * P.cap * GP;
        constexpr int Q4 = GP / 4;
        const size_t pl4 = (size_t)P.cap * Q4;  // float4 units per plane
        const bool on8 = P.chunk_pos >= P.chunk_len - 8, on16 = P.chunk_pos >= P.chunk_len - 16,
                   on32 = P.chunk_pos >= P.chunk_len - 32;
        const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
        // four units (slot, 4 heads) per thread and pass, all loads issued before the first use
        constexpr int U = 4;
        const int units = n * Q4;
        const int h0 = (tid % Q4) * 4;  // THREADS is a multiple of Q4: a thread keeps its head quad
        float4 mq, iq;                  // maxima and 1 / normalisers of this thread's heads
        mq.x = h0 + 0 < G ? s_M[h0 + 0] : 0.f;  iq.x = h0 + 0 < G ? s_invL[h0 + 0] : 0.f;
        mq.y = h0 + 1 < G ? s_M[h0 + 1] : 0.f;  iq.y = h0 + 1 < G ? s_invL[h0 + 1] : 0.f;
        mq.z = h0 + 2 < G ? s_M[h0 + 2] : 0.f;  iq.z = h0 + 2 < G ? s_invL[h0 + 2] : 0.f;
        mq.w = h0 + 3 < G ? s_M[h0 + 3] : 0.f;  iq.w = h0 + 3 < G ? s_invL[h0 + 3] : 0.f;
        const float4* lg4 = reinterpret_cast<const float4*>(lg_row);
        float4* f4 = reinterpret_cast<float4*>(frow);
        for (int t0 = tid; t0 < units; t0 += C::THREADS * U) {
            float4 s[U], w[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int t = min(t0 + u * C::THREADS, units - 1);
                s[u] = lg4[t];
                w[u] = f4[FEAT_WL * pl4 + t];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int t = t0 + u * C::THREADS;
                if (t >= units) break;
                // padded heads: their logits are 0 and iq is 0, so p = 0
                const float4 p = make_float4(exp2f(s[u].x - mq.x) * iq.x, exp2f(s[u].y - mq.y) * iq.y,
                                             exp2f(s[u].z - mq.z) * iq.z, exp2f(s[u].w - mq.w) * iq.w);
                float4* f = f4 + t;
                if (t / Q4 == new_slot) {
                    f[FEAT_W8 * pl4] = keep_if(on8, p);
                    f[FEAT_W16 * pl4] = keep_if(on16, p);
                    f[FEAT_W32 * pl4] = keep_if(on32, p);
                    f[FEAT_WL * pl4] = p;
                    f[FEAT_CUM * pl4] = zero;
                    f[FEAT_DEC * pl4] = zero;
                } else {
                    f[FEAT_WL * pl4] = make_float4(w[u].x + p.x, w[u].y + p.y, w[u].z + p.z, w[u].w + p.w);
                    if (on32) feat_add(f + FEAT_W32 * pl4, p);
                    if (on16) feat_add(f + FEAT_W16 * pl4, p);
                    if (on8) feat_add(f + FEAT_W8 * pl4, p);
                }
            }
        }
    }
    finish(!one_split);
}

// fp32, short rows that all fit the chip: a workgroup of sixteen wavefronts for every query head, rows not split.  The vector instructions of
// the group's heads are what such a step waits for (one head on four wavefronts takes 4.3 us at two rows of 144 pairs of head_dim 64, eight
// take 7.6, and of that 1.6 for merging splits); K and V are read once per head, from the L2.  How long rows may be for it depends on how full
// the chip is: few rows split are spread over more CUs, many are not.  us a step with splits and so, from a sweep of 1 to 256 rows and seven to
// ten lengths a group size (the lines lie where the two are equal, or below):
//   D = 64   g = 1   8 rows of 350 5.4 and 5.4, 32 of 500 6.4 and 6.0, 128 of 390 7.4 and 5.8, 64 of 858 7.9 and 8.0
//            g = 2   8 rows of 265 5.6 and 5.4, of 450 5.7 and 6.0, 32 of 450 6.5 and 6.3;  g = 3  8 of 335 6.0 and 5.7, of 468 6.1 and 6.4
//            g = 4   8 rows of 567 7.2 and 6.6, of 810 7.2 and 7.7, 64 of 810 9.2 and 8.8;  g = 8  8 of 1370 12.1 and 10.1
//   D = 128  g = 1   8 rows of 125 5.0 and 4.7, of 200 5.1 and 5.4, 32 of 220 5.9 and 5.6, 128 of 250 8.3 and 6.8
//            g = 2   8 rows of 150 5.5 and 5.5, of 255 5.7 and 6.3, 128 of 300 11.1 and 8.6;  g = 3  8 of 350 7.5 and 7.0, of 500 7.8 and 8.5
//            g = 4   8 rows of 350 8.0 and 7.0, of 700 9.3 and 9.8, 64 of 700 13.8 and 12.9;  g = 8  8 of 1500 19.1 and 16.6, of 1875 19.3 and 19.6
// The heads of a row share an XCD's L2 where the rows are a multiple of eight; otherwise the copies have to fit all of them together (D = 128, g =
// 4, 21 rows of 350 8.5 and 7.8, of 489 9.1 and 10.5).
static bool attn_by_head(int rows, int g, int max_len, int head_dim) {
    if ((long long)rows * g > 256) return false;
    static constexpr short kLongest[2][3][4] = {{{390, 340, 340, 600}, {500, 450, 570, 690}, {800, 660, 830, 810}},    // head_dim 64: up to 15, 63, 256
                                                {{140, 140, 380, 450}, {250, 200, 420, 600}, {350, 300, 800, 900}}};   // rows by the heads of a group
    const int longest = g <= 4 ? kLongest[head_dim == 128][rows < 16 ? 0 : rows < 64 ? 1 : 2][g - 1] : head_dim == 64 ? 250 + 140 * g : 200 * g - 100;
    return max_len <= longest && (rows % 8 == 0 || (long long)rows * g * max_len * head_dim <= (1 << 22));
}

template <typename T, int D, int G>
static fk_status attn_launch(const fk_cache_desc* d, const AttnParams& base, int max_len, void* ws, hipStream_t st) {
    using C = AttnCfg<T, D, G>;
    {
        if (base.feat) {  // feature variant: one workgroup per row, the logit scratch sits behind the counters
            AttnParams P = base;
            P.split_len = (d->capacity + 31) / 32 * 32;  // the whole row, whatever max_len says
            P.nsplit = 1;
            P.row_cnt = reinterpret_cast<uint32_t*>(ws);
            P.rec = nullptr;
            P.logit = reinterpret_cast<float*>(reinterpret_cast<char*>(ws) + attn_counter_bytes(d));
            const int frows = d->batch * d->n_kv_heads;
            if constexpr (C::PVM) {
                if ((d->flags & FK_CACHE_COLD) || (D == 128 && (size_t)frows * max_len * D * sizeof(T) * 2 >= kStreamNtBytes)) {
                    auto kern = attn_kernel<T, D, G, true, true>;
                    static bool lds_ok[kMaxDevices] = {};
                    if (!allow_dynamic_lds((const void*)kern, C::LDS_BYTES_FEAT, lds_ok)) return FK_ERR_LAUNCH;
                    hipLaunchKernelGGL(kern, dim3(1, frows), dim3(C::THREADS), C::LDS_BYTES_FEAT, st, P);
                    return launch_status();
                }
            }
            auto kern = attn_kernel<T, D, G, true, false>;
            static bool lds_ok[kMaxDevices] = {};  // per template instantiation
            if (!allow_dynamic_lds((const void*)kern, C::LDS_BYTES_FEAT, lds_ok)) return FK_ERR_LAUNCH;
            hipLaunchKernelGGL(kern, dim3(1, frows), dim3(C::THREADS), C::LDS_BYTES_FEAT, st, P);
            return launch_status();
        }
    }
    const AttnPlan p = attn_plan(attn_shape(d), max_len);
    const int rows = d->batch * d->n_kv_heads;
    AttnParams P = base;
    P.split_len = p.split_len;
    P.nsplit = p.nsplit;
    P.rotate = p.rotate ? 1 : 0;
    P.row_cnt = reinterpret_cast<uint32_t*>(ws);
    P.rec = reinterpret_cast<float*>(reinterpret_cast<char*>(ws) + attn_counter_bytes(d));
    if constexpr (C::PVM) {
        // not cache resident (head_dim 64 with split rows: ragged ones, whose hint says more bytes than there are, lose 5 to 8 % to
        // the streamed loads, 288 rows of up to 21676 194 -> 208 us; rows of one length would gain 9 %)
        if ((d->flags & FK_CACHE_COLD) || ((D == 128 || p.nsplit == 1) && (size_t)rows * max_len * D * sizeof(T) * 2 >= kStreamNtBytes)) {
            // More rows than CUs: one workgroup per CU (LDS it does not use keeps the second one out) and the longest rows first, so
            // that a ragged batch ends everywhere at about the same time.  With all rows on the chip at once every row gets the same
            // share of the bandwidth, the longest are left alone at the end, and few workgroups cannot fill the memory system: 512
            // rows of 1024 to 32768 pairs 806 -> 693 us.  One workgroup per CU and the look-up (about 1 us each) cost rows of one
            // length a little, 512 rows of 8000 306 -> 313 us, of 4000 157 -> 156; hence the bound on the bytes, and no such order
            // where a last round of fewer than 128 workgroups would not fill the memory system (rows of one length end up there).
            P.by_length = p.nsplit == 1 && rows > 256 && rows <= 8192 && (rows % 256 == 0 || rows % 256 >= 128) && (size_t)rows * max_len * D * sizeof(T) * 2 >= ((size_t)1 << 30);
            constexpr size_t kAlone = 84 * 1024;   // more than half of a CU's 160 KB
            const size_t lds = P.by_length && C::LDS_BYTES < kAlone ? kAlone : C::LDS_BYTES;
            auto kern = attn_kernel<T, D, G, false, true>;
            static bool lds_ok[kMaxDevices] = {};
            if (!allow_dynamic_lds((const void*)kern, kAlone > C::LDS_BYTES ? kAlone : C::LDS_BYTES, lds_ok)) return FK_ERR_LAUNCH;
            hipLaunchKernelGGL(kern, dim3(p.nsplit, rows), dim3(C::THREADS), lds, st, P);
            return launch_status();
        }
    }
    if constexpr (!C::PVM) {
        if (attn_by_head(rows, G, max_len, D)) {
            using H = AttnCfg<T, D, 1, true>;
            P.split_len = (d->capacity + 31) / 32 * 32;   // the whole row, whatever max_len says
            P.nsplit = 1;
            static_assert(H::LDS_BYTES <= 64 * 1024, "within the limit that kernels have from the start");
            hipLaunchKernelGGL((attn_kernel<T, D, 1, false, false, true>), dim3(rows, G), dim3(H::THREADS), H::LDS_BYTES, st, P);
            return launch_status();
        }
    }
    auto kern = attn_kernel<T, D, G, false, false>;
    static bool lds_ok[kMaxDevices] = {};  // per template instantiation
    if (!allow_dynamic_lds((const void*)kern, C::LDS_BYTES, lds_ok)) return FK_ERR_LAUNCH;
    hipLaunchKernelGGL(kern, dim3(p.nsplit, rows), dim3(C::THREADS), C::LDS_BYTES, st, P);
    return launch_status();
}

template <typename T, int D>
static fk_status attn_dispatch_g(int g, const fk_cache_desc* d, const AttnParams& P, int max_len, void* ws, hipStream_t st) {
    switch (g) {
        case 1: return attn_launch<T, D, 1>(d, P, max_len, ws, st);
        case 2: return attn_launch<T, D, 2>(d, P, max_len, ws, st);
        case 3: return attn_launch<T, D, 3>(d, P, max_len, ws, st);
        case 4: return attn_launch<T, D, 4>(d, P, max_len, ws, st);
        case 5: return attn_launch<T, D, 5>(d, P, max_len, ws, st);
        case 6: return attn_launch<T, D, 6>(d, P, max_len, ws, st);
        case 7: return attn_launch<T, D, 7>(d, P, max_len, ws, st);
        case 8: return attn_launch<T, D, 8>(d, P, max_len, ws, st);
    }
    return FK_ERR_UNSUPPORTED;
}

static size_t feat_workspace_bytes(const fk_cache_desc* d) {
    const size_t g = d->n_q_heads / d->n_kv_heads;
    return attn_counter_bytes(d) + (size_t)d->batch * d->n_kv_heads * d->capacity * (g <= 4 ? 4 : 8) * sizeof(float);
}

static fk_status attn_entry(const fk_cache_desc* desc, AttnParams P, int max_len, float softmax_scale, void* workspace,
                            size_t workspace_bytes, void* stream) {
    if (max_len <= 0 || max_len > desc->capacity) return FK_ERR_INVALID_ARG;
    const size_t need = P.feat ? feat_workspace_bytes(desc) : fk_decode_attn_workspace(desc, max_len);
    if (!workspace || workspace_bytes < need || !aligned16(workspace)) return FK_ERR_WORKSPACE;
    const int g = desc->n_q_heads / desc->n_kv_heads;
    P.scale_log2e = softmax_scale * 1.4426950408889634f;
    P.n_kv = desc->n_kv_heads;
    P.cap = desc->capacity;
    hipStream_t st = (hipStream_t)stream;
    if (desc->dtype == FK_F32) {
        if (desc->head_dim == 64) return attn_dispatch_g<float, 64>(g, desc, P, max_len, workspace, st);
        return attn_dispatch_g<float, 128>(g, desc, P, max_len, workspace, st);
    }
    if (desc->head_dim == 64) return attn_dispatch_g<bf16_t, 64>(g, desc, P, max_len, workspace, st);
    return attn_dispatch_g<bf16_t, 128>(g, desc, P, max_len, workspace, st);
}

}  // namespace fk

using namespace fk;

extern "C" size_t fk_decode_attn_workspace(const fk_cache_desc* desc, int32_t max_len) {
    if (check_desc(desc) != FK_OK || max_len <= 0 || max_len > desc->capacity) return 0;
    // sized for the largest split count any max_len can get, so one workspace serves every call
    const size_t g = desc->n_q_heads / desc->n_kv_heads;
    return attn_counter_bytes(desc) +
           (size_t)desc->batch * desc->n_kv_heads * attn_max_splits(attn_shape(desc)) * g * (desc->head_dim + 2) * sizeof(float);
}

extern "C" fk_status fk_decode_attn(const fk_cache_desc* desc, const void* q, const void* K, const void* V,
                                    const int32_t* len, int32_t max_len, float softmax_scale, void* out,
                                    void* workspace, size_t workspace_bytes, void* stream) {
    fk_status s = check_desc(desc);
    if (s != FK_OK) return s;
    if (!q || !K || !V || !len || !out) return FK_ERR_INVALID_ARG;
    if (!aligned16(q) || !aligned16(K) || !aligned16(V) || !aligned16(out)) return FK_ERR_INVALID_ARG;
    AttnParams P = {};
    P.q = q;
    P.K = const_cast<void*>(K);
    P.V = const_cast<void*>(V);
    P.len = const_cast<int32_t*>(len);
    P.out = out;
    return attn_entry(desc, P, max_len, softmax_scale, workspace, workspace_bytes, stream);
}

extern "C" fk_status fk_decode_step(const fk_cache_desc* desc, const void* q, void* K, void* V, int32_t* pos,
                                    int32_t* len, const void* k_new, const void* v_new, const int32_t* pos_new,
                                    int32_t max_len, float softmax_scale, void* out, void* workspace,
                                    size_t workspace_bytes, void* stream) {
    fk_status s = check_desc(desc);
    if (s != FK_OK) return s;
    if (!q || !K || !V || !pos || !len || !k_new || !v_new || !pos_new || !out) return FK_ERR_INVALID_ARG;
    if (!aligned16(q) || !aligned16(K) || !aligned16(V) || !aligned16(out) || !aligned16(k_new) || !aligned16(v_new))
        return FK_ERR_INVALID_ARG;
    AttnParams P = {};
    P.q = q;
    P.K = K;
    P.V = V;
    P.pos = pos;
    P.len = len;
    P.k_new = k_new;
    P.v_new = v_new;
    P.pos_new = pos_new;
    P.out = out;
    return attn_entry(desc, P, max_len, softmax_scale, workspace, workspace_bytes, stream);
}

// ---------------------------------------------------------------------------------------------------------
// fk_decode_window: the steps of a window at once (window.hip) where that is possible, else step by step
// ---------------------------------------------------------------------------------------------------------
namespace fk {
static bool overlap(const void* a, size_t na, const void* b, size_t nb) {
    const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
    return x < y + nb && y < x + na;
}

// At once: bf16, two steps or more, every pointer as fk_decode_step wants it (otherwise the step path reports the error), and
// no buffer that the window writes shares memory with one that it reads for a later step, nor with another one that
// it writes (one step's output used as a later step's input, new rows that lie in the cache): such calls have an order.
static bool window_at_once(const fk_cache_desc* d, const void* q, const void* K, const void* V, const void* pos, const void* len,
                           const void* k, const void* v, const void* pos_seq, int32_t T, const void* out, const void* ws, const void* feat) {
    if (d->dtype != FK_BF16 || T < 2) return false;
    if (!aligned16(q) || !aligned16(K) || !aligned16(V) || !aligned16(out) || !aligned16(k) || !aligned16(v) || !pos || !len) return false;
    const size_t rows = (size_t)d->batch * d->n_kv_heads, row_bytes = (size_t)d->head_dim * 2;
    if ((size_t)T * (d->n_q_heads / d->n_kv_heads) * rows >= (size_t)1 << 27) return false;   // 32-bit counts of queries
    const size_t nq = (size_t)T * d->batch * d->n_q_heads * row_bytes, nn = (size_t)T * rows * row_bytes, nc = rows * d->capacity * row_bytes;
    const size_t np = rows * d->capacity * 4, nl = rows * 4, ns = (size_t)T * d->batch * 4;
    const size_t nf = feat ? np * kFeatPlanes * (d->n_q_heads / d->n_kv_heads <= 4 ? 4 : 8) : 0, nw = feat ? feat_workspace_bytes(d) : nl;
    // the first seven are written
    const struct { const void* p; size_t n; } buf[] = {{out, nq}, {K, nc}, {V, nc}, {pos, np}, {len, nl}, {ws, nw}, {feat, nf},
                                                       {q, nq},   {k, nn}, {v, nn}, {pos_seq, ns}};
    for (int i = 0; i < 7; ++i)
        for (int j = i + 1; j < 11; ++j)
            if (buf[i].n && buf[j].n && overlap(buf[i].p, buf[i].n, buf[j].p, buf[j].n)) return false;
    return true;
}

// Whether the steps at once are the faster way (the results are the same).  A workgroup, one per CU, walks its row alone whatever
// the number of its steps: 2.6 us for 256 pairs (head_dim 64: 1.8) and 4.2 us for every split of a split row; a single step spreads the
// row over the chip: its bytes at 10 TB/s, 0.8 us for 256 pairs of a split, and the merge.  us, at once and one by one:
//   D = 128:  g = 8, 16 rows of 1896  T = 8: 47 and 73;  4 rows of 2393  T = 8: 56 and 77;  8 rows of 444  T = 2: 11 and 18
//   D = 64:  g = 8, 4 rows of 567  T = 4: 20 and 31;  64 rows of 1711  T = 4: 33 and 42;  g = 1, 1 row of 1682  T = 8: 37 and 46
// Of 220 such pairs (g 1 to 8; 1 to 256 rows; 100 to 8192 pairs; T 2 to 32) the slower way, by more than a tenth, at 2.
static bool window_pays(const fk_cache_desc* d, int32_t T, int32_t max_len) {
    const int g = d->n_q_heads / d->n_kv_heads, spg = 16 / g;   // 16 / g steps, or twice as many, to a workgroup
    const AttnShape shape = attn_shape(d);
    const AttnPlan p = attn_plan(shape, max_len);
    const double rows = shape.rows, groups = rows * ((T + spg - 1) / spg), rounds = groups <= 256 ? 1.0 : (groups / 2 + 255) / 256;
    const bool split = p.nsplit > 1;
    const double at_once = rounds * (6.5 + (split ? 4.2 * p.nsplit : 0.0) + max_len / 256.0 * (d->head_dim == 64 ? 1.8 : 2.6));
    const double step = 4.6 + rows * max_len * d->head_dim * 4 / 1e7 + max_len / 256.0 / p.nsplit * 0.8 + (split ? 0.7 + 0.11 * p.nsplit : 0.0);
    return T * step >= at_once;
}

static WindowParams window_params(const fk_cache_desc* d, const void* q, void* K, void* V, int32_t* pos, int32_t* len, const void* k, const void* v,
                                 const int32_t* pos_seq, int32_t T, float scale, void* out, void* ws) {
    WindowParams P = {};
    P.q_seq = q;
    P.k_seq = k;
    P.v_seq = v;
    P.K = K;
    P.V = V;
    P.pos = pos;
    P.len = len;
    P.pos_seq = pos_seq;
    P.out_seq = out;
    P.scale_log2e = scale * 1.4426950408889634f;
    P.batch = d->batch;
    P.n_kv = d->n_kv_heads;
    P.g = d->n_q_heads / d->n_kv_heads;
    P.cap = d->capacity;
    P.T = T;
    P.rows = d->batch * d->n_kv_heads;
    P.row_cnt = reinterpret_cast<uint32_t*>(ws);
    return P;
}
}  // namespace fk

extern "C" fk_status fk_decode_window(const fk_cache_desc* desc, const void* q_seq, void* K, void* V, int32_t* pos,
                                      int32_t* len, const void* k_seq, const void* v_seq, const int32_t* pos_seq,
                                      int32_t n_steps, int32_t max_len_first, float softmax_scale, void* out_seq,
                                      void* workspace, size_t workspace_bytes, void* stream) {
    fk_status s = check_desc(desc);
    if (s != FK_OK) return s;
    if (n_steps < 0 || max_len_first <= 0 || max_len_first > desc->capacity) return FK_ERR_INVALID_ARG;
    if (!q_seq || !k_seq || !v_seq || !pos_seq || !out_seq) return FK_ERR_INVALID_ARG;
    const size_t e = desc->dtype == FK_F32 ? 4 : 2;
    const size_t q_step = (size_t)desc->batch * desc->n_q_heads * desc->head_dim * e;   // bytes per step, multiples of 16
    const size_t kv_step = (size_t)desc->batch * desc->n_kv_heads * desc->head_dim * e;
    if (window_at_once(desc, q_seq, K, V, pos, len, k_seq, v_seq, pos_seq, n_steps, out_seq, workspace, nullptr) &&
        window_pays(desc, n_steps, max_len_first)) {
        const size_t need = fk_decode_attn_workspace(desc, max_len_first);
        if (!workspace || workspace_bytes < need || !aligned16(workspace)) return FK_ERR_WORKSPACE;
        WindowParams P = window_params(desc, q_seq, K, V, pos, len, k_seq, v_seq, pos_seq, n_steps, softmax_scale, out_seq, workspace);
        P.shape = attn_shape(desc);
        P.max_len_first = max_len_first;
        // (the splits of a row never get fewer as its length grows)
        const int64_t ml = (int64_t)max_len_first + n_steps - 1;
        const bool split = attn_plan(P.shape, ml > desc->capacity ? desc->capacity : (int)ml).nsplit > 1;
        return window_attn(P, split, (hipStream_t)stream);
    }
    for (int32_t t = 0; t < n_steps; ++t) {
        const int64_t ml = (int64_t)max_len_first + t;
        s = fk_decode_step(desc, static_cast<const char*>(q_seq) + t * q_step, K, V, pos, len,
                           static_cast<const char*>(k_seq) + t * kv_step, static_cast<const char*>(v_seq) + t * kv_step,
                           pos_seq + (size_t)t * desc->batch, ml > desc->capacity ? desc->capacity : (int32_t)ml, softmax_scale,
                           static_cast<char*>(out_seq) + t * q_step, workspace, workspace_bytes, stream);
        if (s != FK_OK) return s;
    }
    return FK_OK;
}

// ---------------------------------------------------------------------------------------------------------
// fk_decode_step_static: fk_decode_step for callers that cannot allocate.  The workspace (row arrival counters
// and split records) is a fixed array in the library's device image; every GPU the library runs on holds
// its own copy at its own address, looked up once per device.
// ---------------------------------------------------------------------------------------------------------
namespace fk {
static constexpr size_t kStaticScratchBytes = FK_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
static void* g_scratch_ptr[kMaxDevices] = {};  // device address of `scratch` on each device, null until looked up
static std::mutex g_scratch_mutex;

__global__ void scratch_clear_kernel(uint4* p, size_t n16) {
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += stride) p[i] = make_uint4(0, 0, 0, 0);
}

// Device address of the static scratch on the current device; on the first call on a device the address is looked
// up and the array is cleared on `st` (a fill kernel, no memset node: the caller may be capturing a graph), which
// orders the clear before the first launch that uses it.  Null on failure.
static void* static_scratch(hipStream_t st) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return nullptr;
        hipLaunchKernelGGL(scratch_clear_kernel, dim3(256), dim3(256), 0, st, reinterpret_cast<uint4*>(ptr), kStaticScratchBytes / 16);
        if (hipGetLastError() != hipSuccess) return nullptr;
        g_scratch_ptr[dev] = ptr;
    }
    return g_scratch_ptr[dev];
}
}  // namespace fk

extern "C" fk_status fk_decode_step_static(const fk_cache_desc* desc, const void* q, void* K, void* V, int32_t* pos,
                                           int32_t* len, const void* k_new, const void* v_new, const int32_t* pos_new,
                                           int32_t max_len, float softmax_scale, void* out, void* stream) {
    fk_status s = check_desc(desc);
    if (s != FK_OK) return s;
    if (max_len <= 0 || max_len > desc->capacity) return FK_ERR_INVALID_ARG;
    if (fk_decode_attn_workspace(desc, max_len) > kStaticScratchBytes) return FK_ERR_WORKSPACE;  // beyond the fixed scratch
    if (!q || !K || !V || !pos || !len || !k_new || !v_new || !pos_new || !out) return FK_ERR_INVALID_ARG;
    void* ws = static_scratch((hipStream_t)stream);
    if (!ws) return FK_ERR_LAUNCH;
    return fk_decode_step(desc, q, K, V, pos, len, k_new, v_new, pos_new, max_len, softmax_scale, out, ws, kStaticScratchBytes, stream);
}

extern "C" size_t fk_decode_step_feat_workspace(const fk_cache_desc* desc) {
    if (check_desc(desc) != FK_OK) return 0;
    return feat_workspace_bytes(desc);
}

extern "C" fk_status fk_decode_step_feat(const fk_cache_desc* desc, const void* q, void* K, void* V, int32_t* pos,
                                         int32_t* len, const void* k_new, const void* v_new, const int32_t* pos_new,
                                         int32_t max_len, float softmax_scale, float* feat, int32_t chunk_pos,
                                         int32_t chunk_len, void* out, void* workspace, size_t workspace_bytes,
                                         void* stream) {
    fk_status s = check_desc(desc);
    if (s != FK_OK) return s;
    if (!q || !K || !V || !pos || !len || !k_new || !v_new || !pos_new || !out || !feat) return FK_ERR_INVALID_ARG;
    if (!aligned16(q) || !aligned16(K) || !aligned16(V) || !aligned16(out) || !aligned16(k_new) || !aligned16(v_new) ||
        !aligned16(feat))
        return FK_ERR_INVALID_ARG;
    if (chunk_len <= 0 || chunk_pos < 0 || chunk_pos >= chunk_len) return FK_ERR_INVALID_ARG;
    AttnParams P = {};
    P.q = q;
    P.K = K;
    P.V = V;
    P.pos = pos;
    P.len = len;
    P.k_new = k_new;
    P.v_new = v_new;
    P.pos_new = pos_new;
    P.out = out;
    P.feat = feat;
    P.chunk_pos = chunk_pos;
    P.chunk_len = chunk_len;
    return attn_entry(desc, P, max_len, softmax_scale, workspace, workspace_bytes, stream);
}

// fk_decode_step_feat for the steps from chunk_pos_first to the end of a window inside one chunk, enqueued by one call
extern "C" fk_status fk_decode_window_feat(const fk_cache_desc* desc, const void* q_seq, void* K, void* V, int32_t* pos,
                                           int32_t* len, const void* k_seq, const void* v_seq, const int32_t* pos_seq,
                                           int32_t n_steps, int32_t max_len_first, float softmax_scale, float* feat,
                                           int32_t chunk_pos_first, int32_t chunk_len, void* out_seq, void* workspace,
                                           size_t workspace_bytes, void* stream) {
    fk_status s = check_desc(desc);
    if (s != FK_OK) return s;
    if (n_steps < 0 || max_len_first <= 0 || max_len_first > desc->capacity) return FK_ERR_INVALID_ARG;
    if (!q_seq || !k_seq || !v_seq || !pos_seq || !out_seq) return FK_ERR_INVALID_ARG;
    if (chunk_len <= 0 || chunk_pos_first < 0 || (int64_t)chunk_pos_first + n_steps > chunk_len) return FK_ERR_INVALID_ARG;
    // At once where the buffers allow it and the two floats per query fit the logit scratch, but two steps of short rows (the second
    // launch: 8 rows of 300 pairs 21 us against 18, 256 rows of 1024 60 against 58, 128 rows of 2048 58 against 64; three steps 22
    // against 26, 65 against 87 and 58 against 95).
    const int g = desc->n_q_heads / desc->n_kv_heads;
    if (desc->head_dim == 128 && feat && aligned16(feat) && (n_steps > 2 || max_len_first >= 2048) && (int64_t)n_steps * g * 2 <= (int64_t)desc->capacity * (g <= 4 ? 4 : 8) &&
        window_at_once(desc, q_seq, K, V, pos, len, k_seq, v_seq, pos_seq, n_steps, out_seq, workspace, feat)) {
        if (!workspace || workspace_bytes < feat_workspace_bytes(desc) || !aligned16(workspace)) return FK_ERR_WORKSPACE;
        WindowParams P = window_params(desc, q_seq, K, V, pos, len, k_seq, v_seq, pos_seq, n_steps, softmax_scale, out_seq, workspace);
        P.stat = reinterpret_cast<float2*>(static_cast<char*>(workspace) + attn_counter_bytes(desc));
        P.feat = feat;
        P.chunk_pos = chunk_pos_first;
        P.chunk_len = chunk_len;
        const int64_t ml = (int64_t)max_len_first + n_steps - 1;
        return window_feat(P, ml > desc->capacity ? desc->capacity : (int)ml, (hipStream_t)stream);
    }
    const size_t e = desc->dtype == FK_F32 ? 4 : 2;
    const size_t q_step = (size_t)desc->batch * desc->n_q_heads * desc->head_dim * e;   // bytes per step, multiples of 16
    const size_t kv_step = (size_t)desc->batch * desc->n_kv_heads * desc->head_dim * e;
    for (int32_t t = 0; t < n_steps; ++t) {
        const int64_t ml = (int64_t)max_len_first + t;
        s = fk_decode_step_feat(desc, static_cast<const char*>(q_seq) + t * q_step, K, V, pos, len,
                                static_cast<const char*>(k_seq) + t * kv_step, static_cast<const char*>(v_seq) + t * kv_step,
                                pos_seq + (size_t)t * desc->batch, ml > desc->capacity ? desc->capacity : (int32_t)ml,
                                softmax_scale, feat, chunk_pos_first + t, chunk_len,
                                static_cast<char*>(out_seq) + t * q_step, workspace, workspace_bytes, stream);
        if (s != FK_OK) return s;
    }
    return FK_OK;
}

extern "C" fk_status fk_decode_step_packed(const fk_step_args* a) {
    if (!a) return FK_ERR_INVALID_ARG;
    if (a->feat)
        return fk_decode_step_feat(&a->desc, a->q, a->K, a->V, a->pos, a->len, a->k_new, a->v_new, a->pos_new, a->max_len, a->softmax_scale,
                                   a->feat, a->chunk_pos, a->chunk_len, a->out, a->workspace, a->workspace_bytes, a->stream);
    return fk_decode_step(&a->desc, a->q, a->K, a->V, a->pos, a->len, a->k_new, a->v_new, a->pos_new, a->max_len, a->softmax_scale, a->out,
                          a->workspace, a->workspace_bytes, a->stream);
}
