// fk_decode_window on tokens that are all known when the call is made: the attention of n_steps consecutive decode steps
// as ONE contraction (Appendix A, "Problem Setup"; Section 3.1 for the appends).
//
// Step t attends over the slots [0, min(n0 + t + 1, capacity)) of a row, n0 the row's length before the window.  The
// n_steps * g queries of a row therefore share its K and V: read once per window, not once per step, and the work per
// byte is that of a matrix product.  A step by itself is bound by HBM (22 us for 139 MB at 128 rows of 2112 pairs); the
// window is bound by the matrix cores, the LDS and the exponentials, about 30 us each at 128 rows of 2112 pairs and 128 steps and
// only partly overlapped: 90 us (0.79 PFLOP/s) against 2.9 ms.
//
// Work decomposition.  A query (t, h) is number t * g + h of its row.  A workgroup of four wavefronts owns 32 * WQ queries
// of a row and walks the row's keys in tiles of KT; a wavefront owns 32 queries and KW keys of every tile (WQ * WK == 4:
// with many rows the wavefronts take different queries, WK = 1; with few rows they share the queries and split the
// keys, merged through LDS at the end, so that more workgroups exist).
//   S^T = K Q^T   v_mfma_f32_32x32x16_bf16, A = 32 keys from LDS (padded rows), B = the wavefront's queries in registers;
//                 a lane's results all belong to ONE query (lane % 32), so maximum, sum and rescaling are per lane
//   O^T = V^T P^T A = 32 channels from LDS (V transposed while it is staged, 4 keys x 8 channels per thread), B = the
//                 probabilities straight from the S^T registers: the order of the keys inside a k-step of 16 is free, so V^T
//                 is staged in the order in which the result layout holds them (keys 0-3, 8-11 | 4-7, 12-15)
// The next tile is fetched into registers while the current one is in use.  The new keys and values are read from
// k_seq / v_seq, never from the cache, so the appends (the first query tile's workgroup) need no ordering; the last
// workgroup of a row to arrive sets its length.
#include "chunk.h"
#include <cfloat>

namespace fk {

typedef __attribute__((ext_vector_type(8))) __bf16 cbf16x8_t;
typedef __attribute__((ext_vector_type(2))) __bf16 cbf16x2_t;
typedef __attribute__((ext_vector_type(2))) float cf32x2_t;
typedef __attribute__((ext_vector_type(16))) float cf32x16_t;
typedef __attribute__((ext_vector_type(4))) short cs16x4_t;
typedef __attribute__((ext_vector_type(4))) uint32_t cu32x4_t;   // (a builtin vector: arrays of HIP's uint4 end up in scratch memory)
union CB128 {
    cu32x4_t u;
    uint32_t w[4];
    cs16x4_t h[2];
    cbf16x8_t v;
};
union CB32 {
    uint32_t u;
    cbf16x2_t v;
};

static constexpr float kChunkNegBig = -1.0e30f;  // "no key seen yet"

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    CB32 r;
    r.v = __builtin_convertvector((cf32x2_t){a, b}, cbf16x2_t);
    return r.u;
}
// Transposing LDS read: sixteen lanes name four rows of sixteen 16-bit values, lane i the values (i % 4) * 4 .. + 3 of row
// i / 4, and receive a column each: lane i the i-th value of the four rows.
__device__ __forceinline__ cs16x4_t read_tr(const unsigned char* p) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) cs16x4_t*)p);
}

// WQ wavefronts take different queries, WK share the same ones and split the keys of every tile
template <int D, int WQ, int WK> struct ChunkCfg {
    static constexpr int THREADS = WQ * WK * kWave;
    static constexpr int KW = WK == 1 ? 64 : 32;       // keys of a tile per wavefront
    static constexpr int KT = KW * WK;                 // keys per tile
    static constexpr int CH = D / 8;                   // 16-byte chunks of a K or V row
    // Byte strides of the padded LDS rows (64 banks of 4 bytes).  K is read 16 bytes a lane, 16 rows at a time: 16 rows start
    // on 16 different groups of four banks.  V is read by transposing reads, four rows of 64 bytes at a time: they lie on
    // four different groups of sixteen banks.
    static constexpr int KRS = D * 2 + 16;
    static constexpr int VRS = D * 2 + 64;
    static constexpr size_t K_BYTES = (size_t)KT * KRS, V_BYTES = (size_t)KT * VRS;
    static constexpr size_t TILE_BYTES = K_BYTES + V_BYTES;
    static constexpr size_t MERGE_BYTES = WK > 1 ? (size_t)(WK - 1) * WQ * (D / 2 + 2) * kWave * 4 : 0;   // reuses the tiles
    static constexpr size_t LDS_BYTES = 2 * TILE_BYTES > MERGE_BYTES ? 2 * TILE_BYTES : MERGE_BYTES;
};

template <int D, int WQ, int WK>
__global__ __launch_bounds__((WQ * WK * kWave), (WQ * WK == 4 ? 1 : 2)) void chunk_attn_kernel(const ChunkParams P) {
    using C = ChunkCfg<D, WQ, WK>;
    constexpr int THREADS = C::THREADS, KW = C::KW, KT = C::KT, CH = C::CH, KRS = C::KRS, VRS = C::VRS;
    constexpr int NT = KW / 32;          // S^T tiles of a wavefront
    constexpr int KS = D / 16;           // k-steps of S^T
    constexpr int DT = D / 32;           // O^T tiles
    constexpr bool SPLIT_P = D == 64;    // probabilities as bf16 head + remainder (head_dim 128: rounded to bf16)
    constexpr int LD = KT * CH / THREADS;   // 16-byte loads of K, and of V, per thread and tile

    // The workgroups of one row sit on one XCD (blocks are dealt to the eight XCDs round robin) and share its L2.
    const int row = (int)(blockIdx.x / 8 / P.qtiles) * 8 + (int)(blockIdx.x % 8), qt = (int)(blockIdx.x / 8) % P.qtiles;
    if (row >= P.rows) return;
    const int b = row / P.n_kv, hkv = row % P.n_kv;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int l32 = lane & 31, half = lane >> 5;
    const int wq = wave % WQ, wk = wave / WQ;
    const int v_row = (lane & 15) >> 2, v_col = ((lane >> 4) & 1) * 32 + (lane & 3) * 8;   // this lane's part of a transposing read
    const int G = P.g, M = P.T * G;
    const int n0 = min(max(P.len[row], 0), P.cap);
    const int n1 = min(n0 + P.T, P.cap);   // after the window

    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ int s_bad;

    const cu32x4_t* Kr = reinterpret_cast<const cu32x4_t*>(P.K) + (size_t)row * P.cap * CH;
    const cu32x4_t* Vr = reinterpret_cast<const cu32x4_t*>(P.V) + (size_t)row * P.cap * CH;
    const cu32x4_t* kn = reinterpret_cast<const cu32x4_t*>(P.k_seq) + (size_t)row * CH;   // step t: + t * new_stride
    const cu32x4_t* vn = reinterpret_cast<const cu32x4_t*>(P.v_seq) + (size_t)row * CH;
    const size_t new_stride = (size_t)P.rows * CH;

    if (tid == 0) s_bad = 0;
    if (qt == 0) {   // append: slots [n0, n1) are read by nobody in this launch
        cu32x4_t* Kw = reinterpret_cast<cu32x4_t*>(P.K) + ((size_t)row * P.cap + n0) * CH;
        cu32x4_t* Vw = reinterpret_cast<cu32x4_t*>(P.V) + ((size_t)row * P.cap + n0) * CH;
        for (int i = tid; i < (n1 - n0) * CH; i += THREADS) {
            const int t = i / CH, ch = i % CH;
            Kw[i] = kn[t * new_stride + ch];
            Vw[i] = vn[t * new_stride + ch];
        }
        for (int t = tid; t < n1 - n0; t += THREADS) P.pos[(size_t)row * P.cap + n0 + t] = P.pos_seq[(size_t)t * P.batch + b];
    }

    // this lane's query
    const int q_first = qt * 32 * WQ, q_mine = q_first + wq * 32 + l32;
    const bool q_live = q_mine < M;
    const int tq = min(q_mine, M - 1) / G, hq = min(q_mine, M - 1) % G;
    const int lim = min(n0 + tq + 1, P.cap);                                          // keys it sees
    const int lim_first = min(n0 + q_first / G + 1, P.cap);                           // ... the fewest of the workgroup
    const int lim_last = min(n0 + min(q_first + 32 * WQ - 1, M - 1) / G + 1, P.cap);  // ... the most
    const size_t q_off = (((size_t)tq * P.batch + b) * P.n_kv + hkv) * G + hq;        // row of q_seq / out_seq
    CB128 q[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        q[ks].u = q_live ? reinterpret_cast<const cu32x4_t*>(P.q_seq)[q_off * CH + ks * 2 + half] : cu32x4_t{0, 0, 0, 0};
        if (P.scale_log2e < 0.f) {   // |scale| with the sign in the query: the maximum of the raw products is that of the logits
#pragma unroll
            for (int w = 0; w < 4; ++w) q[ks].w[w] ^= 0x80008000u;
        }
    }
    const float sc = P.scale_log2e == 0.f ? FLT_MIN : fabsf(P.scale_log2e);   // (never 0: a hidden key's logit is -inf)

    float m_run = kChunkNegBig, l_run = 0.f;
    cf32x16_t o[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[dt][i] = 0.f;

    cu32x4_t kr[LD], vr[LD];
    auto fetch = [&](int base) {
        if (base + KT <= n0) {   // a whole tile of cached pairs: scalar bases, constant offsets
            const cu32x4_t *kt = Kr + (size_t)base * CH, *vt = Vr + (size_t)base * CH;
#pragma unroll
            for (int i = 0; i < LD; ++i) kr[i] = kt[(uint32_t)tid + i * THREADS];
#pragma unroll
            for (int i = 0; i < LD; ++i) vr[i] = vt[(uint32_t)tid + i * THREADS];
            return;
        }
#pragma unroll
        for (int i = 0; i < LD; ++i) {
            const int item = tid + i * THREADS, ch = item % CH, key = base + item / CH, kc = min(key, n1 - 1);
            CB128 x;
            if (kc < n0) {
                kr[i] = Kr[(size_t)kc * CH + ch];
                x.u = Vr[(size_t)kc * CH + ch];
            } else {
                kr[i] = kn[(size_t)(kc - n0) * new_stride + ch];
                x.u = vn[(size_t)(kc - n0) * new_stride + ch];
            }
            // Keys that not every query of the window sees: a hidden pair has weight 0, which must not meet an infinity or a
            // NaN of a later step's value.  Those are staged as 0 and added back at the end for the queries that do see
            // them (rare); rows past the row's end are 0.
            if (key >= n0) {
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    if (key >= n1) x.w[w] = 0;
                    if ((x.w[w] & 0x7f80u) == 0x7f80u) {
                        s_bad = 1;
                        x.w[w] &= 0xffff0000u;
                    }
                    if ((x.w[w] & 0x7f800000u) == 0x7f800000u) {
                        s_bad = 1;
                        x.w[w] &= 0xffffu;
                    }
                }
            }
            vr[i] = x.u;
        }
    };
    auto stage = [&](int buf) {
        unsigned char *s_k = smem + buf * C::TILE_BYTES, *s_v = s_k + C::K_BYTES;
#pragma unroll
        for (int i = 0; i < LD; ++i) {
            const int item = tid + i * THREADS;
            *reinterpret_cast<cu32x4_t*>(s_k + (item / CH) * KRS + (item % CH) * 16) = kr[i];
            *reinterpret_cast<cu32x4_t*>(s_v + (item / CH) * VRS + (item % CH) * 16) = vr[i];
        }
    };

    __syncthreads();   // s_bad is set up
    fetch(0);
    stage(0);
    __syncthreads();
    for (int base = 0, buf = 0; base < lim_last; base += KT, buf ^= 1) {
        const bool more = base + KT < lim_last;
        if (more) fetch(base + KT);
        const unsigned char *s_k = smem + buf * C::TILE_BYTES, *s_v = s_k + C::K_BYTES;
        const int kb = base + wk * KW;             // this wavefront's keys
        const bool masked = kb + KW > lim_first;   // the same for the whole wavefront
        // S^T; element i of tile nt is key kb + nt * 32 + (i / 4) * 8 + half * 4 + i % 4
        cf32x16_t s[NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int i = 0; i < 16; ++i) s[nt][i] = 0.f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                CB128 a;
                a.u = *reinterpret_cast<const cu32x4_t*>(s_k + (wk * KW + nt * 32 + l32) * KRS + ks * 32 + half * 16);
                s[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.v, q[ks].v, s[nt], 0, 0, 0);
            }
        if (masked) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    if (kb + nt * 32 + (i / 4) * 8 + half * 4 + i % 4 >= lim) s[nt][i] = kChunkNegBig;
        }
        float mx = s[0][0];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int i = 0; i < 16; ++i) mx = fmaxf(mx, s[nt][i]);
        mx = fmaxf(mx, __shfl_xor(mx, 32)) * sc;
        // (Letting the reference point lag behind the maximum by up to 2^8 saves rescaling, 94 -> 90 us at 128 rows of 2112 pairs
        // and 128 steps, but then the largest weight is no longer exactly 1 and the error against 64 bits grows by 6 %.)
        if (__any(mx > m_run)) {
            const float mn = fmaxf(m_run, mx);
            const float corr = __builtin_amdgcn_exp2f(m_run - mn);
            l_run *= corr;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int i = 0; i < 16; ++i) o[dt][i] *= corr;
            m_run = mn;
        }
        if (masked) {   // weight 0 whatever the scale is
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    if (kb + nt * 32 + (i / 4) * 8 + half * 4 + i % 4 >= lim) s[nt][i] = -__builtin_inff();
        }
        CB128 ph[NT][2], pl[NT][2];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
            for (int i = 0; i < 16; ++i) s[nt][i] = __builtin_amdgcn_exp2f(fmaf(s[nt][i], sc, -m_run));
            if constexpr (SPLIT_P) {
#pragma unroll
                for (int i = 0; i < 16; ++i) l_run += s[nt][i];
            }
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    const float p0 = s[nt][j * 8 + 2 * w], p1 = s[nt][j * 8 + 2 * w + 1];
                    ph[nt][j].w[w] = pack_bf16(p0, p1);
                    if constexpr (SPLIT_P) {
                        pl[nt][j].w[w] = pack_bf16(p0 - bf16_lo(ph[nt][j].w[w]), p1 - bf16_hi(ph[nt][j].w[w]));
                    } else {   // the rounded weights feed the normaliser: they stay exactly normalised
                        CB32 x, one;
                        x.u = ph[nt][j].w[w];
                        one.u = 0x3f803f80u;
                        l_run = __builtin_amdgcn_fdot2_f32_bf16(x.v, one.v, l_run, false);
                    }
                }
        }
        // O^T += V^T P^T
        const unsigned char* v_base = s_v + (wk * KW + half * 4 + v_row) * VRS + v_col;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) {
                    // slots 0-3 of this lane's eight: keys 4 half + 0..3 of the k-step, slots 4-7: keys 8 + 4 half + 0..3
                    CB128 a;
                    a.h[0] = read_tr(v_base + (nt * 32 + j * 16) * VRS + dt * 64);
                    a.h[1] = read_tr(v_base + (nt * 32 + j * 16 + 8) * VRS + dt * 64);
                    o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.v, ph[nt][j].v, o[dt], 0, 0, 0);
                    if constexpr (SPLIT_P) o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.v, pl[nt][j].v, o[dt], 0, 0, 0);
                }
        if (more) stage(buf ^ 1);   // last read a tile ago, before the barrier
        __syncthreads();
    }

    // ---- merge the wavefronts that share queries -----------------------------------------------------------
    if constexpr (WK > 1) {   // (the tiles are free)
        float* mine = reinterpret_cast<float*>(smem) + (size_t)(wave - WQ) * (D / 2 + 2) * kWave + lane;
        if (wk > 0) {
            mine[0] = m_run;
            mine[kWave] = l_run;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int i = 0; i < 16; ++i) mine[(2 + dt * 16 + i) * kWave] = o[dt][i];
        }
        __syncthreads();
        if (wk == 0) {
#pragma unroll
            for (int k = 1; k < WK; ++k) {
                const float* p = reinterpret_cast<const float*>(smem) + (size_t)(k * WQ + wq - WQ) * (D / 2 + 2) * kWave + lane;
                const float mn = fmaxf(m_run, p[0]);
                const float c0 = __builtin_amdgcn_exp2f(m_run - mn), c1 = __builtin_amdgcn_exp2f(p[0] - mn);
                l_run = l_run * c0 + p[kWave] * c1;
#pragma unroll
                for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                    for (int i = 0; i < 16; ++i) o[dt][i] = o[dt][i] * c0 + p[(2 + dt * 16 + i) * kWave] * c1;
                m_run = mn;
            }
        }
    }
    if (wk == 0) {
        l_run += __shfl_xor(l_run, 32);
        if (s_bad) {   // infinities and NaN among the new values: p v is infinite or NaN whatever the weight p is
            for (int t = 0; t < n1 - n0; ++t) {
                const uint16_t* v = reinterpret_cast<const uint16_t*>(vn + (size_t)t * new_stride);
#pragma unroll
                for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const uint32_t x = v[dt * 32 + (i / 4) * 8 + half * 4 + i % 4];
                        if (t <= tq && (x & 0x7f80u) == 0x7f80u) o[dt][i] += __uint_as_float(x << 16);
                    }
            }
        }
        if (q_live) {
            const float inv = 1.0f / l_run;
            uint2* out = reinterpret_cast<uint2*>(P.out_seq) + q_off * (D / 4);
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int i4 = 0; i4 < 4; ++i4) {
                    uint2 w;
                    w.x = pack_bf16(o[dt][i4 * 4] * inv, o[dt][i4 * 4 + 1] * inv);
                    w.y = pack_bf16(o[dt][i4 * 4 + 2] * inv, o[dt][i4 * 4 + 3] * inv);
                    out[dt * 8 + i4 * 2 + half] = w;
                }
        }
    }
    // the last workgroup of the row sets its length: all of them have read it by then
    __syncthreads();
    if (tid == 0) {
        const bool last = P.qtiles == 1 || __hip_atomic_fetch_add(&P.row_cnt[row], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (uint32_t)P.qtiles - 1;
        if (last) {
            if (P.qtiles > 1) __hip_atomic_store(&P.row_cnt[row], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            P.len[row] = n1;
        }
    }
}

template <int D, int WQ, int WK>
static fk_status chunk_launch(ChunkParams P, hipStream_t st) {
    using C = ChunkCfg<D, WQ, WK>;
    P.qtiles = (P.T * P.g + 32 * WQ - 1) / (32 * WQ);
    auto kern = chunk_attn_kernel<D, WQ, WK>;
    static bool lds_ok[kMaxDevices] = {};
    if (!allow_dynamic_lds((const void*)kern, C::LDS_BYTES, lds_ok)) return FK_ERR_LAUNCH;
    hipLaunchKernelGGL(kern, dim3((P.rows + 7) / 8 * 8 * P.qtiles), dim3(C::THREADS), C::LDS_BYTES, st, P);
    return launch_status();
}

template <int D>
static fk_status chunk_pick(const ChunkParams& P, hipStream_t st) {
    auto groups = [&](int q) { return (long long)P.rows * ((P.T * P.g + q - 1) / q); };
    if (groups(256) >= 256) return chunk_launch<D, 8, 1>(P, st);
    if (groups(128) >= 256) return chunk_launch<D, 4, 2>(P, st);
    if (groups(64) >= 256) return chunk_launch<D, 2, 4>(P, st);
    return chunk_launch<D, 1, 4>(P, st);
}

fk_status chunk_window(const fk_cache_desc* d, const ChunkParams& P, hipStream_t st) {
    return d->head_dim == 64 ? chunk_pick<64>(P, st) : chunk_pick<128>(P, st);
}

}  // namespace fk
