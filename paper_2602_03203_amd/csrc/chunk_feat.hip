// fk_decode_window_feat on tokens that are all known when the call is made: the steps of a window at once, with the
// results of the single steps bit for bit (bf16, head_dim 128).
//
// fk_decode_step_feat reads a row's K and V once per step (one workgroup per row, 27 us per step at 128 rows of 2112 pairs).
// Here a step's arithmetic stays what it is there - the same 16x16x32 matrix products, the same tiles of 32 keys dealt to eight
// wavefronts, the same online softmax, the same merge - and what is shared between steps is the data: the sixteen rows of a
// matrix product hold SPG = 16 / g steps of the group's g heads instead of one step and zeros, a workgroup runs
// kGroups such groups on every tile it has loaded, and a launch has the workgroups of all steps.  New pairs are read from
// k_seq / v_seq, so the steps need no order among themselves.  128 rows, 2048 pairs, 128 steps: 271 + 106 us against 3.47 ms;
// bound by the vector work of the softmax (one product of 16 rows with 32 keys takes 16 matrix and some 200 vector
// instructions).  Two groups: with one the K and V tiles are read twice as often, with three the registers spill (524 us a window and
// its scores against 380).
//
// The feature planes are sums over the steps IN ORDER, one fp32 addition per step: a second launch recomputes the logits (the
// same products again: the same bits) with a pair per lane, its wavefronts walking the steps in order, so every plane is
// read and written once per window, not once per step.
#include "chunk.h"

namespace fk {

typedef __attribute__((ext_vector_type(8))) __bf16 xbf16x8_t;
typedef __attribute__((ext_vector_type(4))) float xf32x4_t;
typedef __attribute__((ext_vector_type(4))) uint32_t xu32x4_t;
union X128 {
    xu32x4_t u;
    uint32_t w[4];
    xbf16x8_t v;
};

static constexpr float kXNegBig = -1.0e30f;
static constexpr int kXWaves = 8, kXThreads = kXWaves * kWave;
static constexpr int kXD = 128, kXCH = kXD / 8;     // head_dim, 16-byte chunks of a row
static constexpr int kXKT = 32, kXKRS = 272;        // keys of a tile, padded byte stride of a K row in LDS
static constexpr int kXPS = kXKT + 8;               // bf16 row stride of a P tile
static constexpr int kGroups = 2;                   // groups of SPG steps per workgroup
// dynamic LDS: K tiles [8][32][272] bytes (a wavefront's partial accumulator [16][128] reuses its own), P tiles
// [8][kGroups][16][40] bf16, then m, l, exact l, weights [8][16] floats each
static constexpr size_t kXKBytes = (size_t)kXWaves * kXKT * kXKRS, kXPBytes = (size_t)kXWaves * kGroups * 16 * kXPS * 2;
static constexpr size_t kXLds = kXKBytes + kXPBytes + 4 * sizeof(float) * kXWaves * 16;

__device__ __forceinline__ float xrow16_max(float v) {
    v = fmaxf(v, dpp_f<DPP_QUAD_XOR1>(v));
    v = fmaxf(v, dpp_f<DPP_QUAD_XOR2>(v));
    v = fmaxf(v, dpp_f<DPP_ROW_HALF_MIRROR>(v));
    v = fmaxf(v, dpp_f<DPP_ROW_MIRROR>(v));
    return v;
}

__global__ __launch_bounds__(kXThreads, 2) void window_feat_attn_kernel(const ChunkParams P, int spg, int blocks) {
    // the workgroups of one row on one XCD (blocks are dealt to the eight XCDs round robin): they share its L2
    const int row = (int)(blockIdx.x / 8 / blocks) * 8 + (int)(blockIdx.x % 8), blk = (int)(blockIdx.x / 8) % blocks;
    if (row >= P.rows) return;
    const int b = row / P.n_kv, hkv = row % P.n_kv, G = P.g;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave, n16 = lane & 15, quad = lane >> 4;
    const int n0 = min(max(P.len[row], 0), P.cap), n1 = min(n0 + P.T, P.cap);

    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    unsigned char* my_k = smem + (size_t)wave * kXKT * kXKRS;
    uint16_t* my_pb = reinterpret_cast<uint16_t*>(smem + kXKBytes) + (size_t)wave * kGroups * 16 * kXPS;
    float* s_m = reinterpret_cast<float*>(smem + kXKBytes + kXPBytes);   // [8][16]
    float *s_l = s_m + kXWaves * 16, *s_lx = s_l + kXWaves * 16, *s_w = s_lx + kXWaves * 16;
    __shared__ int s_bad;
    __shared__ __attribute__((aligned(16))) unsigned char s_q[kGroups * 16 * kXKRS];

    const xu32x4_t* Kr = reinterpret_cast<const xu32x4_t*>(P.K) + (size_t)row * P.cap * kXCH;
    const xu32x4_t* Vr = reinterpret_cast<const xu32x4_t*>(P.V) + (size_t)row * P.cap * kXCH;
    const xu32x4_t* kn = reinterpret_cast<const xu32x4_t*>(P.k_seq) + (size_t)row * kXCH;
    const xu32x4_t* vn = reinterpret_cast<const xu32x4_t*>(P.v_seq) + (size_t)row * kXCH;
    const size_t new_stride = (size_t)P.rows * kXCH;
    if (tid == 0) s_bad = 0;
    if (blk == 0) {   // append: slots [n0, n1) are read by nobody in this launch
        if (tid == 0) P.row_cnt[row] = 0;   // for the second launch (the workspace comes uninitialised)
        xu32x4_t* Kw = reinterpret_cast<xu32x4_t*>(P.K) + ((size_t)row * P.cap + n0) * kXCH;
        xu32x4_t* Vw = reinterpret_cast<xu32x4_t*>(P.V) + ((size_t)row * P.cap + n0) * kXCH;
        for (int i = tid; i < (n1 - n0) * kXCH; i += kXThreads) {
            const int t = i / kXCH, ch = i % kXCH;
            Kw[i] = kn[t * new_stride + ch];
            Vw[i] = vn[t * new_stride + ch];
        }
        for (int t = tid; t < n1 - n0; t += kXThreads) P.pos[(size_t)row * P.cap + n0 + t] = P.pos_seq[(size_t)t * P.batch + b];
    }

    // matrix row r of group k: step (blk * kGroups + k) * spg + r / G, head r % G
    const int t_first = blk * kGroups * spg, t_last = min(t_first + kGroups * spg, P.T) - 1;
    auto step_of = [&](int k, int r) { return t_first + k * spg + r / G; };
    auto live = [&](int k, int r) { return r < spg * G && step_of(k, r) < P.T; };
    auto q_row = [&](int k, int r) { return (((size_t)min(step_of(k, r), P.T - 1) * P.batch + b) * P.n_kv + hkv) * G + r % G; };
    const int n_max = min(n0 + t_last + 1, P.cap);   // keys of the last step
    int lim[kGroups][4];                             // keys that this lane's result rows quad * 4 + i see
    float m_run[kGroups][4], l_run[kGroups][4], lx_run[kGroups][4];
    xf32x4_t o[kGroups][8];
#pragma unroll
    for (int k = 0; k < kGroups; ++k) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            lim[k][i] = live(k, quad * 4 + i) ? min(n0 + step_of(k, quad * 4 + i) + 1, P.cap) : 0;
            m_run[k][i] = kXNegBig;
            l_run[k][i] = lx_run[k][i] = 0.f;
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) o[k][e] = (xf32x4_t){0.f, 0.f, 0.f, 0.f};
    }

    for (int i = tid; i < kGroups * 16 * kXCH; i += kXThreads) {   // the queries, for all wavefronts
        const int k = i / (16 * kXCH), r = i / kXCH % 16, ch = i % kXCH;
        const xu32x4_t q = reinterpret_cast<const xu32x4_t*>(P.q_seq)[q_row(k, r) * kXCH + ch];
        *reinterpret_cast<xu32x4_t*>(s_q + (k * 16 + r) * kXKRS + ch * 16) = live(k, r) ? q : xu32x4_t{0, 0, 0, 0};
    }
    __syncthreads();

    const int ntiles = (n_max + kXKT - 1) / kXKT;
    // The next tile's K is fetched a tile ahead, V while the tile's logits and weights are formed.
    X128 kr[8], vr[8];   // lane (quad, n16): key base + quad * 8 + u, 16-byte chunk n16
    auto fetch = [&](const xu32x4_t* cache, const xu32x4_t* fresh, int base, X128 (&x)[8]) {
        if (base + kXKT <= n0) {
#pragma unroll
            for (int u = 0; u < 8; ++u) x[u].u = cache[(size_t)(base + quad * 8 + u) * kXCH + n16];
        } else {
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int kc = min(base + quad * 8 + u, n_max - 1);
                if (kc < n0) x[u].u = cache[(size_t)kc * kXCH + n16];
                else x[u].u = fresh[(size_t)(kc - n0) * new_stride + n16];
            }
        }
    };
    if (wave < ntiles) fetch(Kr, kn, wave * kXKT, kr);
    for (int t = wave; t < ntiles; t += kXWaves) {
        const int base = t * kXKT;
#pragma unroll
        for (int u = 0; u < 8; ++u) *reinterpret_cast<xu32x4_t*>(my_k + (quad * 8 + u) * kXKRS + n16 * 16) = kr[u].u;
        fetch(Vr, vn, base, vr);
        if (t + kXWaves < ntiles) fetch(Kr, kn, base + kXWaves * kXKT, kr);
        __builtin_amdgcn_wave_barrier();
        const bool partial = base + kXKT > min(n0 + t_first + 1, P.cap);   // some step does not see the whole tile
#pragma unroll
        for (int k = 0; k < kGroups; ++k) {
            xf32x4_t c[2];
            c[0] = c[1] = (xf32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                X128 qa;
                qa.u = *reinterpret_cast<const xu32x4_t*>(s_q + (k * 16 + n16) * kXKRS + (ks * 4 + quad) * 16);
#pragma unroll
                for (int nt = 0; nt < 2; ++nt) {
                    X128 kb;
                    kb.u = *reinterpret_cast<const xu32x4_t*>(my_k + (nt * 16 + n16) * kXKRS + (ks * 4 + quad) * 16);
                    c[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qa.v, kb.v, c[nt], 0, 0, 0);
                }
            }
            bool in[2][4], changed = false;
            float x[3][4];   // arguments of the exponentials: both keys of a row, and its correction
            float lo = 0.f;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                in[0][i] = !partial || base + n16 < lim[k][i];
                in[1][i] = !partial || base + 16 + n16 < lim[k][i];
                const float s0 = in[0][i] ? c[0][i] * P.scale_log2e : kXNegBig, s1 = in[1][i] ? c[1][i] * P.scale_log2e : kXNegBig;
                const float mn = fmaxf(m_run[k][i], xrow16_max(fmaxf(s0, s1)));
                changed |= mn > m_run[k][i];
                x[0][i] = s0 - mn;
                x[1][i] = s1 - mn;
                x[2][i] = m_run[k][i] - mn;
                lo = fminf(lo, fminf(x[0][i], fminf(x[1][i], x[2][i])));
                m_run[k][i] = mn;
            }
            if (__any(lo < -126.f)) {   // exp2f's way round denormal results, only where there can be one
#pragma unroll
                for (int j = 0; j < 3; ++j)
#pragma unroll
                    for (int i = 0; i < 4; ++i) x[j][i] = exp2f(x[j][i]);
            } else {
#pragma unroll
                for (int j = 0; j < 3; ++j)
#pragma unroll
                    for (int i = 0; i < 4; ++i) x[j][i] = __builtin_amdgcn_exp2f(x[j][i]);
            }
            uint16_t* pb = my_pb + k * 16 * kXPS;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float e0 = in[0][i] ? x[0][i] : 0.f, e1 = in[1][i] ? x[1][i] : 0.f;   // 0 also where a step sees none of the tile
                const uint32_t u0 = __float_as_uint(e0) + 0x8000u, u1 = __float_as_uint(e1) + 0x8000u;
                l_run[k][i] = fmaf(l_run[k][i], x[2][i], __uint_as_float(u0 & 0xffff0000u)) + __uint_as_float(u1 & 0xffff0000u);
                lx_run[k][i] = fmaf(lx_run[k][i], x[2][i], e0) + e1;
                pb[(quad * 4 + i) * kXPS + n16] = (uint16_t)(u0 >> 16);
                pb[(quad * 4 + i) * kXPS + 16 + n16] = (uint16_t)(u1 >> 16);
            }
            if (__any(changed)) {
#pragma unroll
                for (int e = 0; e < 8; ++e)
#pragma unroll
                    for (int i = 0; i < 4; ++i) o[k][e][i] *= x[2][i];
            }
        }
        if (base + kXKT > n0) {
            // A step that does not see a pair gives it weight 0, which must not meet an infinity or a NaN of a new value: those
            // count as 0 here and are added back at the end for the steps that do see them (rare).
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                if (base + quad * 8 + u < n0) continue;
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    if ((vr[u].w[w] & 0x7f80u) == 0x7f80u) {
                        s_bad = 1;
                        vr[u].w[w] &= 0xffff0000u;
                    }
                    if ((vr[u].w[w] & 0x7f800000u) == 0x7f800000u) {
                        s_bad = 1;
                        vr[u].w[w] &= 0xffffu;
                    }
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
        // B operand of P.V: tile e = channel n16 * 8 + e over this lane's 8 keys (8x8 transpose in registers)
        X128 pa[kGroups];
#pragma unroll
        for (int k = 0; k < kGroups; ++k) pa[k].u = *reinterpret_cast<const xu32x4_t*>(my_pb + k * 16 * kXPS + n16 * kXPS + quad * 8);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;
            X128 vb;
#pragma unroll
            for (int w = 0; w < 4; ++w) vb.w[w] = __builtin_amdgcn_perm(vr[2 * w + 1].w[e >> 1], vr[2 * w].w[e >> 1], sel);
#pragma unroll
            for (int k = 0; k < kGroups; ++k) o[k][e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pa[k].v, vb.v, o[k][e], 0, 0, 0);
        }
        __builtin_amdgcn_wave_barrier();
    }

    // ---- merge the wavefronts' partials, one group after the other -------------------------------------------
#pragma unroll
    for (int k = 0; k < kGroups; ++k) {
        float* dst = reinterpret_cast<float*>(my_k);   // [16][128]: the loop is over
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = quad * 4 + i;
            const float ls = group_sum<16>(l_run[k][i]), lxs = group_sum<16>(lx_run[k][i]);
            *reinterpret_cast<float4*>(dst + r * kXD + n16 * 8) = make_float4(o[k][0][i], o[k][1][i], o[k][2][i], o[k][3][i]);
            *reinterpret_cast<float4*>(dst + r * kXD + n16 * 8 + 4) = make_float4(o[k][4][i], o[k][5][i], o[k][6][i], o[k][7][i]);
            if (n16 == 0) {
                s_m[wave * 16 + r] = m_run[k][i];
                s_l[wave * 16 + r] = ls;
                s_lx[wave * 16 + r] = lxs;
            }
        }
        __syncthreads();
        if (tid < kXWaves * 16) {   // weight of every partial; row maximum and exact normaliser for the second launch
            const int r = tid % 16;
            float mn = kXNegBig;
#pragma unroll
            for (int g2 = 0; g2 < kXWaves; ++g2) mn = fmaxf(mn, s_m[g2 * 16 + r]);
            s_w[tid] = exp2f(s_m[tid] - mn);
            if (tid < 16 && live(k, r)) {
                float ls = 0.f;
#pragma unroll
                for (int g2 = 0; g2 < kXWaves; ++g2) ls = fmaf(s_lx[g2 * 16 + r], exp2f(s_m[g2 * 16 + r] - mn), ls);
                P.stat[((size_t)row * P.T + step_of(k, r)) * G + r % G] = make_float2(mn, 1.0f / ls);
            }
        }
        __syncthreads();
        for (int idx = tid; idx < 16 * kXD; idx += kXThreads) {
            const int r = idx / kXD, d = idx % kXD;
            if (!live(k, r)) break;   // rows ascend with idx
            float a = 0.f, ls = 0.f;
#pragma unroll
            for (int g2 = 0; g2 < kXWaves; ++g2) a = fmaf(reinterpret_cast<const float*>(smem + (size_t)g2 * kXKT * kXKRS)[r * kXD + d], s_w[g2 * 16 + r], a);
#pragma unroll
            for (int g2 = 0; g2 < kXWaves; ++g2) ls = fmaf(s_l[g2 * 16 + r], s_w[g2 * 16 + r], ls);
            if (s_bad) {   // infinities and NaN among the new values: p v is infinite or NaN whatever the weight p is
                for (int t = 0; t <= step_of(k, r) && t < n1 - n0; ++t) {
                    const uint32_t x = reinterpret_cast<const uint16_t*>(vn + (size_t)t * new_stride)[d];
                    if ((x & 0x7f80u) == 0x7f80u) a += __uint_as_float(x << 16);
                }
            }
            store_out(reinterpret_cast<bf16_t*>(P.out_seq) + q_row(k, r) * kXD + d, a / ls);
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------------------------------------
// The planes.  A wavefront owns 32 keys (two tiles of a 16x16x32 product, K as the B operand in registers for the whole walk) and
// takes 16 padded queries at a time, GP heads of SPT = 16 / GP steps, from LDS.  Matrix row r is head r / SPT, step r % SPT:
// the four results of a lane belong to one key and to HPL = 4 / SPT heads, their steps in order.
// ---------------------------------------------------------------------------------------------------------
static constexpr int kFeatQ = 64;   // padded queries per staged block

template <int GP>
__global__ __launch_bounds__(kXThreads) void window_feat_planes_kernel(const ChunkParams P) {
#pragma clang fp contract(off)   // a step's weight is rounded before it is added, as in the single steps
    constexpr int SPT = 16 / GP, HPL = 4 / SPT, QRS = kXKRS;
    constexpr int LD = kFeatQ * kXCH / kXThreads;
    const int row = blockIdx.y, b = row / P.n_kv, hkv = row % P.n_kv, G = P.g, T = P.T;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave, n16 = lane & 15, quad = lane >> 4;
    const int n0 = min(max(P.len[row], 0), P.cap), n1 = min(n0 + T, P.cap);
    // steps from which the windows of the last 8, 16 and 32 queries of the chunk are open
    const int on8 = P.chunk_len - 8 - P.chunk_pos, on16 = on8 - 8, on32 = on8 - 24;

    __shared__ __attribute__((aligned(16))) unsigned char s_q[2][kFeatQ * QRS];
    __shared__ __attribute__((aligned(16))) float s_max[2][kFeatQ], s_inv[2][kFeatQ];   // of every padded query, in matrix row order
    const xu32x4_t* Kr = reinterpret_cast<const xu32x4_t*>(P.K) + (size_t)row * P.cap * kXCH;
    const float2* stat = P.stat + (size_t)row * T * G;
    float* feat = P.feat + (size_t)row * kFeatPlanes * P.cap * GP;
    const size_t plane = (size_t)P.cap * GP;

    for (int k0 = blockIdx.x * (kXWaves * 32); k0 < n1; k0 += gridDim.x * (kXWaves * 32)) {
        const int kb = k0 + wave * 32;
        X128 kreg[2][4];
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) kreg[nt][ks].u = Kr[(size_t)min(kb + nt * 16 + n16, n1 - 1) * kXCH + ks * 4 + quad];
        // this lane's sums: key kb + nt * 16 + n16, head quad * HPL + h; a new pair's start from zero
        float wl[2][HPL], w32[2][HPL], w16[2][HPL], w8[2][HPL];
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
#pragma unroll
            for (int h = 0; h < HPL; ++h) {
                const int key = kb + nt * 16 + n16;
                const float* f = feat + (size_t)min(key, n1 - 1) * GP + quad * HPL + h;
                const bool old = key < n0;
                wl[nt][h] = old ? f[3 * plane] : 0.f;
                w32[nt][h] = old && T > on32 ? f[2 * plane] : 0.f;
                w16[nt][h] = old && T > on16 ? f[plane] : 0.f;
                w8[nt][h] = old && T > on8 ? f[0] : 0.f;
            }
        xu32x4_t qr[LD];
        float2 st;
        // padded query x of a block: 16-row tile x / 16, matrix row x % 16
        auto fetch = [&](int t0) {
#pragma unroll
            for (int i = 0; i < LD; ++i) {
                const int x = (tid + i * kXThreads) / kXCH, h = (x % 16) / SPT, t = t0 + x / 16 * SPT + x % SPT;
                const size_t off = (((size_t)min(t, T - 1) * P.batch + b) * P.n_kv + hkv) * G + min(h, G - 1);
                const xu32x4_t q = reinterpret_cast<const xu32x4_t*>(P.q_seq)[off * kXCH + tid % kXCH];
                qr[i] = h < G ? q : xu32x4_t{0, 0, 0, 0};
            }
            const int x = tid % kFeatQ, h = (x % 16) / SPT, t = t0 + x / 16 * SPT + x % SPT;
            st = stat[(size_t)min(t, T - 1) * G + min(h, G - 1)];
            if (t >= T || h >= G) st = make_float2(0.f, 0.f);   // padding: weight 0
        };
        auto stage = [&](int buf) {
#pragma unroll
            for (int i = 0; i < LD; ++i)
                *reinterpret_cast<xu32x4_t*>(s_q[buf] + (tid + i * kXThreads) / kXCH * QRS + tid % kXCH * 16) = qr[i];
            if (tid < kFeatQ) {
                s_max[buf][tid] = st.x;
                s_inv[buf][tid] = st.y;
            }
        };
        constexpr int TB = kFeatQ / GP;   // steps of a block
        const int t_lo = k0 > n0 ? (k0 - n0) / TB * TB : 0;   // the first block that any of this workgroup's keys takes part in
        fetch(t_lo);
        stage(0);
        __syncthreads();
        for (int tb = t_lo, buf = 0; tb < T; tb += TB, buf ^= 1) {
            const bool more = tb + TB < T;
            if (more) fetch(tb + TB);
#pragma unroll
            for (int qt = 0; qt < kFeatQ / 16; ++qt) {
                const int t0 = tb + qt * SPT;     // first step of the tile
                X128 a[4];
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) a[ks].u = *reinterpret_cast<const xu32x4_t*>(s_q[buf] + (qt * 16 + n16) * QRS + (ks * 4 + quad) * 16);
                const float4 mx = *reinterpret_cast<const float4*>(&s_max[buf][qt * 16 + quad * 4]);
                const float4 iv = *reinterpret_cast<const float4*>(&s_inv[buf][qt * 16 + quad * 4]);
                const float m4[4] = {mx.x, mx.y, mx.z, mx.w}, i4[4] = {iv.x, iv.y, iv.z, iv.w};
                const bool plain = kb + 32 <= n0 + t0 + 1 && t0 + SPT <= min(on32, T);   // nothing hidden, no window open
#pragma unroll
                for (int nt = 0; nt < 2; ++nt) {
                    xf32x4_t c = (xf32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int ks = 0; ks < 4; ++ks) c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[ks].v, kreg[nt][ks].v, c, 0, 0, 0);
                    float x[4], lo = 0.f;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        x[i] = c[i] * P.scale_log2e - m4[i];
                        lo = fminf(lo, x[i]);
                    }
                    if (__any(lo < -126.f)) {   // exp2f's way round denormal results, only where there can be one
#pragma unroll
                        for (int i = 0; i < 4; ++i) x[i] = exp2f(x[i]);
                    } else {
#pragma unroll
                        for (int i = 0; i < 4; ++i) x[i] = __builtin_amdgcn_exp2f(x[i]);
                    }
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int h = i / SPT, t = t0 + i % SPT;   // element i: matrix row quad * 4 + i
                        const float p = x[i] * i4[i];
                        if (plain) {
                            wl[nt][h] += p;
                        } else if (kb + nt * 16 + n16 <= n0 + t && t < T) {
                            wl[nt][h] += p;
                            if (t >= on32) w32[nt][h] += p;
                            if (t >= on16) w16[nt][h] += p;
                            if (t >= on8) w8[nt][h] += p;
                        }
                    }
                }
            }
            if (more) stage(buf ^ 1);
            __syncthreads();
        }
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
#pragma unroll
            for (int h = 0; h < HPL; ++h) {
                const int key = kb + nt * 16 + n16;
                if (key >= n1) continue;
                float* f = feat + (size_t)key * GP + quad * HPL + h;
                f[3 * plane] = wl[nt][h];
                if (key >= n0 || T > on32) f[2 * plane] = w32[nt][h];
                if (key >= n0 || T > on16) f[plane] = w16[nt][h];
                if (key >= n0 || T > on8) f[0] = w8[nt][h];
                if (key >= n0) f[4 * plane] = f[5 * plane] = 0.f;
            }
    }
    // the last workgroup of the row sets its length: all of them have read it by then
    __syncthreads();
    if (tid == 0 && __hip_atomic_fetch_add(&P.row_cnt[row], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1) {
        __hip_atomic_store(&P.row_cnt[row], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        P.len[row] = n1;
    }
}

fk_status chunk_window_feat(const ChunkParams& P, int max_len, hipStream_t st) {
    const int spg = 16 / P.g, blocks = (P.T + spg * kGroups - 1) / (spg * kGroups);
    static bool lds_ok[kMaxDevices] = {};
    if (!allow_dynamic_lds((const void*)window_feat_attn_kernel, kXLds, lds_ok)) return FK_ERR_LAUNCH;
    hipLaunchKernelGGL(window_feat_attn_kernel, dim3((P.rows + 7) / 8 * 8 * blocks), dim3(kXThreads), kXLds, st, P, spg, blocks);
    if (launch_status() != FK_OK) return FK_ERR_LAUNCH;
    const dim3 grid((max_len + kXWaves * 32 - 1) / (kXWaves * 32), P.rows);
    if (P.g <= 4) hipLaunchKernelGGL(window_feat_planes_kernel<4>, grid, dim3(kXThreads), 0, st, P);
    else hipLaunchKernelGGL(window_feat_planes_kernel<8>, grid, dim3(kXThreads), 0, st, P);
    return launch_status();
}

}  // namespace fk
