// Windows of decode steps on tokens that are all known when the call is made (fk_decode_window, fk_decode_window_feat): the
// steps at once, with the results of the single steps bit for bit (bf16; with features head_dim 128).
//
// A single step reads a row's K and V once per step.  Here a step's arithmetic stays what it is in attn_kernel - the same 16x16x32
// matrix products, the same splits of the row, the same tiles of 32 keys dealt to eight wavefronts, the same online softmax, the
// same merges - and what is shared between steps is the data: the sixteen columns of a matrix product hold SPG = 16 / g steps of
// the group's g heads instead of one step and zeros, a workgroup runs up to GROUPS such groups on every tile it has loaded,
// and a launch has the workgroups of all steps.  New pairs are read from k_seq / v_seq, so the steps need no order among
// themselves.
//
// Operands change places against attn_kernel (logits K.Q^T, outputs V^T.P^T: the same products, transposed), so that every
// result of a lane belongs to ONE query: a row maximum takes two cross-lane steps instead of four for each of four queries, and a
// correction is one exponential instead of four.  Lane (quad, n16): query n16, keys quad * 8 .. + 7 of the tile (attn_qk_key), which are the keys
// of its share of P.V: the probabilities become an operand in the registers they are in.
//
// A step that splits a row merges the splits' records eight at a time, weighed by the largest maximum of the eight.  A workgroup here
// meets the splits one after the other, so it walks the keys once before, for the maxima alone (SPLIT).
//
// Bound by what two wavefronts a SIMD can hide of the L2's and the LDS's latency.  By the counters, its share of start and merge included, a tile
// of 32 keys with two groups of 16 queries takes 34 matrix and 304 vector instructions (349 with the weights added up by them: 4 % more time), 4100
// cycles for the two wavefronts of a SIMD; of a workgroup's 45 000 cycles 2700 are its start and 5000 its merge.  The SIMDs issue in 67 % of
// their cycles (vector 53 %, matrix 20 %, both 6 %), a wavefront waits 29 % of its time, the tiles come at 24 bytes a cycle and CU.  128 rows of
// 2048 pairs, 128 steps: 162 us with the copy that resets the lengths (0.44 PFLOP/s; 169 to 179 repeated without a pause, at a lower clock)
// against 2.9 ms step by step; with features 7 us more and 91 us for the planes.  It was 206 us with the probabilities through LDS, a merge of every group by itself with scalar reads
// (6600 cycles), a branch per group in every loop, a walk whose counter was not known to be the same for a
// wavefront (masks in every tile), and V waited for together with the next tile's K.  Measured and not kept: K as operand straight from the
// L2 (16 rows of 64 bytes a load: 218 us against 182); all of a tile's operands read ahead, higher wavefront priority around the products:
// no difference; references that follow the maximum only where it is 64 times above them, 55 of 390 vector instructions of a tile fewer: 2
// %, and split rows 5 to 12 % slower; V of the next tile behind P.V: 1 to 4 % slower.  Two groups: with one the K and V tiles are read twice as often, with three the registers spill.
//
// The feature planes are sums over the steps IN ORDER, one fp32 addition per step: a second launch recomputes the logits (the
// same products again: the same bits) with a pair per lane, its wavefronts walking the steps in order, so every plane is
// read and written once per window, not once per step.
#include "window.h"
#include <climits>

namespace fk {

typedef __attribute__((ext_vector_type(8))) __bf16 xbf16x8_t;
typedef __attribute__((ext_vector_type(4))) float xf32x4_t;
typedef __attribute__((ext_vector_type(4))) uint32_t xu32x4_t;   // (a builtin vector: arrays of HIP's uint4 end up in scratch memory)
typedef __attribute__((ext_vector_type(2))) uint32_t xu32x2_t;
union X128 {
    xu32x4_t u;
    uint32_t w[4];
    xbf16x8_t v;
};

static constexpr float kXNegBig = -1.0e30f;
static constexpr int kXWaves = 8, kXThreads = kXWaves * kWave;
static constexpr int kXKT = 32;                     // keys of a tile
static constexpr int kSplitBatch = 64;              // splits whose maxima are held at once (a multiple of the merge's eight)

// GROUPS: groups of SPG steps per workgroup, at most
template <int D, int GROUPS, bool SPLIT = false> struct WindowCfg {
    static constexpr int CH = D / 8, ET = D / 16, KS = D / 32;   // 16-byte chunks of a row, channel tiles, k-steps
    static constexpr int KRS = D * 2 + 16;                       // padded byte stride of a K or query row in LDS
    static constexpr int TERMS = D == 64 ? 3 : 1;                // bf16 terms of a probability
    static constexpr int PART = D + 4;                           // float stride of a wavefront's partial accumulator [16][D]
    // dynamic LDS: per wavefront K tile [32][KRS] bytes, later in its place the partial accumulators [JOINT][TERMS][16][PART] (JOINT: groups
    // merged at once) | queries [GROUPS][16][KRS] | m, l, exact l, weights [8][16] floats each | with splits:
    // maxima [kSplitBatch][GROUPS * 16], merged splits [GROUPS * 16][D], their maxima [GROUPS * 16] and normalisers [2][GROUPS * 16], correction and
    // weight of the split being merged [16]
    static constexpr int JOINT = !SPLIT && TERMS == 1 ? GROUPS : 1;
    static constexpr size_t K_BYTES = (size_t)kXKT * KRS, PART_BYTES = (size_t)TERMS * 16 * PART * 4;
    static constexpr size_t WAVE_BYTES = K_BYTES > JOINT * PART_BYTES ? K_BYTES : JOINT * PART_BYTES;
    static constexpr size_t Q_BYTES = (size_t)GROUPS * 16 * KRS;
    static constexpr size_t LDS_BYTES = kXWaves * WAVE_BYTES + Q_BYTES + 4 * sizeof(float) * JOINT * kXWaves * 16;
    static constexpr size_t MERGE_BYTES = sizeof(float) * (GROUPS * 16 * (kSplitBatch + D + 3) + 32);
};

// maximum / sum over the four lanes that share a query (lane % 16)
__device__ __forceinline__ float quads_max(float v) {
    auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float quads_sum(float v) {
    auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// order-preserving map of floats to unsigned words (no NaN), for maxima by LDS atomics
__device__ __forceinline__ uint32_t float_order(float f) {
    const uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : u | 0x80000000u;
}
__device__ __forceinline__ float order_float(uint32_t o) { return __uint_as_float((o & 0x80000000u) ? o ^ 0x80000000u : ~o); }

template <int D, bool FEAT, bool SPLIT, int GROUPS>
__global__ __launch_bounds__(kXThreads, 2) void window_attn_kernel(const WindowParams P, int spg, int blocks) {
    using C = WindowCfg<D, GROUPS, SPLIT>;
    constexpr int CH = C::CH, ET = C::ET, KS = C::KS, KRS = C::KRS, TERMS = C::TERMS, PART = C::PART, JOINT = C::JOINT, STAT = JOINT * kXWaves * 16;
    constexpr int KL = CH / 2;   // 16-byte K loads per lane and tile
    // The workgroups of one row sit on one XCD (blocks are dealt to the eight XCDs round robin) and share its L2; fewer than eight
    // rows are spread over the XCDs.
    const bool few = P.rows < 8;
    const int row = few ? (int)blockIdx.x % P.rows : (int)(blockIdx.x / 8 / blocks) * 8 + (int)(blockIdx.x % 8);
    const int blk = few ? (int)blockIdx.x / P.rows : (int)(blockIdx.x / 8) % blocks;
    if (row >= P.rows) return;
    const int b = row / P.n_kv, hkv = row % P.n_kv, G = P.g;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave, n16 = lane & 15, quad = lane >> 4;
    const int n0 = min(max(P.len[row], 0), P.cap), n1 = min(n0 + P.T, P.cap);

    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    unsigned char* my_k = smem + (size_t)wave * C::WAVE_BYTES;
    unsigned char* s_q = smem + kXWaves * C::WAVE_BYTES;
    float* s_m = reinterpret_cast<float*>(s_q + C::Q_BYTES);   // [JOINT][8][16]
    float *s_l = s_m + STAT, *s_lx = s_l + STAT, *s_w = s_lx + STAT;
    uint32_t* s_top = reinterpret_cast<uint32_t*>(s_w + STAT);   // [kSplitBatch][GROUPS * 16] maxima of the splits
    float* s_out = reinterpret_cast<float*>(s_top + kSplitBatch * GROUPS * 16);   // [GROUPS * 16][D]
    float *s_out_m = s_out + GROUPS * 16 * D, *s_out_l = s_out_m + GROUPS * 16, *s_c = s_out_l + 2 * GROUPS * 16, *s_cw = s_c + 16;
    __shared__ int s_bad;   // a new value that not every step of a run sees is infinite or NaN
    __shared__ int s_split_len[GROUPS * 16], s_nsplit[GROUPS * 16], s_tiles[GROUPS * 16];

    const xu32x4_t* Kr = reinterpret_cast<const xu32x4_t*>(P.K) + (size_t)row * P.cap * CH;
    const xu32x4_t* Vr = reinterpret_cast<const xu32x4_t*>(P.V) + (size_t)row * P.cap * CH;
    const xu32x4_t* kn = reinterpret_cast<const xu32x4_t*>(P.k_seq) + (size_t)row * CH;
    const xu32x4_t* vn = reinterpret_cast<const xu32x4_t*>(P.v_seq) + (size_t)row * CH;
    const size_t new_stride = (size_t)P.rows * CH;
    if (blk == 0) {   // append: slots [n0, n1) are read by nobody in this launch
        if (FEAT && tid == 0) P.row_cnt[row] = 0;   // for the second launch (that workspace comes uninitialised)
        xu32x4_t* Kw = reinterpret_cast<xu32x4_t*>(P.K) + ((size_t)row * P.cap + n0) * CH;
        xu32x4_t* Vw = reinterpret_cast<xu32x4_t*>(P.V) + ((size_t)row * P.cap + n0) * CH;
        for (int i = tid; i < (n1 - n0) * CH; i += kXThreads) {
            const int t = i / CH, ch = i % CH;
            Kw[i] = kn[t * new_stride + ch];
            Vw[i] = vn[t * new_stride + ch];
        }
        for (int t = tid; t < n1 - n0; t += kXThreads) P.pos[(size_t)row * P.cap + n0 + t] = P.pos_seq[(size_t)t * P.batch + b];
    }

    // matrix column r of group k: step t_first + k * spg + r / G, head r % G
    const int t_first = blk * GROUPS * spg, t_end = min(t_first + GROUPS * spg, P.T);
    auto step_of = [&](int k, int r) { return t_first + k * spg + r / G; };
    auto q_row = [&](int k, int r) { return (((size_t)min(step_of(k, r), P.T - 1) * P.batch + b) * P.n_kv + hkv) * G + r % G; };

    for (int i = tid; i < GROUPS * 16 * CH; i += kXThreads) {   // the queries, for all wavefronts
        const int k = i / (16 * CH), r = i / CH % 16, ch = i % CH;
        const bool live = r < spg * G && step_of(k, r) < P.T;
        const xu32x4_t q = reinterpret_cast<const xu32x4_t*>(P.q_seq)[q_row(k, r) * CH + ch];
        *reinterpret_cast<xu32x4_t*>(s_q + (k * 16 + r) * KRS + ch * 16) = live ? q : xu32x4_t{0, 0, 0, 0};
    }
    const float scale = P.scale_log2e;
    if (tid == 0) s_bad = 0;
    if constexpr (SPLIT) {   // the splits of every step; what its tile walks depend on beside their lengths
        if (tid < t_end - t_first) {
            const int t = t_first + tid;
            const AttnPlan p = attn_plan(P.shape, (int)min((long long)P.max_len_first + t, (long long)P.cap));
            s_split_len[tid] = p.nsplit > 1 ? p.split_len : INT_MAX;
            s_nsplit[tid] = p.nsplit;
            s_tiles[tid] = p.rotate ? (min(n0 + t + 1, P.cap) + kXKT - 1) / kXKT : 0;
        }
    }
    __syncthreads();
    // Counted here, where all wavefronts have the row's length, and looked at when the results are out (at the end, the answer took 1 us to come).
    uint32_t arrived = 0;
    if (!FEAT && blocks > 1 && tid == 0) arrived = __hip_atomic_fetch_add(&P.row_cnt[row], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

    // A run of steps of one plan is taken together (nearly always all of the workgroup's).  A step that does not see a pair gives it
    // weight 0, which must not meet an infinity or a NaN of a new value: where there are any, the run starts over one step at a time.
    bool together = true;
    for (int ta = t_first, tb; ta < t_end; ta = tb) {
        int split_len = INT_MAX, nsplit = 1, rotate = 0;
        tb = together ? t_end : ta + 1;
        if constexpr (SPLIT) {
            const int i = ta - t_first;
            split_len = s_split_len[i];
            nsplit = s_nsplit[i];
            rotate = s_tiles[i];
            for (int t = ta + 1; t < tb; ++t)
                if (s_split_len[t - t_first] != split_len || s_nsplit[t - t_first] != nsplit || s_tiles[t - t_first] != rotate) tb = t;
        }
        const int n_first = min(n0 + ta + 1, P.cap), n_max = min(n0 + tb, P.cap);   // keys of the first and of the last step
        const int nused = !SPLIT ? 1 : min((n_max - 1) / split_len + 1, nsplit);       // splits in use (a step with fewer sees nothing of the others)
        int lim[GROUPS];                                                            // keys that this lane's query sees
#pragma unroll
        for (int k = 0; k < GROUPS; ++k) {
            const int t = step_of(k, n16);
            lim[k] = n16 < spg * G && t >= ta && t < tb ? min(n0 + t + 1, P.cap) : 0;
        }
        auto pair_of = [&](const xu32x4_t* cache, const xu32x4_t* fresh, int key) -> const xu32x4_t* {
            const int kc = min(key, n_max - 1);
            return kc < n0 ? cache + (size_t)kc * CH : fresh + (size_t)(kc - n0) * new_stride;
        };
        // K of a tile in the layout of the matrix operand: lane (quad, n16) holds key attn_qk_key(nt, n16), 16-byte chunk ks * 4 + quad
        auto fetch_operand = [&](int base, X128 (&x)[2 * KS]) {
#pragma unroll
            for (int nt = 0; nt < 2; ++nt) {
                const xu32x4_t* p = pair_of(Kr, kn, base + attn_qk_key<D>(nt, n16));
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) x[nt * KS + ks].u = p[ks * 4 + quad];
            }
        };
        auto query = [&](int k, int ks) {
            X128 q;
            q.u = *reinterpret_cast<const xu32x4_t*>(s_q + (k * 16 + n16) * KRS + (ks * 4 + quad) * 16);
            return q;
        };

        for (int sp = 0; sp < nused && tb > ta; ++sp) {
            const int start = sp == 0 ? 0 : sp * split_len, stop = sp == nsplit - 1 || split_len >= n_max - start ? n_max : start + split_len;
            if (SPLIT && nused > 1 && sp % kSplitBatch == 0) {
                // The merge weighs eight records at a time by their largest maximum, so the maxima come first: one walk over the keys of the
                // next kSplitBatch splits for the logits alone.  A wavefront walks a stretch of its own.
                const int sp_end = min(sp + kSplitBatch, nused), last = sp_end == nsplit ? n_max : min(sp_end * split_len, n_max);
                for (int i = tid; i < kSplitBatch * GROUPS * 16; i += kXThreads) s_top[i] = float_order(kXNegBig);
                __syncthreads();
                const int tiles = (last - start + kXKT - 1) / kXKT, per = (tiles + kXWaves - 1) / kXWaves;
                const int w0 = min(wave * per, tiles), w1 = min(w0 + per, tiles);
                X128 kb[2 * KS];
                float mx[GROUPS];
#pragma unroll
                for (int k = 0; k < GROUPS; ++k) mx[k] = kXNegBig;
                if (w0 < w1) fetch_operand(start + w0 * kXKT, kb);
                for (int t = w0; t < w1; ++t) {
                    const int base = start + t * kXKT, mine = min(base / split_len, nsplit - 1);
#pragma unroll
                    for (int k = 0; k < GROUPS; ++k) {
                        xf32x4_t c[2];
                        c[0] = c[1] = (xf32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int ks = 0; ks < KS; ++ks) {
                            const X128 q = query(k, ks);
#pragma unroll
                            for (int nt = 0; nt < 2; ++nt) c[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kb[nt * KS + ks].v, q.v, c[nt], 0, 0, 0);
                        }
#pragma unroll
                        for (int nt = 0; nt < 2; ++nt)
#pragma unroll
                            for (int i = 0; i < 4; ++i) mx[k] = fmaxf(mx[k], base + attn_qk_key<D>(nt, quad * 4 + i) < lim[k] ? attn_logit(c[nt][i], scale) : kXNegBig);
                    }
                    if (t + 1 == w1 || min((base + kXKT) / split_len, nsplit - 1) != mine) {
#pragma unroll
                        for (int k = 0; k < GROUPS; ++k) {
                            const float v = quads_max(mx[k]);
                            if (quad == 0) atomicMax(&s_top[(mine - sp) * (GROUPS * 16) + k * 16 + n16], float_order(v));
                            mx[k] = kXNegBig;
                        }
                    }
                    if (t + 1 < w1) fetch_operand(base + kXKT, kb);
                }
                __syncthreads();
            }

            int tile_tid = threadIdx.x;   // (opaque as well: what this split needs does not take registers in the walk above)
            asm volatile("" : "+v"(tile_tid));
            const int lane = tile_tid & (kWave - 1), n16 = lane & 15, quad = lane >> 4;
            const int wave = __builtin_amdgcn_readfirstlane(tile_tid / kWave);   // (the walk and its addresses are the wavefront's: scalars, branches)
            const int ntiles = (stop - start + kXKT - 1) / kXKT;
            const int rot = rotate ? attn_rotation(row, sp, ntiles) : 0;
            float m_run[GROUPS], l_run[GROUPS][4], lx_run[GROUPS][4];   // l, lx: one sum per key of a quarter of the tile, as in a single step
            // l as a channel of ones (head_dim 128): the matrix cores add what took sixteen of some 115 vector instructions of a tile and group: 128
            // rows of 2048 pairs, 128 steps 168.4 us, so 162.0 (logits into their exponentials' arguments by one fma: 162.6).  [0] is rescaled and used.
            xf32x4_t ol[GROUPS];
            X128 ones;
            ones.u = xu32x4_t{0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
            xf32x4_t o[GROUPS][ET];                                       // o[k][e][i]: channel (quad * 4 + i) * ET + e, un-normalised
            xf32x4_t o2[GROUPS][TERMS > 1 ? ET : 1], o3[GROUPS][TERMS > 1 ? ET : 1];   // those of the second and third terms
#pragma unroll
            for (int k = 0; k < GROUPS; ++k) {
                m_run[k] = kXNegBig;
                ol[k] = (xf32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int i = 0; i < 4; ++i) l_run[k][i] = lx_run[k][i] = 0.f;
#pragma unroll
                for (int e = 0; e < ET; ++e) {
                    o[k][e] = (xf32x4_t){0.f, 0.f, 0.f, 0.f};
                    if constexpr (TERMS > 1) o2[k][e] = o3[k][e] = o[k][e];
                }
            }
            auto base_of = [&](int t) { return start + (t + rot < ntiles ? t + rot : t + rot - ntiles) * kXKT; };
            // The next tile's K is fetched a tile ahead, V before the tile's logits and weights are formed.
            X128 kr[KL], vr[8];   // K: lane holds the keys lane / CH * KL + u, 16-byte chunk lane % CH; V: key quad * 8 + u, a 16th of the row
            const int kkey = lane / CH * KL, kch = lane % CH, krow = attn_qk_row<D>(kkey);   // (kkey: a multiple of KL, 4 or 8)
            auto fetch_k = [&](int base) {
                if (base + kXKT <= n0) {   // a whole tile of cached pairs: one address, constant offsets
                    const xu32x4_t* p = Kr + (size_t)(base + kkey) * CH + kch;
#pragma unroll
                    for (int u = 0; u < KL; ++u) kr[u].u = p[u * CH];
                    return;
                }
#pragma unroll
                for (int u = 0; u < KL; ++u) kr[u].u = pair_of(Kr, kn, base + kkey + u)[kch];
            };
            if (wave < ntiles) fetch_k(base_of(wave));
            for (int t = wave; t < ntiles; t += kXWaves) {
                const int base = base_of(t);
#pragma unroll
                for (int u = 0; u < KL; ++u) *reinterpret_cast<xu32x4_t*>(my_k + (krow + attn_qk_row<D>(u)) * KRS + kch * 16) = kr[u].u;
                auto load_v = [&](const xu32x4_t* p, X128& x) {
                    if constexpr (D == 128) {
                        x.u = p[n16];
                    } else {
                        const xu32x2_t y = reinterpret_cast<const xu32x2_t*>(p)[n16];
                        x.w[0] = y.x;
                        x.w[1] = y.y;
                    }
                };
                // The next tile's K before this one's V: what waits for V (the last loads) then finds K there too.
                if (t + kXWaves < ntiles) fetch_k(base_of(t + kXWaves));
                if (base + kXKT <= n0) {
                    const xu32x4_t* p = Vr + (size_t)(base + quad * 8) * CH;
#pragma unroll
                    for (int u = 0; u < 8; ++u) load_v(p + u * CH, vr[u]);
                } else {
#pragma unroll
                    for (int u = 0; u < 8; ++u) load_v(pair_of(Vr, vn, base + quad * 8 + u), vr[u]);
                }
                __builtin_amdgcn_wave_barrier();
                const bool partial = base + kXKT > n_first;   // some step does not see the whole tile
                xf32x4_t c[GROUPS][2];
#pragma unroll
                for (int k = 0; k < GROUPS; ++k) c[k][0] = c[k][1] = (xf32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    X128 kb[2];
#pragma unroll
                    for (int nt = 0; nt < 2; ++nt) {
                        kb[nt].u = *reinterpret_cast<const xu32x4_t*>(my_k + (nt * 16 + n16) * KRS + (ks * 4 + quad) * 16);
                    }
#pragma unroll
                    for (int k = 0; k < GROUPS; ++k) {
                        const X128 q = query(k, ks);
#pragma unroll
                        for (int nt = 0; nt < 2; ++nt) c[k][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kb[nt].v, q.v, c[k][nt], 0, 0, 0);
                    }
                }
                float x[GROUPS][9];   // arguments of the exponentials: eight keys and the correction
                auto key_of = [&](int j) { return attn_qk_key<D>(j / 4, quad * 4 + j % 4); };
                float lo = 0.f;
                bool changed[GROUPS];
#pragma unroll
                for (int k = 0; k < GROUPS; ++k) {
                    const int left = lim[k] - base;   // this lane's query sees the tile's keys [0, left)
#pragma unroll
                    for (int j = 0; j < 8; ++j) x[k][j] = attn_logit(c[k][j / 4][j % 4], scale);
                    if (partial) {
#pragma unroll
                        for (int j = 0; j < 8; ++j)
                            if (key_of(j) >= left) x[k][j] = -INFINITY;   // of no weight, also where a step sees none of the tile
                    }
                    float mn = x[k][0];
#pragma unroll
                    for (int j = 1; j < 8; ++j) mn = fmaxf(mn, x[k][j]);
                    mn = fmaxf(m_run[k], quads_max(mn));
                    changed[k] = mn > m_run[k];
                    x[k][8] = m_run[k];
#pragma unroll
                    for (int j = 0; j < 9; ++j) {
                        x[k][j] -= mn;
                        lo = fminf(lo, x[k][j]);
                    }
                    m_run[k] = mn;
                }
                if (__any(lo < -126.f)) {   // exp2f's way round denormal results, only where there can be one
#pragma unroll
                    for (int k = 0; k < GROUPS; ++k)
#pragma unroll
                        for (int j = 0; j < 9; ++j) x[k][j] = exp2f(x[k][j]);
                } else {
#pragma unroll
                    for (int k = 0; k < GROUPS; ++k)
#pragma unroll
                        for (int j = 0; j < 9; ++j) x[k][j] = __builtin_amdgcn_exp2f(x[k][j]);
                }
                X128 pa[GROUPS][TERMS];   // probabilities of query n16 in bf16, term by term: the keys of this lane's logits, quad * 8 + u
                auto at = [](int u) { return D == 128 ? u % 2 * 4 + u / 2 : u; };   // the u-th of these keys is logit at(u)
#pragma unroll
                for (int k = 0; k < GROUPS; ++k) {
                    float y[8];   // rounded
#pragma unroll
                    for (int w = 0; w < 4; ++w) {
                        pa[k][0].w[w] = pack_bf16(x[k][at(2 * w)], x[k][at(2 * w + 1)]);
                        y[at(2 * w)] = bf16_lo(pa[k][0].w[w]);
                        y[at(2 * w + 1)] = bf16_hi(pa[k][0].w[w]);
                    }
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        if constexpr (TERMS > 1) l_run[k][i] = fmaf(l_run[k][i], x[k][8], x[k][i]) + x[k][4 + i];
                        if constexpr (FEAT) lx_run[k][i] = fmaf(lx_run[k][i], x[k][8], x[k][i]) + x[k][4 + i];
                    }
                    if constexpr (TERMS > 1) {   // each term of what the ones before leave (the third has no bits beyond bf16)
#pragma unroll
                        for (int w = 0; w < 4; ++w) {
                            const float r0 = x[k][at(2 * w)] - y[at(2 * w)], r1 = x[k][at(2 * w + 1)] - y[at(2 * w + 1)];
                            pa[k][1].w[w] = pack_bf16(r0, r1);
                            pa[k][2].w[w] = pack_bf16(r0 - bf16_lo(pa[k][1].w[w]), r1 - bf16_hi(pa[k][1].w[w]));
                        }
                    }
                }
                if (t != wave) {   // (at the first tile there is nothing yet)
#pragma unroll
                    for (int k = 0; k < GROUPS; ++k) {
                        if (!__any(changed[k])) continue;
                        if constexpr (TERMS == 1) ol[k][0] *= x[k][8];
#pragma unroll
                        for (int e = 0; e < ET; ++e)
#pragma unroll
                            for (int i = 0; i < 4; ++i) {
                                o[k][e][i] *= x[k][8];
                                if constexpr (TERMS > 1) {
                                    o2[k][e][i] *= x[k][8];
                                    o3[k][e][i] *= x[k][8];
                                }
                            }
                    }
                }
                // V^T: tile e = channel n16 * ET + e over this lane's 8 keys (8 x ET transpose in registers)
                auto transposed = [&](int e) {
                    const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;
                    X128 vb;
#pragma unroll
                    for (int w = 0; w < 4; ++w) vb.w[w] = __builtin_amdgcn_perm(vr[2 * w + 1].w[e >> 1], vr[2 * w].w[e >> 1], sel);
                    return vb;
                };
                bool bad = false;
                if (base + kXKT > n0) {
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const int key = base + quad * 8 + u;
#pragma unroll
                        for (int w = 0; w < D / 32; ++w) {
                            if (key >= n_max) vr[u].w[w] = 0;   // rows past the last step's end
                            bad |= key >= n0 && pair_not_finite(vr[u].w[w]);
                        }
                    }
                }
                if (bad && tb - ta > 1) s_bad = 1;
                if constexpr (TERMS == 1) {
#pragma unroll
                    for (int k = 0; k < GROUPS; ++k) ol[k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones.v, pa[k][0].v, ol[k], 0, 0, 0);
                }
#pragma unroll
                for (int e = 0; e < ET; ++e) {
                    const X128 vb = transposed(e);
#pragma unroll
                    for (int k = 0; k < GROUPS; ++k) {
                        o[k][e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vb.v, pa[k][0].v, o[k][e], 0, 0, 0);
                        if constexpr (TERMS > 1) {
                            o2[k][e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vb.v, pa[k][1].v, o2[k][e], 0, 0, 0);
                            o3[k][e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vb.v, pa[k][2].v, o3[k][e], 0, 0, 0);
                        }
                    }
                }
                __builtin_amdgcn_wave_barrier();
            }

            // ---- merge the wavefronts' partials, JOINT groups at once ------------------------------------
            int tid = threadIdx.x;   // (opaque: or everything that the merge derives from it is kept in registers over the tile loop)
            asm volatile("" : "+v"(tid));
#pragma unroll
            for (int k0 = 0; k0 < GROUPS; k0 += JOINT) {
                auto live = [&](int k, int r) { return r < spg * G && step_of(k, r) >= ta && step_of(k, r) < tb; };
                auto publish = [&](float* to, const xf32x4_t* x) {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
#pragma unroll
                        for (int e = 0; e < ET; e += 4) *reinterpret_cast<float4*>(to + i * ET + e) = make_float4(x[e][i], x[e + 1][i], x[e + 2][i], x[e + 3][i]);
                };
#pragma unroll
                for (int g = 0; g < JOINT; ++g) {
                    const int k = k0 + g;
                    float* dst = reinterpret_cast<float*>(my_k + g * C::PART_BYTES) + n16 * PART + quad * 4 * ET;   // the loop is over
                    publish(dst, o[k]);
                    if constexpr (TERMS > 1) {
                        publish(dst + 16 * PART, o2[k]);
                        publish(dst + 32 * PART, o3[k]);
                    }
                    const float ls = TERMS == 1 ? ol[k][0] : quads_sum((l_run[k][0] + l_run[k][1]) + (l_run[k][2] + l_run[k][3]));
                    const float lxs = FEAT ? quads_sum((lx_run[k][0] + lx_run[k][1]) + (lx_run[k][2] + lx_run[k][3])) : 0.f;
                    if (quad == 0) {
                        const int i = (g * kXWaves + wave) * 16 + n16;
                        s_m[i] = m_run[k];
                        s_l[i] = ls;
                        if (FEAT) s_lx[i] = lxs;
                    }
                }
                __syncthreads();
                if (s_bad && tb - ta > 1) {   // (the same for every thread: all tiles of the split are done)
                    together = false;
                    tb = ta;
                    break;
                }
                const bool merging = SPLIT && nused > 1;
                if (tid < JOINT * kXWaves * 16) {   // weight of every partial; row maximum and exact normaliser for the second launch
                    const int r = tid % 16, g = tid / (kXWaves * 16), at = g * kXWaves * 16 + r;
                    float mn = kXNegBig;
#pragma unroll
                    for (int g2 = 0; g2 < kXWaves; ++g2) mn = fmaxf(mn, s_m[at + g2 * 16]);
                    s_w[tid] = exp2f(s_m[tid] - mn);
                    if (FEAT && tid % (kXWaves * 16) < 16 && live(k0 + g, r)) {
                        float lx = 0.f;
#pragma unroll
                        for (int g2 = 0; g2 < kXWaves; ++g2) lx = fmaf(s_lx[at + g2 * 16], exp2f(s_m[at + g2 * 16] - mn), lx);
                        P.stat[((size_t)row * P.T + step_of(k0 + g, r)) * G + r % G] = make_float2(mn, 1.0f / lx);
                    }
                } else if (merging && tid < (kXWaves + 1) * 16) {   // (JOINT = 1) the split's record joins the others as in a single step: c0, weight
                    const int r = tid % 16, q = k0 * 16 + r;
                    const uint32_t* tops = s_top + (sp % kSplitBatch) * (GROUPS * 16) + q;
                    float cm = sp == 0 ? kXNegBig : s_out_m[q], c0 = 1.f;
                    if (sp % 8 == 0) {
                        const float before = cm;
                        for (int u = 0; u < 8 && sp + u < nused; ++u) cm = fmaxf(cm, order_float(tops[u * (GROUPS * 16)]));
                        c0 = exp2f(before - cm);
                        s_out_m[q] = cm;
                    }
                    s_c[r] = c0;
                    s_cw[r] = exp2f(order_float(tops[0]) - cm);
                }
                __syncthreads();
#pragma unroll
                for (int g = 0; g < JOINT; ++g) {
                    const int k = k0 + g;
                    if (tid < 16 * D / 4) {   // four channels of a query
                        const int r = tid / (D / 4), d = tid % (D / 4) * 4;
                        float a[4] = {0.f, 0.f, 0.f, 0.f}, a2[4] = {0.f, 0.f, 0.f, 0.f}, a3[4] = {0.f, 0.f, 0.f, 0.f}, l = 0.f;
                        auto add = [](const float* p, float w, float (&to)[4]) {
                            const float4 v = *reinterpret_cast<const float4*>(p);
                            to[0] = fmaf(v.x, w, to[0]);
                            to[1] = fmaf(v.y, w, to[1]);
                            to[2] = fmaf(v.z, w, to[2]);
                            to[3] = fmaf(v.w, w, to[3]);
                        };
#pragma unroll
                        for (int g2 = 0; g2 < kXWaves; ++g2) {
                            const float *p = reinterpret_cast<const float*>(smem + (size_t)g2 * C::WAVE_BYTES + g * C::PART_BYTES) + r * PART + d, w = s_w[(g * kXWaves + g2) * 16 + r];
                            add(p, w, a);
                            if constexpr (TERMS > 1) {
                                add(p + 16 * PART, w, a2);
                                add(p + 32 * PART, w, a3);
                            }
                            l = fmaf(s_l[(g * kXWaves + g2) * 16 + r], w, l);
                        }
                        if constexpr (TERMS > 1) {
#pragma unroll
                            for (int i = 0; i < 4; ++i) a[i] = add_terms(a[i], a2[i], a3[i]);
                        }
                        if (merging) {
                            float* sum = s_out + (k * 16 + r) * D + d;
                            const float c0 = s_c[r], cw = s_cw[r];
#pragma unroll
                            for (int i = 0; i < 4; ++i) {
                                const float before = sp == 0 ? 0.f : sum[i] * c0;
                                sum[i] = a[i] = fmaf(a[i], cw, before);
                            }
                            l = fmaf(l, cw, sp == 0 ? 0.f : s_out_l[(sp & 1) * 16 * GROUPS + k * 16 + r] * c0);
                            if (d == 0) s_out_l[((sp & 1) ^ 1) * 16 * GROUPS + k * 16 + r] = l;   // (read by the others of the row before the next barrier)
                        }
                        if (sp == nused - 1 && live(k, r)) {
                            const xu32x2_t v = {pack_bf16(a[0] / l, a[1] / l), pack_bf16(a[2] / l, a[3] / l)};
                            *reinterpret_cast<xu32x2_t*>(reinterpret_cast<bf16_t*>(P.out_seq) + q_row(k, r) * D + d) = v;
                        }
                    }
                }
                __syncthreads();
            }
        }
    }
    if (!FEAT && tid == 0 && arrived == (uint32_t)blocks - 1) {   // the last workgroup of the row sets its length: all of them have read it by then
        if (blocks > 1) __hip_atomic_store(&P.row_cnt[row], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        P.len[row] = n1;
    }
}

// ---------------------------------------------------------------------------------------------------------
// The planes.  A wavefront owns 16 keys (a tile of a 16x16x32 product, K as the B operand in registers for the whole walk) and
// takes 16 padded queries at a time, GP heads of SPT = 16 / GP steps, from LDS.  Matrix row r is head r / SPT, step r % SPT:
// the four results of a lane belong to one key and to HPL = 4 / SPT heads, their steps in order.
// Bound by instruction issue and by how evenly the wavefronts fill the chip: 128 rows of 2176 keys, 128 steps 106 us with 32 keys a wavefront, four
// wavefronts a SIMD (2.1 rounds of workgroups) and branches on the keys by lane; 91 with 16 keys and six wavefronts.  Two and four tiles of
// queries at a time: 0 to 30 % slower, the registers leave five wavefronts or spill.
// ---------------------------------------------------------------------------------------------------------
static constexpr int kFeatQ = 64;   // padded queries per staged block
static constexpr int kFeatKeys = kXWaves * 16;   // keys of a workgroup

template <int GP>
__global__ __launch_bounds__(kXThreads, 6) void window_feat_planes_kernel(const WindowParams P) {
#pragma clang fp contract(off)   // a step's weight is rounded before it is added, as in the single steps
    constexpr int SPT = 16 / GP, HPL = 4 / SPT, QRS = WindowCfg<128, 2>::KRS, kXCH = WindowCfg<128, 2>::CH;
    constexpr int LD = kFeatQ * kXCH / kXThreads;
    const int row = blockIdx.y, b = row / P.n_kv, hkv = row % P.n_kv, G = P.g, T = P.T;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), n16 = lane & 15, quad = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);   // (scalar: so are the branches on its keys)
    const int n0 = min(max(P.len[row], 0), P.cap), n1 = min(n0 + T, P.cap);
    // steps from which the windows of the last 8, 16 and 32 queries of the chunk are open
    const int on8 = P.chunk_len - 8 - P.chunk_pos, on16 = on8 - 8, on32 = on8 - 24;

    __shared__ __attribute__((aligned(16))) unsigned char s_q[2][kFeatQ * QRS];
    __shared__ __attribute__((aligned(16))) float s_max[2][kFeatQ], s_inv[2][kFeatQ];   // of every padded query, in matrix row order
    const xu32x4_t* Kr = reinterpret_cast<const xu32x4_t*>(P.K) + (size_t)row * P.cap * kXCH;
    const float2* stat = P.stat + (size_t)row * T * G;
    float* feat = P.feat + (size_t)row * kFeatPlanes * P.cap * GP;
    const size_t plane = (size_t)P.cap * GP;

    for (int k0 = blockIdx.x * kFeatKeys; k0 < n1; k0 += gridDim.x * kFeatKeys) {
        const int kb = k0 + wave * 16, key = kb + n16;   // the wavefront's first key, the lane's
        X128 kreg[4];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) kreg[ks].u = Kr[(size_t)min(key, n1 - 1) * kXCH + ks * 4 + quad];
        // this lane's sums, head quad * HPL + h; a new pair's start from zero
        float wl[HPL], w32[HPL], w16[HPL], w8[HPL];
#pragma unroll
        for (int h = 0; h < HPL; ++h) {
            const float* f = feat + (size_t)min(key, n1 - 1) * GP + quad * HPL + h;
            const bool old = key < n0;
            wl[h] = old ? f[3 * plane] : 0.f;
            w32[h] = old && T > on32 ? f[2 * plane] : 0.f;
            w16[h] = old && T > on16 ? f[plane] : 0.f;
            w8[h] = old && T > on8 ? f[0] : 0.f;
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
                xf32x4_t c = (xf32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) {
                    X128 q;
                    q.u = *reinterpret_cast<const xu32x4_t*>(s_q[buf] + (qt * 16 + n16) * QRS + (ks * 4 + quad) * 16);
                    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(q.v, kreg[ks].v, c, 0, 0, 0);
                }
                const float4 mx = *reinterpret_cast<const float4*>(&s_max[buf][qt * 16 + quad * 4]);
                const float4 iv = *reinterpret_cast<const float4*>(&s_inv[buf][qt * 16 + quad * 4]);
                const float m4[4] = {mx.x, mx.y, mx.z, mx.w}, i4[4] = {iv.x, iv.y, iv.z, iv.w};
                float x[4], lo = 0.f;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    x[i] = attn_logit(c[i], P.scale_log2e) - m4[i];
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
                for (int i = 0; i < 4; ++i) x[i] *= i4[i];
                if (kb + 16 <= n0 + t0 + 1 && t0 + SPT <= min(on32, T)) {   // nothing hidden, no window open
#pragma unroll
                    for (int i = 0; i < 4; ++i) wl[i / SPT] += x[i];
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int h = i / SPT, t = t0 + i % SPT;   // element i: matrix row quad * 4 + i
                        if (key <= n0 + t && t < T) {
                            wl[h] += x[i];
                            if (t >= on32) w32[h] += x[i];
                            if (t >= on16) w16[h] += x[i];
                            if (t >= on8) w8[h] += x[i];
                        }
                    }
                }
            }
            if (more) stage(buf ^ 1);
            __syncthreads();
        }
#pragma unroll
        for (int h = 0; h < HPL; ++h) {
            if (key >= n1) continue;
            float* f = feat + (size_t)key * GP + quad * HPL + h;
            f[3 * plane] = wl[h];
            if (key >= n0 || T > on32) f[2 * plane] = w32[h];
            if (key >= n0 || T > on16) f[plane] = w16[h];
            if (key >= n0 || T > on8) f[0] = w8[h];
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

template <int D, bool FEAT, bool SPLIT, int GROUPS>
static fk_status window_launch(const WindowParams& P, hipStream_t st) {
    using C = WindowCfg<D, GROUPS, SPLIT>;
    const int spg = 16 / P.g, blocks = (P.T + spg * GROUPS - 1) / (spg * GROUPS);
    auto kern = window_attn_kernel<D, FEAT, SPLIT, GROUPS>;
    const size_t lds = C::LDS_BYTES + (SPLIT ? C::MERGE_BYTES : 0);
    static bool lds_ok[kMaxDevices] = {};
    if (!allow_dynamic_lds((const void*)kern, lds, lds_ok)) return FK_ERR_LAUNCH;
    hipLaunchKernelGGL(kern, dim3((P.rows < 8 ? P.rows : (P.rows + 7) / 8 * 8) * blocks), dim3(kXThreads), lds, st, P, spg, blocks);
    return launch_status();
}

template <int D, bool FEAT, bool SPLIT>
static fk_status window_groups(const WindowParams& P, hipStream_t st) {
    // two groups share every tile that is loaded; one where that leaves CUs without a workgroup
    const int spg = 16 / P.g;
    if ((long long)P.rows * ((P.T + 2 * spg - 1) / (2 * spg)) >= 256) return window_launch<D, FEAT, SPLIT, 2>(P, st);
    return window_launch<D, FEAT, SPLIT, 1>(P, st);
}

fk_status window_attn(const WindowParams& P, bool split, hipStream_t st) {
    if (P.shape.head_dim == 64) return split ? window_groups<64, false, true>(P, st) : window_groups<64, false, false>(P, st);
    return split ? window_groups<128, false, true>(P, st) : window_groups<128, false, false>(P, st);
}

fk_status window_feat(const WindowParams& P, int max_len, hipStream_t st) {
    const fk_status s = window_groups<128, true, false>(P, st);
    if (s != FK_OK) return s;
    const dim3 grid((max_len + kFeatKeys - 1) / kFeatKeys, P.rows);
    if (P.g <= 4) hipLaunchKernelGGL(window_feat_planes_kernel<4>, grid, dim3(kXThreads), 0, st, P);
    else hipLaunchKernelGGL(window_feat_planes_kernel<8>, grid, dim3(kXThreads), 0, st, P);
    return launch_status();
}

}  // namespace fk
