// Golden Eviction label builder (Section 3.2 Eq. 3-5) on dense causal attention matrices.
//
//   pool   a~[h'][t][i] = 1/(g L) * sum over the g heads of group h' and the queries q of block t
//                         (B + tL <= q < min(B + (t+1)L, T)) of A[h][q][i]          (Eq. 3, 4)
//   future alpha[h'][t][i] = max_{j >= t} a~[h'][j][i]                               (Eq. 5, first half)
//   trace  step t keeps the L newest pairs and, of the other B the cache holds, the B - L with
//          the largest alpha[.][t] (ties: lower position), evicted pairs never return  (Eq. 5, second half)
//
// pool is the only kernel that touches the O(T^2) input and is HBM bound: a workgroup owns one
// (key tile, block, group) and streams g * L row segments of 256 to 1024 bytes (16 bytes a lane, eight loads in flight
// per thread); chunks wholly above the diagonal are never read (A is causal), so the traffic is the lower triangle below
// query B + L.  future is a running maximum down the block axis; trace is sequential by nature: one workgroup per group walks the M steps.
#include "select_common.h"

namespace fk {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
static constexpr int kPoolThreads = 512;
static constexpr int kPoolU = 8;   // loads in flight per thread

template <int W>   // value i (lower lanes) and i + W (upper lanes) of both halves added up, i < W
__device__ __forceinline__ void fold_halves(float* v) {
#pragma unroll
    for (int i = 0; i < W; ++i) v[i] = add_halves(v[i], v[i + W]);
}
template <int W>   // the same for the odd and even rows of 16 lanes
__device__ __forceinline__ void fold_rows(float* v) {
#pragma unroll
    for (int i = 0; i < W; ++i) v[i] = add_rows(v[i], v[i + W]);
}
// Bound by HBM.  32 heads of 8192 tokens, bf16: 2.0 GB of causal entries in 320 us, 6.3 TB/s (343 us, 5.9, while tiles and XCDs went in step: see below).
// The loads of a pass are under no condition where the whole pass is there: behind a condition the compiler waited for the first seven
// before it issued the eighth.  Partial sums of a wavefront are added in registers (through LDS, sixteen to a key, no slower).
template <typename T, int LPR>   // LPR: lanes of a row segment, 16, 32 or 64
__global__ __launch_bounds__(kPoolThreads) void golden_pool_kernel(const T* __restrict__ A, int g, int Tn, size_t ld,
                                                                   int budget, int L, int M,
                                                                   float* __restrict__ a_tilde) {
    constexpr int EPC = Vec16<T>::N;   // elements per 16-byte chunk
    constexpr int KT = LPR * EPC;      // keys per tile
    constexpr int RG = kPoolThreads / LPR, U = kPoolU;   // row groups of the workgroup, loads in flight
    // Block t has `live(t)` tiles with keys that its queries see, more the later it is; the first and the last block, the second and the last but
    // one, ... share the workgroups of a row of the grid, so that hardly any finds nothing to do.  From row to row the tiles move on by one
    // workgroup: tile i always on XCD i % 8 would read through two of the sixteen channels of that XCD's L2 only.
    const int tiles = (Tn + KT - 1) / KT, hp = blockIdx.z;
    auto live = [&](int t) { return (min(budget + (t + 1) * L, Tn) + KT - 1) / KT; };
    int t = blockIdx.y + 1, tile = blockIdx.x + blockIdx.y;
    if (tile >= (int)gridDim.x) tile %= (int)gridDim.x;
    if (tile >= live(t)) {
        tile -= live(t);
        if (M - (int)blockIdx.y == t) return;
        t = M - blockIdx.y;
        if (tile >= live(t)) return;
    }
    const int i0 = tile * KT;
    const int q0 = budget + t * L, q1 = min(q0 + L, Tn);
    const int c = threadIdx.x % LPR, rg = threadIdx.x / LPR;
    const int i_mine = i0 + c * EPC;   // this lane's first key; queries before it see none of its keys
    float acc[EPC];
#pragma unroll
    for (int e = 0; e < EPC; ++e) acc[e] = 0.f;
    const int qs = max(q0, i0), rows = q1 - qs;
    float* to = a_tilde + ((size_t)hp * M + (t - 1)) * Tn + i0;
    if (i_mine < q1 && (size_t)i_mine < ld) {
        // This row group takes the pairs (head, query) rg, rg + RG, ...: dh heads and dq queries on, one head more where that leaves the block.
        const int total = rows * g;
        int dh = 0, dq = RG, h = 0, q = rg;
        if (rows <= RG) {   // (four divisions before the first load: a launch of a few us is 0.3 longer by them)
            dh = RG / rows, dq = RG % rows;
            h = rg / rows, q = rg % rows;
        }
        const size_t step = ((size_t)dh * Tn + dq) * ld, wrap = (size_t)(Tn - rows) * ld;
        const T* p = A + ((size_t)(hp * g + h) * Tn + qs + q) * ld + i_mine;
        const bool below = qs >= i0 + KT - 1;   // every query sees every key of the tile
        for (int r0 = 0; r0 < total; r0 += RG * U) {
            u32x4 v[U];
            // (read once, never again: non-temporal, so the lines do not push anything out of the caches)
            auto load = [](const T* p) { return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p)); };
            auto advance = [&]() {
                p += step;
                q += dq;
                if (q >= rows) {
                    q -= rows;
                    p += wrap;
                }
            };
            if (below && r0 + RG * U <= total) {   // (no load under a condition)
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    v[u] = load(p);
                    advance();
                }
            } else {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    v[u] = (u32x4){0, 0, 0, 0};
                    if (r0 + rg + u * RG < total && qs + q >= i_mine) v[u] = load(p);
                    advance();
                }
            }
            float x[EPC], y[EPC];
            auto sum = [&](int u, float (&to)[EPC]) {   // of four
                float a[EPC], b[EPC];
                auto pair = [&](int w, float (&z)[EPC]) {
                    float z1[EPC];
                    Vec16<T>::unpack(make_uint4(v[w].x, v[w].y, v[w].z, v[w].w), z);
                    Vec16<T>::unpack(make_uint4(v[w + 1].x, v[w + 1].y, v[w + 1].z, v[w + 1].w), z1);
#pragma unroll
                    for (int e = 0; e < EPC; ++e) z[e] += z1[e];
                };
                pair(u, a);
                pair(u + 2, b);
#pragma unroll
                for (int e = 0; e < EPC; ++e) to[e] = a[e] + b[e];
            };
            sum(0, x);
            sum(4, y);
#pragma unroll
            for (int e = 0; e < EPC; ++e) acc[e] += x[e] + y[e];
        }
    }
    for (int z = tile + live(t); z < tiles; z += live(t))   // tiles above the diagonal
        for (int k = threadIdx.x; k < KT && z * KT + k < Tn; k += kPoolThreads) to[(z - tile) * KT + k] = 0.f;
    // the row groups of a wavefront in registers (a lane ends with its share of its chunk's keys), the wavefronts through LDS
    constexpr int WAVES = kPoolThreads / kWave, E = EPC * LPR / kWave;
    __shared__ float s_acc[WAVES][KT];
    int first = c * EPC;   // this lane's first key of the tile
    if constexpr (LPR <= 32) {
        fold_halves<EPC / 2>(acc);
        first += (int)threadIdx.x / 32 % 2 * (EPC / 2);
    }
    if constexpr (LPR == 16) {
        fold_rows<E>(acc);
        first += (int)threadIdx.x / 16 % 2 * E;
    }
#pragma unroll
    for (int e = 0; e < E; ++e) s_acc[threadIdx.x / kWave][first + e] = acc[e];
    __syncthreads();
    for (int k = threadIdx.x; k < KT && i0 + k < Tn; k += kPoolThreads) {
        float s = 0.f;
#pragma unroll
        for (int r = 0; r < WAVES; ++r) s += s_acc[r][k];
        to[k] = s / ((float)g * (float)L);
    }
}

// alpha[t] = max(a~[t], alpha[t + 1]), walking the blocks from the last to the first; one thread per key, U blocks' loads in
// flight (a wavefront or two a SIMD: a walk of 223 blocks of 4096 tokens waits for memory 28 times with eight, seven times with 32: 6 us less;
// no more of them than blocks)
template <int U>
__global__ void golden_future_kernel(const float* __restrict__ a_tilde, int Tn, int M, float* __restrict__ alpha) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x, hp = blockIdx.y;
    if (i >= Tn) return;
    const size_t o0 = (size_t)hp * M * Tn + i;
    float run = -INFINITY;
    for (int t = M; t >= 1; t -= U) {
        float a[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int back = U == 8 ? t - u - 1 : max(t - u - 1, 0);   // (past the first block that one again; eight or fewer: nothing, 0.2 us less)
            a[u] = back >= 0 ? a_tilde[o0 + (size_t)back * Tn] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (t - u >= 1) {
                run = t - u == M ? a[u] : fmaxf(run, a[u]);
                alpha[o0 + (size_t)(t - u - 1) * Tn] = run;
            }
        }
    }
}

static constexpr int kTraceMaxCache = 12288;               // B + L
static constexpr int kTraceMaxLds = 152 * 1024;            // dynamic
static constexpr int kTrThreads = 1024, kTrHold = 512;     // threads of the workgroup; those that hold the candidates
static constexpr int kTrWrite = kTrThreads - kTrHold - kWave, kTrWriteWaves = kTrWrite / kWave;   // those that write; one wavefront finds the cut
static constexpr int kTrBins = 512, kTrCap = 8, kTrCut = 320;   // bins, places of a bin, bin of the last step's cut
static constexpr int kTraceSlots = 4096, kTrFresh = 5;      // golden_trace_kernel: budget; newest pairs of a writing thread, at most
static constexpr uint32_t kStays = 0x80000000u, kTrDown = 0xfffffffeu;   // a position p is compared as kTrDown - p, the lower one above

// The eviction trace.  One workgroup per KV group walks the M steps; what bounds it is the chain of one step after the other, so
// a step has two barriers, and what the next step does not wait for runs beside it.
//   Half of the workgroup holds the B candidates, each in a register slot of some thread, in no order.  Candidates are ranked
// by (future score, then position, the lower one above), all different, so "the E = L lowest go" is one threshold.  A slot
// whose pair goes takes one of the L newest pairs, candidates from the next step on: nothing is moved.
//   The threshold: the cut moves little from step to step, so the keys around the last one are counted in 512 bins of the bit pattern,
// its bin the 320th, and a bin has places for the first eight pairs themselves.  Keys above the bins are not counted, keys below
// them by vote.  One wavefront finds the bin in which the count from the bottom reaches E and ranks its pairs; bins get finer or
// coarser as they fill.  A bin with more pairs, up to 64, is gathered and ranked by one wavefront.  One with more still (ties), and all
// pairs at the first step and where the cut has left the bins, are counted again over their own range, of the keys or, if those are
// equal, of the positions.  After a cut among equal keys the next one is taken to be among the same keys, until their number says otherwise.
//   The other wavefronts write the results two steps later: they keep the candidates in position order, each with the slot that holds it,
// look up which slots were given away, close the gaps and append the newest.
//   Step t, first part: cut found | slots given away at t - 1 filled | step t - 2 written.  Second part: who goes, the others counted for
// t + 1 | the newest counted, the gaps of t - 1 looked up.
//   us a step, and with all candidates moved in order at every step (golden_trace_ordered_kernel, four barriers beside those of a range_select):
//     8 groups of 2048 pairs, L = 128: 2.3 and 4.9; 4 of 512, L = 32: 1.4 and 3.4; 8 of 1024, L = 64: 1.6 and 4.3; 8 of 4096, L = 128: 3.6 and 6.8
//     the cut always among hundreds of equal keys: 4.1 and 4.7, 2.6 and 3.7, 3.1 and 4.0, 6.1 and 6.9
//     every step's scores at another scale, the cut never near the last one: 5.1 and 4.9, 3.3 and 3.4, 3.8 and 4.1, 7.3 and 6.7
// What is left is the issue of some 4000 instructions on one CU.  Measured and not kept: the writing wavefronts load the next scores in
// position order for all (3.1: their instructions cost more than the scattered loads); 256 bins (the cut leaves them).  Counting again
// with returned places also over all keys (the whole range rarely has a bin of eight), with a vote per slot for equal bins, and a second
// histogram instead of the gathered 64: 4.8, 2.8 and 7.5 among equal keys, 6.0, 3.2 and 9.3 at another scale every step.
// PER: slots of a holding thread.
struct TraceLds {   // byte offsets in the dynamic LDS
    int sorted, fresh, fresh_slot, gone, bytes;
};
__host__ __device__ inline TraceLds trace_lds(int budget, int L) {
    TraceLds s;
    s.sorted = kTrBins * kTrCap * 8;          // [kTrBins][kTrCap] (position, key)
    s.fresh = s.sorted + 8 * budget;          // [budget] (position, slot) of the candidates in position order
    s.fresh_slot = s.fresh + 16 * L;          // [2][L] keys of the newest pairs at the next two steps
    s.gone = s.fresh_slot + 4 * L;            // [2][L] uint16_t slots that the newest pairs took
    s.bytes = s.gone + budget;                // [budget] uint8_t the slot was given away
    return s;
}

// Where the count over the bins from the bottom reaches E; one wavefront.  bin < 0: it does not.
struct TraceCut {
    int bin;
    uint32_t want, inbin, near, all;   // number of the cut in its bin, pairs of the bin, pairs of the eight bins around it, of all bins
};
__device__ __forceinline__ TraceCut trace_cut(const uint32_t* hist, uint32_t E, int lane) {
    const uint4 a = *reinterpret_cast<const uint4*>(hist + 8 * lane), b = *reinterpret_cast<const uint4*>(hist + 8 * lane + 4);
    const uint32_t c[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
    const uint32_t tot = ((c[0] + c[1]) + (c[2] + c[3])) + ((c[4] + c[5]) + (c[6] + c[7]));
    const uint32_t incl = wave_scan_incl(tot);
    uint32_t left = E - (incl - tot);   // number of the cut from this lane's first pair on
    const unsigned long long who = __ballot(left - 1u < tot);   // 1 <= left <= tot: one lane, or none
    const uint32_t all = __builtin_amdgcn_readlane(incl, kWave - 1);
    if (who == 0) return {-1, 0, 0, 0, all};
    uint32_t sub = 0, in = c[0];
#pragma unroll
    for (int j = 1; j < 8; ++j) {   // past the bins below it
        const bool on = left > in && sub == (uint32_t)j - 1;
        left = on ? left - in : left;
        sub = on ? j : sub;
        in = on ? c[j] : in;
    }
    const int src = __ffsll((long long)who) - 1;
    return {8 * src + (int)__builtin_amdgcn_readlane(sub, src), (uint32_t)__builtin_amdgcn_readlane(left, src),
            (uint32_t)__builtin_amdgcn_readlane(in, src), (uint32_t)__builtin_amdgcn_readlane(tot, src), all};
}
// the want-th lowest of a bin's pairs (inbin <= kTrCap of them): key and position
__device__ __forceinline__ uint2 trace_rank(const uint2* bin, uint32_t inbin, uint32_t want, int lane) {
    const uint2 e = bin[lane & (kTrCap - 1)];
    const unsigned long long me = (unsigned long long)e.y << 32 | e.x;
    uint32_t rank = 0;
#pragma unroll
    for (int q = 0; q < kTrCap; q += 2) {
        const uint4 o = *reinterpret_cast<const uint4*>(bin + q);
        rank += ((unsigned long long)o.y << 32 | o.x) < me && (uint32_t)q < inbin;
        rank += ((unsigned long long)o.w << 32 | o.z) < me && (uint32_t)q + 1 < inbin;
    }
    const int at = __ffsll((long long)__ballot((uint32_t)lane < inbin && rank == want - 1)) - 1;   // one lane: all differ
    return make_uint2(__builtin_amdgcn_readlane(e.y, at), __builtin_amdgcn_readlane(e.x, at));
}

template <int PER>
__global__ __launch_bounds__(kTrThreads) void golden_trace_kernel(const float* __restrict__ alpha, int Tn, int M, int budget, int L,
                                                                  int32_t* __restrict__ kept) {
    constexpr int ORD = PER + (PER + 6) / 7;   // ordered entries of a writing thread: seven wavefronts' for eight's slots
    static_assert(ORD * kTrWrite >= PER * kTrHold, "a place for every candidate");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const TraceLds off = trace_lds(budget, L);
    uint2* s_bin = reinterpret_cast<uint2*>(smem);
    uint2* s_sorted = reinterpret_cast<uint2*>(smem + off.sorted);
    uint2* s_fresh = reinterpret_cast<uint2*>(smem + off.fresh);
    uint16_t* s_fresh_slot = reinterpret_cast<uint16_t*>(smem + off.fresh_slot);
    uint8_t* s_gone = smem + off.gone;
    __shared__ __attribute__((aligned(16))) uint32_t s_hist[3][kTrBins];   // this step's, the next one's; of a recount, zero in between
    // [0] key and [1] position of the highest pair that goes | [2] found: 2 among equal keys | [3] shift of the bins, [4] first key of the
    // bins | not found: the cut is number [5] of the [0] pairs (all ones: it is not known how many) with the [7] keys after [6]; [1]: these
    // are the only keys in its bin, perhaps
    __shared__ __attribute__((aligned(16))) uint32_t s_cut[8];
    __shared__ uint32_t s_taken[2], s_lo, s_hi, s_count[kTrWriteWaves];
    const int hp = blockIdx.x, k = budget - L, wave = threadIdx.x / kWave;
    constexpr int HOLD = kTrHold / kWave;   // wavefronts 0 .. HOLD - 1 hold the candidates, HOLD finds the cut, the others write
    const bool holds = wave < HOLD, cuts = wave == HOLD;
    const float* al = alpha + (size_t)hp * M * Tn;
    int32_t* out = kept + (size_t)hp * M * budget;
    if (k == 0) {   // only the newest stay
        for (int t = 1; t <= M; ++t)
            for (int j = threadIdx.x; j < L; j += kTrThreads) out[(size_t)(t - 1) * budget + j] = budget + (t - 1) * L + j;
        return;
    }
    // Holding threads: position (descending) and key of a candidate (slots without one: all ones, above every candidate), its next key and
    // the score it comes from.  Writing threads: position and slot of the ordered entries, the next two scores of the newest pairs.
    constexpr int FR = ORD < kTrFresh ? ORD : kTrFresh, NX = PER > FR ? PER : FR;   // FR: newest pairs of a writing thread
    uint32_t np[ORD], key[ORD], key_next[PER], gone = 0;   // gone: a bit for every slot given away
    float next[NX], next2[FR];
    {
        const int tid = threadIdx.x;
        for (int j = tid; j < budget; j += kTrThreads) {
            s_sorted[j] = make_uint2(j, j);
            s_gone[j] = 0;
        }
        static_assert(3 * kTrBins <= 2 * kTrThreads, "");
        for (int i = tid; i < 3 * kTrBins; i += kTrThreads) s_hist[i / kTrBins][i % kTrBins] = 0;
        if (tid < 2) s_taken[tid] = 0;
        if (tid == 0) {
            s_lo = 0xffffffffu;
            s_hi = 0;
            s_cut[0] = ~0u;
            s_cut[1] = 0;
            s_cut[2] = 0;   // the first step has no bins
            s_cut[3] = 0;
            s_cut[5] = (uint32_t)L;
            s_cut[6] = 0;
            s_cut[7] = kTrDown;
        }
#pragma unroll
        for (int u = 0; u < ORD; ++u) {
            const int i = u * kTrHold + tid, j = u * kTrWrite + tid - kTrHold - kWave;
            const bool candidate = holds && u < PER && i < budget;
            np[u] = candidate ? kTrDown - (uint32_t)i : 0xffffffffu;
            key[u] = candidate ? score_key(al[i]) : 0xffffffffu;
            if (u < PER) key_next[u] = 0xffffffffu;
            if (u < NX) {
                next[u] = 0.f;
                if (candidate && M > 1) next[u] = al[Tn + i];
                if (wave > HOLD && u < FR && j < L && M > 1) next[u] = al[Tn + budget + j];
            }
            if (u < FR) {
                next2[u] = 0.f;
                if (wave > HOLD && j < L && M > 2) next2[u] = al[2 * (size_t)Tn + budget + j];
            }
        }
    }
    const int stretch = ((budget + kTrWriteWaves - 1) / kTrWriteWaves + kWave - 1) / kWave * kWave;   // ordered entries of a writing wavefront
    __syncthreads();
    for (int t = 1; t <= M + 2; ++t) {   // step t is decided, step t - 2 written
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));   // opaque: what is derived from it would be kept over the whole loop, in registers that spill
        const int lane = tid & (kWave - 1), write_tid = tid - kTrHold - kWave;
        if (holds) {
            uint32_t n = 0, first = 0;
#pragma unroll
            for (int u = 0; u < PER; ++u) n += (uint32_t)__popcll(__ballot((gone >> u) & 1));
            if (lane == 0) first = atomicAdd(&s_taken[t & 1], n);
            if (tid < kTrBins) s_hist[(t + 1) & 1][tid] = 0;
            if (tid == 0) s_taken[(t + 1) & 1] = 0;
            first = __builtin_amdgcn_readfirstlane(first);
#pragma unroll
            for (int u = 0; u < PER; ++u) key_next[u] = np[u] == 0xffffffffu ? 0xffffffffu : score_key(next[u]);
            // the j-th of the slots given away at t - 1 takes the j-th of the then newest pairs (a few at a time, so that the reads overlap)
            constexpr int STEP = PER < 4 ? PER : 4;
#pragma unroll
            for (int u0 = 0; u0 < PER; u0 += STEP) {
                int j[STEP];
                uint2 f[STEP];
#pragma unroll
                for (int v = 0; v < STEP; ++v) {
                    const unsigned long long all = __ballot((gone >> (u0 + v)) & 1);
                    j[v] = min((int)(first + __builtin_amdgcn_mbcnt_hi((uint32_t)(all >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)all, 0))), L - 1);
                    first += (uint32_t)__popcll(all);
                    f[v] = s_fresh[((t - 1) & 1) * L + j[v]];
                }
#pragma unroll
                for (int v = 0; v < STEP; ++v) {
                    const int u = u0 + v;
                    const bool g = (gone >> u) & 1;
                    np[u] = g ? kTrDown - (uint32_t)(budget + (t - 2) * L + j[v]) : np[u];
                    key[u] = g ? f[v].x : key[u];
                    key_next[u] = g ? f[v].y : key_next[u];
                    if (g) {
                        s_gone[u * kTrHold + tid] = 1;
                        s_fresh_slot[((t - 1) & 1) * L + j[v]] = (uint16_t)(u * kTrHold + tid);
                    }
                }
            }
        } else if (cuts) {
            if (t > 1 && t <= M) {
                __builtin_amdgcn_s_setprio(3);   // everything waits for this
                int shift = (int)s_cut[3];
                const TraceCut c = trace_cut(s_hist[t & 1], (uint32_t)L, lane);
                if (c.bin > 0 && c.inbin <= (uint32_t)kTrCap && !(c.bin == kTrCut && s_cut[2] == 2)) {   // (pairs counted by vote are not listed)
                    const uint2 T = trace_rank(s_bin + c.bin * kTrCap, c.inbin, c.want, lane);
                    if (c.near > 24 && shift > 0) --shift;
                    else if (c.near < 6 && shift < 22) ++shift;
                    if (lane == 0) {
                        *reinterpret_cast<uint4*>(s_cut) = make_uint4(T.x, T.y, 1u, (uint32_t)shift);
                        s_cut[4] = __builtin_elementwise_sub_sat(T.x, (uint32_t)kTrCut << shift);
                    }
                } else if (lane == 0) {
                    const bool in = c.bin > 0, guess = c.bin == kTrCut && s_cut[2] == 2 && c.inbin > (uint32_t)kWave && (s_cut[0] - s_cut[4]) >> shift == (uint32_t)kTrCut;
                    const uint32_t lo = guess ? s_cut[0] : in ? s_cut[4] + ((uint32_t)c.bin << shift) : 0u;
                    *reinterpret_cast<uint4*>(s_cut) = make_uint4(in ? c.inbin : ~0u, guess, 0u, (uint32_t)shift);
                    s_cut[5] = in ? c.want : (uint32_t)L;
                    s_cut[6] = lo;
                    s_cut[7] = guess ? 0u : in ? min((1u << shift) - 1u, kTrDown - lo) : kTrDown;
                }
                __builtin_amdgcn_s_setprio(0);
            }
        } else {
            if (t > 2) {   // step t - 2: those that stayed, in order, then the newest
                int32_t* row = out + (size_t)(t - 3) * budget;
                const int new0 = budget + (t - 3) * L;
                uint32_t before = 0;
#pragma unroll
                for (int w = 0; w < kTrWriteWaves; ++w) before += w < wave - HOLD - 1 ? s_count[w] : 0u;
#pragma unroll
                for (int u = 0; u < ORD; ++u) {
                    const bool stays = (key[u] & kStays) != 0;
                    const unsigned long long all = __ballot(stays);
                    if (stays) {
                        const uint32_t dst = before + __builtin_amdgcn_mbcnt_hi((uint32_t)(all >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)all, 0));
                        s_sorted[dst] = make_uint2(np[u], key[u] & ~kStays);
                        row[dst] = (int32_t)np[u];
                    }
                    before += (uint32_t)__popcll(all);
                }
#pragma unroll
                for (int u = 0; u < FR; ++u) {
                    if (u * kTrWrite >= L) break;
                    const int j = u * kTrWrite + write_tid;
                    if (j < L) {
                        s_sorted[k + j] = make_uint2((uint32_t)(new0 + j), s_fresh_slot[(t & 1) * L + j]);
                        row[k + j] = new0 + j;
                    }
                }
            }
            if (t < M) {
#pragma unroll
                for (int u = 0; u < FR; ++u) {
                    if (u * kTrWrite >= L) break;
                    const int j = u * kTrWrite + write_tid;
                    if (j < L) s_fresh[(t & 1) * L + j] = make_uint2(score_key(next[u]), score_key(next2[u]));
                }
            }
        }
        __syncthreads();
        if (__builtin_expect(t <= M && s_cut[2] == 0, 0)) {
            // count the pairs that are left over their own range, of the keys or, if those are equal, of the positions, until they can be ranked
            uint32_t want = s_cut[5], in = s_cut[0], klo = s_cut[6], kspan = s_cut[7];
            uint32_t plo = kTrDown - (uint32_t)(budget + (t - 1) * L - 1), pspan = kTrDown - plo;
            uint32_t* hist = s_hist[2];
            int shift = (int)s_cut[3];
            bool whole = in == ~0u, first = true, guess = s_cut[1] != 0;
            constexpr int STEP = PER < 4 ? PER : 4;   // atomics in flight
            auto member = [&](int u) { return (key[u] - klo <= kspan) & (np[u] - plo <= pspan); };
            for (;;) {
                if (in <= (uint32_t)kWave) {   // few enough for one wavefront
                    if (holds) {
#pragma unroll
                        for (int u0 = 0; u0 < PER; u0 += STEP) {
                            uint32_t place[STEP];
#pragma unroll
                            for (int v = 0; v < STEP; ++v) {
                                place[v] = (uint32_t)kWave;
                                if (member(u0 + v)) place[v] = atomicAdd(&hist[0], 1u);
                            }
#pragma unroll
                            for (int v = 0; v < STEP; ++v)
                                if (place[v] < (uint32_t)kWave) s_bin[place[v]] = make_uint2(np[u0 + v], key[u0 + v]);
                        }
                    }
                    __syncthreads();
                    if (cuts) {
                        const uint2 e = s_bin[lane];
                        in = hist[0];
                        const unsigned long long me = (unsigned long long)e.y << 32 | e.x;
                        uint32_t rank = 0;
#pragma unroll 4
                        for (uint32_t q = 0; q < in; q += 2) {
                            const uint4 o = *reinterpret_cast<const uint4*>(s_bin + q);
                            rank += ((unsigned long long)o.y << 32 | o.x) < me;
                            rank += ((unsigned long long)o.w << 32 | o.z) < me && q + 1 < in;
                        }
                        const int at = __ffsll((long long)__ballot((uint32_t)lane < in && rank == want - 1)) - 1;   // one lane: all differ
                        const uint32_t T = __builtin_amdgcn_readlane(e.y, at), p = __builtin_amdgcn_readlane(e.x, at);
                        const bool equal = __ballot((uint32_t)lane < in && e.y != T) == 0;
                        if (first && !equal) shift = max(shift - (30 - __clz((int)in)), 0);   // (it was this step's bin)
                        if (lane == 0) {
                            *reinterpret_cast<uint4*>(s_cut) = make_uint4(T, p, equal ? 2u : 1u, (uint32_t)shift);
                            s_cut[4] = __builtin_elementwise_sub_sat(T, (uint32_t)kTrCut << shift);
                            hist[0] = 0;
                        }
                    }
                    __syncthreads();
                    break;
                }
                if (kspan != 0) {
                    uint32_t lo = 0xffffffffu, hi = 0;
                    if (holds) {
#pragma unroll
                        for (int u = 0; u < PER; ++u) {
                            const uint32_t d = key[u] - klo;
                            lo = min(lo, d);   // (others are beyond the span)
                            hi = max(hi, d <= kspan ? d : 0u);
                        }
                        wave_min_max(lo, hi);
                        if (lane == 0) {
                            atomicMin(&s_lo, lo);
                            atomicMax(&s_hi, hi);
                        }
                    }
                    __syncthreads();
                    klo += s_lo;
                    kspan = s_hi - s_lo;
                }
                const bool by_key = kspan != 0;
                const uint32_t from = by_key ? klo : plo, span = by_key ? kspan : pspan;
                const int sh = max(23 - __clz((int)span | 1), 0);   // span >> sh < 512
                if (holds) {
                    if (whole && by_key) {   // (hardly ever few to a bin)
#pragma unroll
                        for (int u = 0; u < PER; ++u)
                            if (key[u] - klo <= kspan) atomicAdd(&hist[(key[u] - klo) >> sh], 1u);
                    } else {
#pragma unroll
                        for (int u0 = 0; u0 < PER; u0 += STEP) {
                            uint32_t bin[STEP], place[STEP];
#pragma unroll
                            for (int v = 0; v < STEP; ++v) {
                                bin[v] = ((by_key ? key[u0 + v] : np[u0 + v]) - from) >> sh;
                                place[v] = (uint32_t)kTrCap;
                                if (member(u0 + v)) place[v] = atomicAdd(&hist[bin[v]], 1u);
                            }
#pragma unroll
                            for (int v = 0; v < STEP; ++v)
                                if (place[v] < (uint32_t)kTrCap) s_bin[bin[v] * kTrCap + place[v]] = make_uint2(np[u0 + v], key[u0 + v]);
                        }
                    }
                }
                __syncthreads();
                if (cuts) {
                    const TraceCut c = trace_cut(hist, want, lane);
                    if (guess && c.all != in) {   // other keys beside it
                        if (lane == 0) {
                            const uint32_t lo = s_cut[4] + ((uint32_t)kTrCut << shift);
                            s_cut[6] = lo;
                            s_cut[7] = min((1u << shift) - 1u, kTrDown - lo);
                        }
                    } else {   // it is there
                        const bool found = c.inbin <= (uint32_t)kTrCap && !(whole && by_key);
                        uint2 T = make_uint2(c.inbin, 0u);
                        if (found) T = trace_rank(s_bin + c.bin * kTrCap, c.inbin, c.want, lane);
                        // the next step's bins: two or three pairs to one
                        if (by_key && c.inbin > (uint32_t)kTrCap) shift = min(max(sh - (30 - __clz((int)c.inbin)), 0), 22);
                        else if (by_key && whole) shift = min(sh, 22);
                        if (lane == 0) {
                            const uint32_t lo = (uint32_t)c.bin << sh;
                            *reinterpret_cast<uint4*>(s_cut) = make_uint4(T.x, T.y, found ? by_key ? 1 : 2 : 0, (uint32_t)shift);
                            s_cut[5] = c.want;
                            s_cut[6] = from + lo;
                            s_cut[7] = min((1u << sh) - 1u, span - lo);
                            if (found) s_cut[4] = __builtin_elementwise_sub_sat(T.x, (uint32_t)kTrCut << shift);
                        }
                    }
                    if (lane == 0) {
                        s_lo = 0xffffffffu;
                        s_hi = 0;
                    }
#pragma unroll
                    for (int i = 0; i < kTrBins; i += 4 * kWave) *reinterpret_cast<uint4*>(hist + i + 4 * lane) = make_uint4(0, 0, 0, 0);
                }
                __syncthreads();
                const uint4 c0 = *reinterpret_cast<const uint4*>(s_cut), c1 = *reinterpret_cast<const uint4*>(s_cut + 4);   // (written again after another barrier)
                if (c0.z != 0) break;
                in = c0.x;
                want = c1.y;
                if (by_key || (guess && c0.y != 0)) {
                    klo = c1.z;
                    kspan = c1.w;
                } else {
                    plo = c1.z;
                    pspan = c1.w;
                }
                whole = first = guess = false;
            }
        }
        if (cuts) {
            if (t < M) {   // the newest pairs are candidates of step t + 1
                const uint32_t base = s_cut[4], shift = s_cut[3];
                uint32_t* hist = s_hist[(t + 1) & 1];
                uint32_t low = 0;
                for (int j0 = 0; j0 < L; j0 += kWave) {
                    const int j = min(j0 + lane, L - 1);
                    const uint32_t x = s_fresh[(t & 1) * L + j].x, bin = j0 + lane < L ? __builtin_elementwise_sub_sat(x, base) >> shift : (uint32_t)kTrBins;
                    low += (uint32_t)__popcll(__ballot(bin == 0));
                    if (bin - 1u < (uint32_t)(kTrBins - 1)) {
                        const uint32_t place = atomicAdd(&hist[bin], 1u);
                        if (place < (uint32_t)kTrCap) s_bin[bin * kTrCap + place] = make_uint2(kTrDown - (uint32_t)(budget + (t - 1) * L + j), x);
                    }
                }
                if (lane == 0 && low) atomicAdd(&hist[0], low);
            }
        } else if (holds) {
            gone = 0;
            if (t <= M) {
                const uint4 c4 = *reinterpret_cast<const uint4*>(s_cut);
                const uint32_t base = s_cut[4];
                const unsigned long long cut = (unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane(c4.x) << 32 | (uint32_t)__builtin_amdgcn_readfirstlane(c4.y);
                const int shift = __builtin_amdgcn_readfirstlane(c4.w);
                const float* after = al + (size_t)(t + 1) * Tn;   // scores of step t + 2
                uint32_t* hist = s_hist[(t + 1) & 1];
                uint32_t low = 0, equal = 0;
                const bool crowd = c4.z == 2;   // the cut went through equal keys: atomics on one word take turns, so they are counted by vote
                constexpr int STEP = PER < 4 ? PER : 4;
#pragma unroll
                for (int u0 = 0; u0 < PER; u0 += STEP) {
                    uint32_t bin[STEP], place[STEP];
#pragma unroll
                    for (int v = 0; v < STEP; ++v) {
                        const int u = u0 + v;
                        const bool g = ((unsigned long long)key[u] << 32 | np[u]) <= cut;
                        gone |= g ? 1u << u : 0u;
                        key[u] = key_next[u];
                        bin[v] = __builtin_elementwise_sub_sat(key[u], base) >> shift;
                        bin[v] = g ? (uint32_t)kTrBins : bin[v];
                        low += (uint32_t)__popcll(__ballot(bin[v] == 0));
                        if (crowd) {
                            equal += (uint32_t)__popcll(__ballot(bin[v] == (uint32_t)kTrCut));
                            bin[v] = bin[v] == (uint32_t)kTrCut ? (uint32_t)kTrBins : bin[v];
                        }
                        place[v] = kTrCap;
                        if (bin[v] - 1u < (uint32_t)(kTrBins - 1)) place[v] = atomicAdd(&hist[bin[v]], 1u);
                    }
#pragma unroll
                    for (int v = 0; v < STEP; ++v)
                        if (place[v] < (uint32_t)kTrCap) s_bin[bin[v] * kTrCap + place[v]] = make_uint2(np[u0 + v], key[u0 + v]);
                    if (t + 2 <= M) {
#pragma unroll
                        for (int v = 0; v < STEP; ++v)
                            if (np[u0 + v] != 0xffffffffu) next[u0 + v] = after[kTrDown - np[u0 + v]];
                    }
                }
                if (lane == 0 && low) atomicAdd(&hist[0], low);
                if (lane == 0 && equal) atomicAdd(&hist[kTrCut], equal);
            }
        } else {
            if (t > 1 && t <= M + 1) {   // which of the ordered candidates of step t - 1 stayed
                const int w = wave - HOLD - 1, w0 = min(w * stretch, budget), w1 = min(w0 + stretch, budget);
                uint8_t g[ORD];
                uint32_t n = 0;
#pragma unroll
                for (int u = 0; u < ORD; ++u) {
                    const uint2 e = s_sorted[min(w0 + u * kWave + lane, budget - 1)];
                    np[u] = e.x;
                    key[u] = e.y;
                }
#pragma unroll
                for (int u = 0; u < ORD; ++u) g[u] = s_gone[key[u]];
#pragma unroll
                for (int u = 0; u < ORD; ++u) {
                    const bool live = w0 + u * kWave + lane < w1;
                    if (live && g[u]) s_gone[key[u]] = 0;
                    n += (uint32_t)__popcll(__ballot(live && !g[u]));
                    if (live && !g[u]) key[u] |= kStays;
                }
                if (lane == 0) s_count[w] = n;
            }
#pragma unroll
            for (int u = 0; u < FR; ++u) {   // scores at steps t + 2 and t + 3 of the pairs that are the newest at step t + 1
                if (u * kTrWrite >= L) break;
                const int j = u * kTrWrite + write_tid;
                if (j < L && t + 2 <= M) next[u] = al[(size_t)(t + 1) * Tn + budget + t * L + j];
                if (j < L && t + 3 <= M) next2[u] = al[(size_t)(t + 2) * Tn + budget + t * L + j];
            }
        }
        __syncthreads();
    }
}

// Budgets beyond kTraceSlots, whose slots do not fit the registers (4 groups of 8000, L = 256: 12.3 us a step; with sixteen slots a
// thread, 180 registers of them spilled, 10 to 30), and intervals beyond what the writing threads hold (kTrFresh each).  One workgroup per
// KV group.  LDS holds the cache's positions (ascending; B + L of them: the B of this step and the L that are generated before the next
// one) and the keys of its first B entries under this step's future scores.
// A step: (1) the loads of the NEXT step's future scores at every position that can still be a candidate then are
// issued (they land while the step selects); (2) range_select finds the key of the (B - L)-th best candidate;
// (3) every wavefront walks its own contiguous stretch of the candidates, first to count its survivors, then, with
// the counts of the stretches before it, to move them (position and next key) to the front in order.  Sources are
// in registers before the barrier that precedes the moves, so the compaction is safe in place.
// PER_LANE: candidates one lane holds (stretch of a wavefront / 64) and newest pairs one thread holds (L / 1024), at most.  Four where that
// is enough: 8 groups of 4096, L = 2304: 8.1 us a step, 10.9 with twelve; 4 of 2500, L = 2400: 6.0 and 8.8.
template <int PER_LANE>
__global__ __launch_bounds__(kSelThreads) void golden_trace_ordered_kernel(const float* __restrict__ alpha, int Tn, int M,
                                                                   int budget, int L, int32_t* __restrict__ kept) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    int32_t* s_pos = reinterpret_cast<int32_t*>(smem);                 // [budget + L]
    uint32_t* s_key = reinterpret_cast<uint32_t*>(s_pos + budget + L);  // [budget]
    __shared__ __attribute__((aligned(16))) uint32_t s_range[kRangeWords];   // zero at the start of every step
    __shared__ __attribute__((aligned(16))) uint32_t s_hist[4 * 256];
    __shared__ uint32_t s_wtot[2 * kSelWaves];
    __shared__ uint32_t s_wmm[2 * kSelWaves];   // every wavefront's smallest and largest key of those it wrote for the next step
    const int hp = blockIdx.x, lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int k = budget - L;  // old pairs that stay
    const float* al = alpha + (size_t)hp * M * Tn;
    for (int j = threadIdx.x; j < budget + L; j += kSelThreads) s_pos[j] = j;
    // the range of the next step's keys is gathered while they are written
    uint32_t key_lo = 0xffffffffu, key_hi = 0;
    for (int j = threadIdx.x; j < budget; j += kSelThreads) {
        const uint32_t key = score_key(al[j]);
        s_key[j] = key;
        key_lo = min(key_lo, key);
        key_hi = max(key_hi, key);
    }
    auto publish_range = [&]() {
        wave_min_max(key_lo, key_hi);
        if (lane == 0) {
            s_wmm[2 * wave] = key_lo;
            s_wmm[2 * wave + 1] = key_hi;
        }
    };
    publish_range();
    for (int i = threadIdx.x; i < kRangeWords; i += kSelThreads) s_range[i] = 0;
    __syncthreads();
    const int stretch = ((budget + kSelWaves - 1) / kSelWaves + kWave - 1) / kWave * kWave;  // <= 64 * PER_LANE (host)
    for (int t = 1; t <= M; ++t) {
        int tid = threadIdx.x;
        // opaque: what is derived from it would be kept over the whole loop, 121 registers spilled
        if constexpr (PER_LANE > 4) asm volatile("" : "+v"(tid));
        const int lane = tid & (kWave - 1), wave = tid / kWave, w0 = min(wave * stretch, budget), w1 = min(w0 + stretch, budget);
        int32_t* out = kept + ((size_t)hp * M + (t - 1)) * budget;
        const bool more = t < M;
        const float* aln = al + (size_t)t * Tn;   // future scores of step t + 1
        const int new0 = budget + (t - 1) * L;   // first of the L newest pairs (they stay)
        key_lo = 0xffffffffu;
        key_hi = 0;
#pragma unroll
        for (int w = 0; w < kSelWaves; ++w) {
            key_lo = min(key_lo, s_wmm[2 * w]);
            key_hi = max(key_hi, s_wmm[2 * w + 1]);
        }
        float nxt[PER_LANE], nxt_new[PER_LANE];
#pragma unroll
        for (int u = 0; u < PER_LANE; ++u) {
            const int i = w0 + u * kWave + lane, j = tid + u * kSelThreads;
            nxt[u] = more && i < w1 ? aln[s_pos[i]] : 0.f;
            nxt_new[u] = more && j < L ? aln[new0 + j] : 0.f;
        }
        uint32_t Tk = 0, want = 0, gt = 0, eq = 0;
        uint32_t kv[PER_LANE];
        int32_t pv[PER_LANE];
        if (k > 0) {
            range_select<kSelThreads, 2, true>([&](int i, bool& valid) { valid = true; return s_key[i]; }, budget, (uint32_t)k, s_range, s_hist, s_wtot,
                                               range_plan(key_lo, key_hi), tid, &Tk, &want);
#pragma unroll
            for (int u = 0; u < PER_LANE; ++u) {
                const int i = w0 + u * kWave + lane;
                const bool live = i < w1;
                kv[u] = live ? s_key[i] : 0u;
                pv[u] = live ? s_pos[i] : 0;
                gt += (uint32_t)__popcll(__ballot(live && kv[u] > Tk));
                eq += (uint32_t)__popcll(__ballot(live && kv[u] == Tk));
            }
            if (lane == 0) {
                s_wtot[2 * wave] = gt;
                s_wtot[2 * wave + 1] = eq;
            }
        }
        __syncthreads();  // every source is in registers, the counts are visible, the histogram has been read
        for (int i = tid; i < kRangeWords; i += kSelThreads) s_range[i] = 0;
        key_lo = 0xffffffffu;
        key_hi = 0;
        if (k > 0) {
            uint32_t gt_run = 0, eq_run = 0;
            for (int w = 0; w < wave; ++w) {
                gt_run += s_wtot[2 * w];
                eq_run += s_wtot[2 * w + 1];
            }
#pragma unroll
            for (int u = 0; u < PER_LANE; ++u) {
                const int i = w0 + u * kWave + lane;
                const bool live = i < w1;
                const unsigned long long mg = __ballot(live && kv[u] > Tk), me = __ballot(live && kv[u] == Tk);
                const uint32_t gb = gt_run + __builtin_amdgcn_mbcnt_hi((uint32_t)(mg >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mg, 0));
                const uint32_t eb = eq_run + __builtin_amdgcn_mbcnt_hi((uint32_t)(me >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)me, 0));
                const bool keep = live && (kv[u] > Tk || (kv[u] == Tk && eb < want));
                if (keep) {
                    const uint32_t dst = gb + min(eb, want);
                    const uint32_t key = score_key(nxt[u]);
                    s_pos[dst] = pv[u];
                    s_key[dst] = key;
                    key_lo = min(key_lo, key);
                    key_hi = max(key_hi, key);
                    out[dst] = pv[u];
                }
                gt_run += (uint32_t)__popcll(mg);
                eq_run += (uint32_t)__popcll(me);
            }
        }
        // the L newest stay; then the L pairs generated before the next step join
#pragma unroll
        for (int u = 0; u < PER_LANE; ++u) {
            const int j = tid + u * kSelThreads;
            if (j < L) {
                out[k + j] = new0 + j;
                s_pos[k + j] = new0 + j;
                const uint32_t key = score_key(nxt_new[u]);
                s_key[k + j] = key;
                key_lo = min(key_lo, key);
                key_hi = max(key_hi, key);
                s_pos[k + L + j] = new0 + L + j;
            }
        }
        publish_range();
        __syncthreads();
    }
}

static int golden_steps(int T, int B, int L) {
    const int m = (T - B + L - 1) / L - 1;
    return m < 0 ? 0 : m;
}

}  // namespace fk

using namespace fk;

extern "C" int32_t fk_golden_steps(int32_t T, int32_t budget, int32_t interval) {
    if (T <= 0 || budget <= 0 || interval <= 0 || interval > budget) return -1;
    return golden_steps(T, budget, interval);
}

extern "C" fk_status fk_golden_scores(const void* A, int32_t dtype, int32_t n_q_heads, int32_t n_kv_heads, int32_t T,
                                      int64_t ld, int32_t budget, int32_t interval, float* block_scores, float* alpha,
                                      void* stream) {
    if (!A || !block_scores || !alpha) return FK_ERR_INVALID_ARG;
    if (n_q_heads <= 0 || n_kv_heads <= 0 || n_q_heads % n_kv_heads != 0 || T <= 0 || ld < T) return FK_ERR_INVALID_ARG;
    if (budget <= 0 || interval <= 0 || interval > budget) return FK_ERR_INVALID_ARG;
    if (dtype != FK_F32 && dtype != FK_BF16) return FK_ERR_UNSUPPORTED;
    if (ld % 8 != 0 || !aligned16(A)) return FK_ERR_INVALID_ARG;
    const int M = golden_steps(T, budget, interval);
    if (M == 0) return FK_OK;
    if (M > 65535 || n_kv_heads > 65535) return FK_ERR_UNSUPPORTED;
    const int g = n_q_heads / n_kv_heads;
    hipStream_t st = (hipStream_t)stream;
    auto pool = [&](auto kern, auto* a, int lanes) {
        const int tile = lanes * 16 / (int)sizeof(*a);
        const int most = 2 * ((T + tile - 1) / tile), pair = (int)((2ll * budget + (M + 3ll) * interval) / tile) + 2;   // live tiles of two blocks
        hipLaunchKernelGGL(kern, dim3(pair < most ? pair : most, (M + 1) / 2, n_kv_heads), dim3(kPoolThreads), 0, st, a, g, T, (size_t)ld, budget, interval, M, block_scores);
    };
    // How wide a workgroup's tile is, 1 KB, 512 or 256 bytes of a row, by some 440 shapes of 1000 to 8192 tokens, 1 to 64 heads, blocks of 16 to 256.
    // Wide ones waste the least where rows do not start on a line of 128 bytes (32 heads of 5001 tokens, L = 32: 176 us, 512 bytes 185, 256 bytes
    // 205; 8 of 5200, L = 250: 35, 39 and 46) and leave a short block's workgroups the most to do (8 heads of 4096, L = 32: 47, 62 and 92).  256 bytes
    // where wider ones would leave CUs idle (one group of 2500 tokens, L = 1000: 28, 512 bytes 37, 1 KB 58; 8 heads of 1532, L = 128: 8.6, 10.9 and
    // 16.4) and for large blocks (32 heads of 5504, L = 250: 173, 187 and 185), but where all rows start on the same channels, at a multiple of
    // 1 KB, 512 bytes are spread best (32 heads of 8192: 338, 324 and 343), as they are for blocks of few (head, query) pairs (8 heads of 1856, L =
    // 32: 11.4, 10.7 and 13.1).
    const size_t row_bytes = (size_t)T * (dtype == FK_F32 ? 4 : 2), pitch = (size_t)ld * (dtype == FK_F32 ? 4 : 2);
    const long long wide = (long long)((row_bytes + 1023) / 1024) * M * n_kv_heads, pairs = (long long)g * interval;
    const bool lines = pitch % 128 == 0;
    const int lanes = wide < 128 || (pairs >= 96 && wide < (lines ? 256 : 192)) ? 16
                      : pairs < 96 || !lines                                    ? 64
                      : pitch % 1024 == 0 || pairs < 192                        ? 32
                                                                                : 16;
    if (dtype == FK_F32) {
        const float* a = static_cast<const float*>(A);
        if (lanes == 16) pool(golden_pool_kernel<float, 16>, a, 16);
        else if (lanes == 32) pool(golden_pool_kernel<float, 32>, a, 32);
        else pool(golden_pool_kernel<float, 64>, a, 64);
    } else {
        const bf16_t* a = static_cast<const bf16_t*>(A);
        if (lanes == 16) pool(golden_pool_kernel<bf16_t, 16>, a, 16);
        else if (lanes == 32) pool(golden_pool_kernel<bf16_t, 32>, a, 32);
        else pool(golden_pool_kernel<bf16_t, 64>, a, 64);
    }
    hipLaunchKernelGGL((M <= 8 ? golden_future_kernel<8> : M <= 16 ? golden_future_kernel<16> : golden_future_kernel<32>), dim3((T + 255) / 256, n_kv_heads), dim3(256), 0, st, block_scores, T, M, alpha);
    return launch_status();
}

extern "C" fk_status fk_golden_trace(const float* alpha, int32_t n_kv_heads, int32_t T, int32_t budget, int32_t interval,
                                     int32_t* kept, void* stream) {
    if (!alpha || !kept) return FK_ERR_INVALID_ARG;
    if (n_kv_heads <= 0 || T <= 0 || budget <= 0 || interval <= 0 || interval > budget) return FK_ERR_INVALID_ARG;
    if (budget + interval > kTraceMaxCache) return FK_ERR_UNSUPPORTED;
    const int M = golden_steps(T, budget, interval);
    if (M == 0) return FK_OK;
    auto launch = [&](auto kern, bool (&lds_ok)[kMaxDevices], size_t lds, size_t most) -> fk_status {
        if (!allow_dynamic_lds((const void*)kern, most, lds_ok)) return FK_ERR_LAUNCH;
        hipLaunchKernelGGL(kern, dim3(n_kv_heads), dim3(kTrThreads), lds, (hipStream_t)stream, alpha, T, M, budget, interval, kept);
        return launch_status();
    };
    static bool ok1[kMaxDevices] = {}, ok2[kMaxDevices] = {}, ok4[kMaxDevices] = {}, ok8[kMaxDevices] = {}, ok_ordered4[kMaxDevices] = {}, ok_ordered12[kMaxDevices] = {};
    if (budget > kTraceSlots || interval > kTrWrite * kTrFresh) {
        const size_t lds = sizeof(int32_t) * ((size_t)budget + interval) + sizeof(uint32_t) * (size_t)budget;
        if (budget <= 4 * kSelThreads) return launch(golden_trace_ordered_kernel<4>, ok_ordered4, lds, sizeof(int32_t) * 2 * kTraceMaxCache);
        return launch(golden_trace_ordered_kernel<12>, ok_ordered12, lds, sizeof(int32_t) * 2 * kTraceMaxCache);   // 12 * 1024 = kTraceMaxCache
    }
    const size_t lds = (size_t)trace_lds(budget, interval).bytes;
    const int per = (budget + kTrHold - 1) / kTrHold;   // slots of a thread
    if (per <= 1) return launch(golden_trace_kernel<1>, ok1, lds, kTraceMaxLds);
    if (per <= 2) return launch(golden_trace_kernel<2>, ok2, lds, kTraceMaxLds);
    if (per <= 4) return launch(golden_trace_kernel<4>, ok4, lds, kTraceMaxLds);
    return launch(golden_trace_kernel<8>, ok8, lds, kTraceMaxLds);
}
