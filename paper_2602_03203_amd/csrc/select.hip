// fk_select_keep: deterministic per-row top-k by histogram (Section 3.1: the most recent
// L pairs stay, the others are pruned to the B - L most important; Top-K form of the
// sampling ablation).
//
// One workgroup per row.  Scores are read once, mapped to order-preserving 32-bit keys (larger key =
// more important; -0 -> +0; NaN -> 0, below -inf) and kept in LDS.  One histogram over the range of the keys and a
// short ranked list (range_select; rows beyond LDS and keys that it cannot tell apart: digit by digit, msd_select)
// find the key T of the k-th best candidate and the number `take` of candidates equal to T that still
// fit.  One ordered pass then writes the kept slots
// ascending: every candidate above T, the first `take` candidates equal to T in slot order
// (slot order is position order, so ties go to the lower position), and the protected tail.
#include "select_common.h"

namespace fk {

// LDS (u32): histogram and list of range_select | histograms [4][256] of msd_select | wavefront totals [16][2] | key range
// [kRangePart] | keys [lds_keys] | kSelMerge: their slots [lds_keys]
static constexpr int kSelMaxLdsKeys = 36 * 1024;  // 144 KB of keys beside the histograms
static constexpr int kSelLdsHead = kRangeWords + 4 * 256 + 32 + kRangePart;  // words before the keys
struct SelLds {
    uint32_t *range, *hist, *wtot, *wmm, *key;
    __device__ __forceinline__ explicit SelLds(uint32_t* mem)
        : range(mem), hist(range + kRangeWords), wtot(hist + 4 * 256), wmm(wtot + 32), key(wmm + kRangePart) {}
};
// Two workgroups of sixteen wavefronts share a CU if a wavefront takes no more than 64 vector registers and 80 scalar ones (800 of
// them a SIMD, and sixteen more for every wavefront): 512 rows of 2176 keys 12.8 -> 10.2 us with 78 instead of 93, sampled
// 22.3 -> 16.9 with 78 instead of 90 (20.1 before its range selection, with 58).  The 40 to 45 of them that are spilled to vector lanes do
// not show at 128 rows.
#define FK_TWO_PER_CU __attribute__((amdgpu_num_sgpr(80)))
// (Four wavefronts per row instead of sixteen were measured and dropped: 11.3 against 8.1 us; a pass is a chain
// key -> atomic -> barrier -> scan of LDS round trips, which more wavefronts shorten.)
//
// Long rows of a small batch (one-shot compression of a long prompt: 32 rows of 131072 pairs) would leave most of the
// chip idle with one workgroup per row, and their keys do not fit LDS.  fk_select_keep_ws splits such rows (two launches,
// a workspace between them): workgroups of select_chunk_kernel, one per chunk of a row, each keep the k best candidates of
// their chunk (any pair among the row's k best is among its chunk's k best, under the same total order); kSelMerge
// workgroups, one per row, then select among the chunks' survivors, whose keys fit LDS.  Same result, bit for bit.
enum { kSelWhole = 0, kSelMerge = 1 };
struct SelSplit {
    int nchunk;      // chunks per row
    int chunk_len;   // candidates per chunk (the last chunk runs on to the row's end)
    int32_t* count;  // [rows][nchunk] survivors of every chunk
    int32_t* cand;   // [rows][nchunk][budget - recent] their slots, ascending
};

// Keys of the scores sc[from .. ncand - 1] to LDS, eight loads in flight per thread; their range.
template <int THREADS>
__device__ __forceinline__ void keys_to_lds(const float* __restrict__ sc, int from, int ncand, uint32_t* s_key, KeyRange& kr) {
    for (int i0 = from + threadIdx.x; i0 < ncand; i0 += 8 * THREADS) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = sc[min(i0 + u * THREADS, ncand - 1)];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (i0 + u * THREADS < ncand) {
                const uint32_t key = score_key(v[u]);
                s_key[i0 + u * THREADS] = key;
                kr.add(key);
            }
        }
    }
}

// The ordered pass: of the candidates [0, ncand) those above T and the first `want` equal to T, their slots ascending.  Every
// wavefront owns one contiguous stretch and walks it 64 candidates at a time (coalesced, no barrier inside): first to count
// its kept ones (kept_count), then, with the counts of the stretches before it, to write them in order (kept_write).
// U: candidates in flight per thread.  Between the two every wavefront's counts are in wtot [16][2] (above, equal).
template <int THREADS, int U, bool WRITE, typename KeyFn, typename SlotFn>
__device__ __forceinline__ void kept_walk(KeyFn key_at, SlotFn slot_at, int ncand, uint32_t T, uint32_t want, int32_t* out, uint32_t& gt_run,
                                          uint32_t& eq_run) {
    constexpr int WAVES = THREADS / kWave;
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int stretch = (((ncand + WAVES - 1) / WAVES) + kWave - 1) / kWave * kWave;
    const int w0 = min(wave * stretch, ncand), w1 = min(w0 + stretch, ncand);
    for (int i0 = w0; i0 < w1; i0 += U * kWave) {
        uint32_t kv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) kv[u] = key_at(min(i0 + u * kWave + lane, ncand - 1));
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * kWave + lane;
            const bool live = i < w1;
            const unsigned long long mg = __ballot(live && kv[u] > T), me = __ballot(live && kv[u] == T);
            if constexpr (WRITE) {
                const uint32_t g_below = __builtin_amdgcn_mbcnt_hi((uint32_t)(mg >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mg, 0));
                const uint32_t e_below = __builtin_amdgcn_mbcnt_hi((uint32_t)(me >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)me, 0));
                const uint32_t gb = gt_run + g_below, eb = eq_run + e_below;   // kept counts before slot i
                const int slot = slot_at(i, live);
                if (live && kv[u] > T) out[gb + min(eb, want)] = slot;
                else if (live && kv[u] == T && eb < want) out[gb + eb] = slot;
            }
            gt_run += (uint32_t)__popcll(mg);
            eq_run += (uint32_t)__popcll(me);
        }
    }
}
template <int THREADS, typename KeyFn>
__device__ __forceinline__ void kept_count(KeyFn key_at, bool in_lds, int ncand, uint32_t T, uint32_t* wtot) {
    uint32_t gt = 0, eq = 0;
    auto none = [](int, bool) { return 0; };
    if (in_lds) kept_walk<THREADS, 2, false>(key_at, none, ncand, T, 0u, nullptr, gt, eq);
    else kept_walk<THREADS, 16, false>(key_at, none, ncand, T, 0u, nullptr, gt, eq);
    if ((threadIdx.x & (kWave - 1)) == 0) {
        wtot[2 * (threadIdx.x / kWave)] = gt;
        wtot[2 * (threadIdx.x / kWave) + 1] = eq;
    }
    __syncthreads();
}
template <int THREADS, typename KeyFn, typename SlotFn>
__device__ __forceinline__ void kept_write(KeyFn key_at, SlotFn slot_at, bool in_lds, int ncand, uint32_t T, uint32_t want, const uint32_t* wtot, int32_t* out) {
    uint32_t gt_before = 0, eq_before = 0;
    for (int w = 0; w < (int)threadIdx.x / kWave; ++w) {
        gt_before += wtot[2 * w];
        eq_before += wtot[2 * w + 1];
    }
    if (in_lds) kept_walk<THREADS, 2, true>(key_at, slot_at, ncand, T, want, out, gt_before, eq_before);
    else kept_walk<THREADS, 16, true>(key_at, slot_at, ncand, T, want, out, gt_before, eq_before);
}

template <int THREADS, int MODE>
__global__ __launch_bounds__(THREADS) FK_TWO_PER_CU void select_keep_kernel(const float* __restrict__ scores,
                                                              const int32_t* __restrict__ len,
                                                              int cap, int budget, int recent, int lds_keys,
                                                              int32_t* __restrict__ keep, SelSplit sp) {
    const int row = blockIdx.x;
    const int n = min(len[row], cap);
    int32_t* out = keep + (size_t)row * budget;
    if (n <= budget) {  // nothing to prune: the identity over the whole row, which makes the compaction a no-op
        for (int j = threadIdx.x; j < budget; j += THREADS) out[j] = j;
        return;
    }
    const float* sc = scores + (size_t)row * cap;
    const int k = budget - recent;   // how many of the candidates stay (0 <= k < ncand; kSelMerge: 1 <= k <= ncand)
    int ncand = n - recent;          // candidates: slots [0, ncand), kSelMerge: a list of slots

    extern __shared__ __attribute__((aligned(16))) uint32_t s_sel_mem[];
    const SelLds s(s_sel_mem);
    uint32_t* s_slot = s.key + lds_keys;   // kSelMerge
    constexpr int WAVES = THREADS / kWave;
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    bool listed = MODE == kSelMerge;
    constexpr int kMaxChunks = 16;
    int base_of[kMaxChunks + 1];  // kSelMerge: where every chunk's survivors start in the merged list (registers)
    if constexpr (MODE == kSelMerge) {
        int tot = 0;
#pragma unroll
        for (int c = 0; c < kMaxChunks; ++c) {
            base_of[c] = tot;
            if (c < sp.nchunk) tot += sp.count[(size_t)row * sp.nchunk + c];
        }
        base_of[kMaxChunks] = tot;
        if (tot >= k) ncand = tot;
        else listed = false;   // the chunks' bound was too high: from the whole row
    }

    // The row's keys are read from global memory once and kept in LDS (rows beyond the LDS share of the launch are
    // re-read from global memory in every pass).
    const bool in_lds = MODE == kSelMerge ? listed : ncand <= lds_keys;  // kSelMerge: the host sized the launch so that the survivors are
    KeyRange kr;                                                         // gathered while the keys are written to LDS
    for (int i = threadIdx.x; i < kRangeWords + 4 * 256; i += THREADS) s.range[i] = 0;
    if (MODE == kSelMerge && listed) {
        // Slot, then score: two dependent reads, eight of either in flight per thread (one survivor at a time, this gather took 15 of 37 us at 32
        // rows of 15360 survivors); a wavefront stays with one chunk.
        const int group = WAVES / sp.nchunk, step = group * kWave;   // wavefronts of a chunk (2 <= nchunk <= 16)
        const int c = wave / group, at = (wave - c * group) * kWave + lane;
        if (c < sp.nchunk) {
            int base = 0, cnt = 0;
#pragma unroll
            for (int x = 0; x < kMaxChunks; ++x)
                if (x == c) {
                    base = base_of[x];
                    cnt = base_of[x + 1] - base;
                }
            const int32_t* list = sp.cand + ((size_t)row * sp.nchunk + c) * k;
            for (int i0 = at; i0 < cnt; i0 += 8 * step) {
                int slot[8];
                float v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) slot[u] = list[min(i0 + u * step, cnt - 1)];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = sc[slot[u]];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    if (i0 + u * step < cnt) {
                        const uint32_t key = score_key(v[u]);
                        s_slot[base + i0 + u * step] = (uint32_t)slot[u];
                        s.key[base + i0 + u * step] = key;
                        kr.add(key);
                    }
                }
            }
        }
    } else if (MODE == kSelWhole && in_lds) {
        keys_to_lds<THREADS>(sc, 0, ncand, s.key, kr);
    }
    RangePlan rp = {};
    if (in_lds) rp = kr.plan(s.wmm);
    else __syncthreads();
    auto key_at = [&](int i) { return in_lds ? s.key[i] : score_key(sc[i]); };
    uint32_t T = 0, want = 0;   // kept: keys above T and the first `want` equal to it (k == 0: no candidate)
    if (k > 0) {   // (rows read from global memory: 16 loads in flight per thread)
        auto key_of = [&](int i, bool& valid) { valid = true; return key_at(i); };
        if (in_lds) range_select<THREADS, 2>(key_of, ncand, (uint32_t)k, s.range, s.hist, s.wtot, rp, threadIdx.x, &T, &want);
        else msd_select<THREADS, 16>(key_of, ncand, (uint32_t)k, s.hist, 0u, ~0u, &T, &want);
        auto slot_at = [&](int i, bool live) { return MODE == kSelMerge && listed ? (live ? (int)s_slot[i] : 0) : i; };
        kept_count<THREADS>(key_at, in_lds, ncand, T, s.wtot);
        kept_write<THREADS>(key_at, slot_at, in_lds, ncand, T, want, s.wtot, out);
    }
    for (int j = threadIdx.x; j < recent; j += THREADS) out[k + j] = n - recent + j;
}

// One chunk of a row.  It need not select at all where a bound is known that at least k of the row's pairs reach: it passes on what
// reaches the bound.  The bound is a guess, the same for all chunks of a row: of a sample of the row, one key from each of 2048
// stretches, the r-th best, r so far above the k * 2048 / n expected among the k best (six standard deviations and eight) that fewer
// than k pairs reach it only where scores go by the sample's own places.  The merge counts, and selects from the whole row, by one
// workgroup and out of global memory, if it does: 32 rows of 131072 pairs then take 167 us (55 without a bound).
// A chunk with more than k pairs that reach the bound, but not more above it (equal scores), passes on the latter and the first of
// the others; one with more above it (most of the best in one chunk) selects.
// 32 rows of 131072 pairs, the best 1920, both launches, us, without a bound and with it: normal scores 45.0 and 23.2, all equal 30.5
// and 24.8, two values 42.0 and 27.5, the best in one chunk 47.3 and 39.5, rising scores 48.7 and 34.2.  64 rows, chunks of 32736: 49.5
// and 37.1, 30.5 and 30.2, 52.0 and 32.8, 51.3 and 52.5, 50.9 and 47.5.  What it loses is the sample's time where every chunk still walks all its
// pairs: 32 rows of 32768, all equal, 17.2 and 17.7.  (With a row's chunks on all XCDs, each of which then fetches the sample, the first
// launch takes 21 us, not 14.)
static constexpr int kSelSample = 2048;

template <int THREADS>
__global__ __launch_bounds__(THREADS) void select_chunk_kernel(const float* __restrict__ scores, const int32_t* __restrict__ len, int cap,
                                                               int budget, int recent, int lds_keys, SelSplit sp) {
    // blocks are dealt to the eight XCDs in turn: a row's chunks, which all read its sample, on one
    const int rows = gridDim.x / sp.nchunk, per = (int)blockIdx.x / 8;
    const bool deal = rows % 8 == 0;
    const int row = deal ? per / sp.nchunk * 8 + (int)blockIdx.x % 8 : (int)blockIdx.x / sp.nchunk;
    const int chunk = deal ? per % sp.nchunk : (int)blockIdx.x % sp.nchunk;
    const int n = min(len[row], cap);
    if (n <= budget) return;   // nothing to prune
    const int kmax = budget - recent, all = n - recent;   // all: the row's candidates
    const int first = chunk * sp.chunk_len;               // first slot of this chunk's
    const int ncand = max(chunk == sp.nchunk - 1 ? all - first : min(all - first, sp.chunk_len), 0);
    const float* sc = scores + (size_t)row * cap;
    int32_t* out = sp.cand + ((size_t)row * sp.nchunk + chunk) * kmax;
    int32_t* count = sp.count + (size_t)row * sp.nchunk + chunk;

    extern __shared__ __attribute__((aligned(16))) uint32_t s_sel_mem[];
    const SelLds s(s_sel_mem);
    constexpr int WAVES = THREADS / kWave;
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    // On its way while the bound is found: the chunk's first HELD * THREADS pairs.  Those of a chunk that has no more stay in registers, a share of
    // a wavefront's stretch in every thread.
    constexpr int HELD = 16;
    float held[HELD];
    const bool holds = ncand <= HELD * THREADS, in_lds = ncand <= lds_keys;
    if (holds && ncand > 0) {
#pragma unroll
        for (int u = 0; u < HELD; ++u) held[u] = sc[first + min((wave * HELD + u) * kWave + lane, ncand - 1)];
    } else if (in_lds && ncand > 0) {
#pragma unroll
        for (int u = 0; u < HELD; ++u) held[u] = sc[first + u * THREADS + threadIdx.x];
    }
    // A key that at least k pairs of the row reach in all likelihood (0: none was looked for).  Every survivor of a row with a
    // bound reaches it, so k survivors prove that the k best do.
    uint32_t bound = 0, left = 0;   // left: the bound's number among the sampled pairs equal to it, 1 where scores differ
    const float mean = (float)kSelSample * (float)kmax / (float)all;
    const int r = (int)(mean + 6.f * sqrtf(mean)) + 8;
    if (all >= 8 * kSelSample && 4 * r <= kSelSample && lds_keys >= kSelSample) {
        for (int i = threadIdx.x; i < kRangeWords + 4 * 256; i += THREADS) s.range[i] = 0;
        KeyRange kr;
        static_assert(kSelSample == 2 * THREADS, "two stretches a thread");
        const float len = (float)all / kSelSample;
        float v[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {   // a pair of every stretch, its place in it by a hash: no period of the scores fits it
            const int i = threadIdx.x + u * THREADS;
            const float frac = (float)((uint32_t)i * 2654435761u >> 8) * (1.f / 16777216.f);
            v[u] = sc[min((int)(((float)i + frac) * len), all - 1)];
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const uint32_t key = score_key(v[u]);
            s.key[threadIdx.x + u * THREADS] = key;
            kr.add(key);
        }
        const RangePlan rp = kr.plan(s.wmm);
        range_select<THREADS, 2>([&](int i, bool& valid) { valid = true; return s.key[i]; }, kSelSample, (uint32_t)r, s.range, s.hist, s.wtot, rp,
                                 threadIdx.x, &bound, &left);
        __syncthreads();   // the sample gives way to the chunk's keys
    }
    if (ncand == 0 || (ncand <= kmax && bound <= 1)) {  // the whole chunk survives
        if (threadIdx.x == 0) *count = ncand;
        for (int j = threadIdx.x; j < ncand; j += THREADS) out[j] = first + j;
        return;
    }
    if (bound > 1 && holds) {   // what reaches the bound, in order
        auto slot_of = [&](int u) { return (wave * HELD + u) * kWave + lane; };
        auto key_of = [&](int u) { return slot_of(u) < ncand ? score_key(held[u]) : 0u; };
        uint32_t over = 0;
#pragma unroll
        for (int u = 0; u < HELD; ++u) over += (uint32_t)__popcll(__ballot(key_of(u) >= bound));
        if (lane == 0) s.wtot[wave] = over;
        __syncthreads();
        uint32_t before = 0, total = 0;   // pairs that reach the bound
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            before += w < wave ? s.wtot[w] : 0u;
            total += s.wtot[w];
        }
        auto below = [](unsigned long long m) { return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0)); };
        if (total <= (uint32_t)kmax) {
            if (threadIdx.x == 0) *count = (int)total;
#pragma unroll
            for (int u = 0; u < HELD; ++u) {
                const bool in = key_of(u) >= bound;
                const unsigned long long m = __ballot(in);
                if (in) out[before + below(m)] = first + slot_of(u);
                before += (uint32_t)__popcll(m);
            }
            return;
        }
        if (left > 1) {
            over = 0;
#pragma unroll
            for (int u = 0; u < HELD; ++u) over += (uint32_t)__popcll(__ballot(key_of(u) > bound));
            if (lane == 0) s.wtot[WAVES + wave] = over;
            __syncthreads();
            uint32_t gt = 0, above = 0;   // pairs above the bound: before this wavefront's, all
#pragma unroll
            for (int w = 0; w < WAVES; ++w) {
                gt += w < wave ? s.wtot[WAVES + w] : 0u;
                above += s.wtot[WAVES + w];
            }
            if (above <= (uint32_t)kmax) {
                const uint32_t want = (uint32_t)kmax - above;
                uint32_t eq = before - gt;
                if (threadIdx.x == 0) *count = kmax;
#pragma unroll
                for (int u = 0; u < HELD; ++u) {
                    const uint32_t key = key_of(u);
                    const unsigned long long mg = __ballot(key > bound), me = __ballot(key == bound);
                    const uint32_t eb = eq + below(me);
                    if (key > bound || (key == bound && eb < want)) out[gt + below(mg) + min(eb, want)] = first + slot_of(u);
                    gt += (uint32_t)__popcll(mg);
                    eq += (uint32_t)__popcll(me);
                }
                return;
            }
        }
        __syncthreads();   // wtot has been read
    }
    sc += first;
    KeyRange kr;
    for (int i = threadIdx.x; i < kRangeWords + 4 * 256; i += THREADS) s.range[i] = 0;
    if (in_lds && !holds) {
#pragma unroll
        for (int u = 0; u < HELD; ++u) {
            const uint32_t key = score_key(held[u]);
            s.key[u * THREADS + threadIdx.x] = key;
            kr.add(key);
        }
    }
    if (in_lds) keys_to_lds<THREADS>(sc, holds ? 0 : HELD * THREADS, ncand, s.key, kr);
    auto key_at = [&](int i) { return in_lds ? s.key[i] : score_key(sc[i]); };
    auto slot_at = [&](int i, bool) { return first + i; };
    uint32_t T = 0, want = 0;
    const RangePlan rp = kr.plan(s.wmm);
    bool passed = false;
    int k = min(kmax, ncand);
    if (bound > 1 && !holds) {   // the same of longer chunks
        T = bound;
        kept_count<THREADS>(key_at, in_lds, ncand, T, s.wtot);
        uint32_t above = 0, equal = 0;
        for (int w = 0; w < WAVES; ++w) {
            above += s.wtot[2 * w];
            equal += s.wtot[2 * w + 1];
        }
        passed = above <= (uint32_t)kmax;
        if (passed) {
            want = min(equal, (uint32_t)kmax - above);
            k = (int)(above + want);
        } else {
            __syncthreads();   // wtot has been read
        }
    }
    if (threadIdx.x == 0) *count = k;
    if (!passed) {   // (with a bound: more than k pairs reach it, so the k best do)
        auto key_of = [&](int i, bool& valid) { valid = true; return key_at(i); };
        if (in_lds) range_select<THREADS, 2>(key_of, ncand, (uint32_t)k, s.range, s.hist, s.wtot, rp, threadIdx.x, &T, &want);
        else msd_select<THREADS, 16>(key_of, ncand, (uint32_t)k, s.hist, 0u, ~0u, &T, &want);
        kept_count<THREADS>(key_at, in_lds, ncand, T, s.wtot);
    }
    kept_write<THREADS>(key_at, slot_at, in_lds, ncand, T, want, s.wtot, out);
}

// ---------------------------------------------------------------------------------------
// Sampled selection: Top-K multinomial eviction (Section 3.1 Eq. 2, Appendix B.2).
// The n_cand lowest-scored non-recent pairs are candidates; of them E = len - budget are evicted,
// drawn without replacement with probabilities softmax(-score).  The draw is taken in its
// Gumbel-top-k form on noise supplied by the caller: the E candidates with the smallest fp32
// t = score - noise go.  Two radix selects per row: (1) the others - n_cand most important pairs
// are safe; a bitmap in LDS marks the candidates; (2) among the candidates the n_cand - E largest t
// stay (ties to the lower slot).  One ordered pass writes the kept slots ascending.
// ---------------------------------------------------------------------------------------
static constexpr int kSampledMaxLen = 131072;  // bitmap of candidates: 16 KB of LDS

__global__ __launch_bounds__(kSelThreads) void select_keep_sampled_kernel(const float* __restrict__ scores,
                                                                          const float* __restrict__ noise,
                                                                          const int32_t* __restrict__ len, int cap,
                                                                          int budget, int recent, int n_cand,
                                                                          int32_t* __restrict__ keep) {
    const int row = blockIdx.x;
    const int n = min(len[row], cap);  // cap <= kSampledMaxLen (checked on the host)
    int32_t* out = keep + (size_t)row * budget;
    if (n <= budget) {  // nothing to prune: the identity over the whole row
        for (int j = threadIdx.x; j < budget; j += kSelThreads) out[j] = j;
        return;
    }
    const float* sc = scores + (size_t)row * cap;
    const float* nz = noise + (size_t)row * cap;
    const int others = n - recent;  // slots [0, others) are not protected
    const int E = n - budget;       // pairs to evict (1 <= E <= others)
    const int K = min(max(n_cand, E), others);  // candidates
    const int k_safe = others - K;  // most important pairs, never evicted
    const int k2 = K - E;           // candidates that stay

    __shared__ uint32_t s_hist[256];
    __shared__ uint32_t s_sel[2];
    __shared__ unsigned long long s_part[kSelWaves];
    __shared__ unsigned long long s_cand[kSampledMaxLen / 64];  // bit i: slot i is a candidate
    const int lane = threadIdx.x & (kWave - 1);

    // (1) safe set
    uint32_t T1 = 0, want1 = 0;
    if (k_safe > 0)
        radix_threshold(others, (uint32_t)k_safe, [&](int i, bool& valid) { valid = true; return score_key(sc[i]); },
                        s_hist, s_sel, &T1, &want1);
    {
        uint32_t eq_base = 0;
        for (int base = 0; base < others; base += kSelThreads) {
            const int i = base + threadIdx.x;
            uint32_t gt = 0, eq = 0;
            if (i < others && k_safe > 0) {
                const uint32_t key = score_key(sc[i]);
                gt = key > T1;
                eq = key == T1;
            }
            unsigned long long tot;
            const unsigned long long incl = block_scan_incl((unsigned long long)eq, s_part, &tot);
            const uint32_t eq_before = eq_base + (uint32_t)incl - eq;
            const bool safe = gt || (eq && eq_before < want1);
            const unsigned long long bits = __ballot(i < others && !safe);
            if (lane == 0) s_cand[i >> 6] = bits;
            eq_base += (uint32_t)tot;
        }
    }
    __syncthreads();
    auto is_cand = [&](int i) { return (s_cand[i >> 6] >> (i & 63)) & 1ull; };

    // (2) which candidates stay: the k2 largest t = score - noise
    uint32_t T2 = 0, want2 = 0;
    if (k2 > 0)
        radix_threshold(others, (uint32_t)k2,
                        [&](int i, bool& valid) {
                            valid = is_cand(i);
                            return score_key(sc[i] - nz[i]);
                        },
                        s_hist, s_sel, &T2, &want2);

    // (3) ordered output: safe pairs, surviving candidates, protected tail
    unsigned long long run = 0;  // packed running counts: safe << 40 | gt2 << 20 | eq2
    for (int base = 0; base < others; base += kSelThreads) {
        const int i = base + threadIdx.x;
        unsigned long long safe = 0, gt = 0, eq = 0;
        if (i < others) {
            if (!is_cand(i)) {
                safe = 1;
            } else if (k2 > 0) {
                const uint32_t key = score_key(sc[i] - nz[i]);
                gt = key > T2;
                eq = key == T2;
            }
        }
        unsigned long long tot;
        const unsigned long long mine = (safe << 40) | (gt << 20) | eq;
        const unsigned long long before = run + block_scan_incl(mine, s_part, &tot) - mine;
        const uint32_t eq_before = (uint32_t)(before & 0xfffffull);
        if (safe || gt || (eq && eq_before < want2))
            out[(uint32_t)(before >> 40) + (uint32_t)((before >> 20) & 0xfffffull) + min(eq_before, want2)] = i;
        run += tot;
    }
    for (int j = threadIdx.x; j < recent; j += kSelThreads) out[budget - recent + j] = others + j;
}


// The same selection with the row in LDS (rows of up to kSampledLdsKeys candidates): both keys of every slot are formed
// once, the selections and the ordered passes are those of select_keep_kernel (range_select, one ordered
// walk per wavefront stretch), and the candidate marks take the place of the first key once the safe set is known.
// LDS (u32): histogram and list of range_select | histograms [4][256] of msd_select | wavefront totals [16][4] | key ranges
// [2][kRangePart] | key1 / candidate mark [lds_keys] | key2 [lds_keys]
static constexpr int kSampledLdsKeys = 18 * 1024;
static constexpr int kSampledLdsHead = kRangeWords + 4 * 256 + 64 + 2 * kRangePart;  // words before the keys
template <int THREADS>
__global__ __launch_bounds__(THREADS) FK_TWO_PER_CU void select_keep_sampled_lds_kernel(const float* __restrict__ scores,
                                                                          const float* __restrict__ noise,
                                                                          const int32_t* __restrict__ len, int cap,
                                                                          int budget, int recent, int n_cand, int lds_keys,
                                                                          int32_t* __restrict__ keep) {
    const int row = blockIdx.x;
    const int n = min(len[row], cap);
    int32_t* out = keep + (size_t)row * budget;
    if (n <= budget) {  // nothing to prune: the identity over the whole row
        for (int j = threadIdx.x; j < budget; j += THREADS) out[j] = j;
        return;
    }
    const float* sc = scores + (size_t)row * cap;
    const float* nz = noise + (size_t)row * cap;
    const int others = n - recent;  // slots [0, others) are not protected (others <= lds_keys: checked on the host)
    const int E = n - budget;       // pairs to evict (1 <= E <= others)
    const int K = min(max(n_cand, E), others);  // candidates
    const int k_safe = others - K;  // most important pairs, never evicted
    const int k2 = K - E;           // candidates that stay

    extern __shared__ __attribute__((aligned(16))) uint32_t s_sel_mem[];
    uint32_t* s_range = s_sel_mem;           // [kRangeWords]
    uint32_t* s_hist = s_range + kRangeWords;// [4][256]
    uint32_t* s_wtot = s_hist + 4 * 256;     // [16][4]
    uint32_t* s_wmm = s_wtot + 64;           // [2][kRangePart] range of the first keys, of the second keys
    uint32_t* s_k1 = s_wmm + 2 * kRangePart; // [lds_keys] key of the score; later 1 = candidate, 0 = safe
    uint32_t* s_k2 = s_k1 + lds_keys;        // [lds_keys] key of score - noise
    constexpr int WAVES = THREADS / kWave;
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;

    for (int i = threadIdx.x; i < kRangeWords; i += THREADS) s_range[i] = 0;
    KeyRange kr1;   // of the first keys
    for (int i0 = threadIdx.x; i0 < others; i0 += 8 * THREADS) {
        float v[8], z[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = min(i0 + u * THREADS, others - 1);
            v[u] = sc[i];
            z[u] = nz[i];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (i0 + u * THREADS < others) {
                const uint32_t key1 = score_key(v[u]), key2 = score_key(v[u] - z[u]);
                s_k1[i0 + u * THREADS] = key1;
                s_k2[i0 + u * THREADS] = key2;
                kr1.add(key1);
            }
    }
    RangePlan rp1 = {};
    if (k_safe > 0) rp1 = kr1.plan(s_wmm);
    else __syncthreads();

    // every wavefront owns one contiguous stretch of the row (the ordered passes walk it 64 slots at a time)
    const int stretch = (((others + WAVES - 1) / WAVES) + kWave - 1) / kWave * kWave;
    const int w0 = min(wave * stretch, others), w1 = min(w0 + stretch, others);

    // (1) safe set: the k_safe best by score; everything else becomes a candidate
    uint32_t T1 = 0, want1 = 0;
    if (k_safe > 0)
        range_select<THREADS, 2>([&](int i, bool& valid) { valid = true; return s_k1[i]; }, others, (uint32_t)k_safe, s_range, s_hist, s_wtot,
                                 rp1, threadIdx.x, &T1, &want1);
    KeyRange kr2;   // of the candidates' second keys
    {
        uint32_t eq = 0;  // slots equal to T1 in this stretch
        if (k_safe > 0)
            for (int i0 = w0; i0 < w1; i0 += kWave) {
                const int i = i0 + lane;
                eq += (uint32_t)__popcll(__ballot(i < w1 && s_k1[min(i, others - 1)] == T1));
            }
        __syncthreads();   // s_wtot and s_range have been read
        for (int i = threadIdx.x; i < kRangeWords; i += THREADS) s_range[i] = 0;
        if (lane == 0) s_wtot[4 * wave] = eq;
        __syncthreads();
        uint32_t eq_run = 0;
        for (int w = 0; w < wave; ++w) eq_run += s_wtot[4 * w];
        for (int i0 = w0; i0 < w1; i0 += kWave) {
            const int i = i0 + lane;
            const bool live = i < w1;
            const uint32_t key = s_k1[min(i, others - 1)];
            const bool is_eq = k_safe > 0 && live && key == T1;
            const unsigned long long me = __ballot(is_eq);
            const uint32_t e_below = __builtin_amdgcn_mbcnt_hi((uint32_t)(me >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)me, 0));
            const bool safe = k_safe > 0 && (key > T1 || (is_eq && eq_run + e_below < want1));
            if (live) s_k1[i] = safe ? 0u : 1u;
            if (live && !safe) kr2.add(s_k2[i]);
            eq_run += (uint32_t)__popcll(me);
        }
    }
    const RangePlan rp2 = kr2.plan(s_wmm + kRangePart, 4 * K >= others || K >= 512);

    // (2) which candidates stay: the k2 largest t = score - noise among them
    uint32_t T2 = 0, want2 = 0;
    if (k2 > 0)
        range_select<THREADS, 2>([&](int i, bool& valid) { valid = s_k1[i] != 0u; return s_k2[i]; }, others, (uint32_t)k2, s_range, s_hist, s_wtot,
                                 rp2, threadIdx.x, &T2, &want2);

    // (3) ordered output: safe pairs, surviving candidates (ties to the lower slot), protected tail
    auto walk = [&](auto write_, uint32_t& keep_run, uint32_t& eq_run) {
        constexpr bool WRITE = decltype(write_)::value;
        for (int i0 = w0; i0 < w1; i0 += kWave) {
            const int i = i0 + lane;
            const bool live = i < w1;
            const int ii = min(i, others - 1);
            const bool cand = s_k1[ii] != 0u;
            const uint32_t key = s_k2[ii];
            const bool sure = live && (!cand || (k2 > 0 && key > T2));   // kept whatever the ties do
            const bool tie = live && cand && k2 > 0 && key == T2;
            const unsigned long long ms = __ballot(sure), mt = __ballot(tie);
            if constexpr (WRITE) {
                const uint32_t s_below = __builtin_amdgcn_mbcnt_hi((uint32_t)(ms >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)ms, 0));
                const uint32_t t_below = __builtin_amdgcn_mbcnt_hi((uint32_t)(mt >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mt, 0));
                const uint32_t sb = keep_run + s_below, tb = eq_run + t_below;  // kept for sure / tied, before slot i
                if (sure) out[sb + min(tb, want2)] = i;
                else if (tie && tb < want2) out[sb + tb] = i;
            }
            keep_run += (uint32_t)__popcll(ms);
            eq_run += (uint32_t)__popcll(mt);
        }
    };
    uint32_t kept = 0, tied = 0;
    walk(std::false_type{}, kept, tied);
    if (lane == 0) {
        s_wtot[4 * wave + 1] = kept;
        s_wtot[4 * wave + 2] = tied;
    }
    __syncthreads();
    uint32_t kept_before = 0, tied_before = 0;
    for (int w = 0; w < wave; ++w) {
        kept_before += s_wtot[4 * w + 1];
        tied_before += s_wtot[4 * w + 2];
    }
    walk(std::true_type{}, kept_before, tied_before);
    for (int j = threadIdx.x; j < recent; j += THREADS) out[budget - recent + j] = others + j;
}

}  // namespace fk

using namespace fk;

static fk_status select_check(const fk_cache_desc* desc, const float* scores, const int32_t* len, int32_t max_len,
                              int32_t budget, int32_t protect_recent, const int32_t* keep_idx) {
    fk_status s = check_desc(desc);
    if (s != FK_OK) return s;
    if (!scores || !len || !keep_idx) return FK_ERR_INVALID_ARG;
    if (max_len <= 0 || max_len > desc->capacity) return FK_ERR_INVALID_ARG;
    if (budget <= 0 || budget > desc->capacity || protect_recent < 0 || protect_recent > budget)
        return FK_ERR_INVALID_ARG;
    return FK_OK;
}

static fk_status select_whole(const fk_cache_desc* desc, const float* scores, const int32_t* len, int32_t max_len,
                              int32_t budget, int32_t protect_recent, int32_t* keep_idx, hipStream_t st) {
    const int rows = desc->batch * desc->n_kv_heads;
    // LDS share for the keys: rows up to max_len keys (the hint) live in LDS; longer ones are read from global memory
    const int lds_keys = ((max_len < kSelMaxLdsKeys ? max_len : kSelMaxLdsKeys) + 3) & ~3;
    const size_t lds = sizeof(uint32_t) * (kSelLdsHead + (size_t)lds_keys);
    auto kern = select_keep_kernel<kSelThreads, kSelWhole>;
    static bool lds_ok[kMaxDevices] = {};
    if (!allow_dynamic_lds((const void*)kern, 160 * 1024, lds_ok)) return FK_ERR_LAUNCH;
    hipLaunchKernelGGL(kern, dim3(rows), dim3(kSelThreads), lds, st, scores, len, desc->capacity, budget, protect_recent,
                       lds_keys, keep_idx, SelSplit{});
    return launch_status();
}

extern "C" fk_status fk_select_keep(const fk_cache_desc* desc, const float* scores, const int32_t* pos,
                                    const int32_t* len, int32_t max_len, int32_t budget,
                                    int32_t protect_recent, int32_t* keep_idx, void* stream) {
    (void)pos;  // slot order stands for position order (cache precondition)
    const fk_status s = select_check(desc, scores, len, max_len, budget, protect_recent, keep_idx);
    if (s != FK_OK) return s;
    return select_whole(desc, scores, len, max_len, budget, protect_recent, keep_idx, (hipStream_t)stream);
}

// Rows are split when one workgroup per row would leave most CUs idle and the rows are long enough to pay for a
// second launch; the survivors of all chunks (keys and slots) must fit the merge workgroup's LDS.
struct SelPlan {
    int nchunk, chunk_len;
    size_t count_bytes, bytes;
};
static SelPlan select_plan(const fk_cache_desc* d, int max_len, int budget, int recent) {
    SelPlan p = {1, 0, 0, 0};
    const int rows = d->batch * d->n_kv_heads, kmax = budget - recent;
    if (rows > 64 || max_len < 16384 || kmax <= 0) return p;
    int nchunk = 256 / rows;                                   // one workgroup per CU (measured: 128 and 512 are slower)
    const int fit = (kSelMaxLdsKeys / 2) / kmax;               // survivors of all chunks: keys + slots in LDS
    if (nchunk > fit) nchunk = fit;
    if (nchunk > 16) nchunk = 16;  // kMaxChunks of the kernel
    if (nchunk < 2) return p;
    p.nchunk = nchunk;
    p.chunk_len = ((max_len - recent + nchunk - 1) / nchunk + 3) & ~3;
    p.count_bytes = ((size_t)rows * nchunk * sizeof(int32_t) + 255) & ~(size_t)255;
    p.bytes = p.count_bytes + (size_t)rows * nchunk * kmax * sizeof(int32_t);
    return p;
}

extern "C" size_t fk_select_keep_workspace(const fk_cache_desc* desc, int32_t max_len, int32_t budget, int32_t protect_recent) {
    if (check_desc(desc) != FK_OK || max_len <= 0 || max_len > desc->capacity || budget <= 0 || budget > desc->capacity ||
        protect_recent < 0 || protect_recent > budget)
        return 0;
    return select_plan(desc, max_len, budget, protect_recent).bytes;
}

extern "C" fk_status fk_select_keep_ws(const fk_cache_desc* desc, const float* scores, const int32_t* pos,
                                       const int32_t* len, int32_t max_len, int32_t budget, int32_t protect_recent,
                                       int32_t* keep_idx, void* workspace, size_t workspace_bytes, void* stream) {
    (void)pos;
    const fk_status s = select_check(desc, scores, len, max_len, budget, protect_recent, keep_idx);
    if (s != FK_OK) return s;
    hipStream_t st = (hipStream_t)stream;
    const SelPlan p = select_plan(desc, max_len, budget, protect_recent);
    if (p.nchunk < 2) return select_whole(desc, scores, len, max_len, budget, protect_recent, keep_idx, st);
    if (!workspace || workspace_bytes < p.bytes) return FK_ERR_WORKSPACE;
    const int rows = desc->batch * desc->n_kv_heads, kmax = budget - protect_recent;
    SelSplit sp = {p.nchunk, p.chunk_len, reinterpret_cast<int32_t*>(workspace),
                   reinterpret_cast<int32_t*>(static_cast<char*>(workspace) + p.count_bytes)};
    {
        auto kern = select_chunk_kernel<kSelThreads>;
        const int lds_keys = ((p.chunk_len < kSelMaxLdsKeys ? p.chunk_len : kSelMaxLdsKeys) + 3) & ~3;
        const size_t lds = sizeof(uint32_t) * (kSelLdsHead + (size_t)lds_keys);
        static bool lds_ok[kMaxDevices] = {};
        if (!allow_dynamic_lds((const void*)kern, 160 * 1024, lds_ok)) return FK_ERR_LAUNCH;
        hipLaunchKernelGGL(kern, dim3(rows * p.nchunk), dim3(kSelThreads), lds, st, scores, len, desc->capacity, budget,
                           protect_recent, lds_keys, sp);
        if (launch_status() != FK_OK) return FK_ERR_LAUNCH;
    }
    {
        auto kern = select_keep_kernel<kSelThreads, kSelMerge>;
        const int lds_keys = (p.nchunk * kmax + 3) & ~3;  // <= kSelMaxLdsKeys / 2 by the plan
        const size_t lds = sizeof(uint32_t) * (kSelLdsHead + 2 * (size_t)lds_keys);
        static bool lds_ok[kMaxDevices] = {};
        if (!allow_dynamic_lds((const void*)kern, 160 * 1024, lds_ok)) return FK_ERR_LAUNCH;
        hipLaunchKernelGGL(kern, dim3(rows), dim3(kSelThreads), lds, st, scores, len, desc->capacity, budget, protect_recent,
                           lds_keys, keep_idx, sp);
    }
    return launch_status();
}

extern "C" fk_status fk_select_keep_sampled(const fk_cache_desc* desc, const float* scores, const float* noise,
                                            const int32_t* pos, const int32_t* len, int32_t max_len, int32_t budget,
                                            int32_t protect_recent, int32_t n_candidates, int32_t* keep_idx,
                                            void* stream) {
    (void)pos;  // slot order stands for position order (cache precondition)
    fk_status s = check_desc(desc);
    if (s != FK_OK) return s;
    if (!scores || !noise || !len || !keep_idx) return FK_ERR_INVALID_ARG;
    if (max_len <= 0 || max_len > desc->capacity || n_candidates < 0) return FK_ERR_INVALID_ARG;
    if (budget <= 0 || budget > desc->capacity || protect_recent < 0 || protect_recent > budget)
        return FK_ERR_INVALID_ARG;
    if (desc->capacity > kSampledMaxLen) return FK_ERR_UNSUPPORTED;  // the candidate bitmap covers every slot a row can hold
    const int rows = desc->batch * desc->n_kv_heads;
    if (desc->capacity <= kSampledLdsKeys) {  // every row fits LDS with both of its keys
        const int lds_keys = (desc->capacity + 3) & ~3;
        const size_t lds = sizeof(uint32_t) * (kSampledLdsHead + 2 * (size_t)lds_keys);
        auto kern = select_keep_sampled_lds_kernel<kSelThreads>;
        static bool lds_ok[kMaxDevices] = {};
        if (!allow_dynamic_lds((const void*)kern, 160 * 1024, lds_ok)) return FK_ERR_LAUNCH;
        hipLaunchKernelGGL(kern, dim3(rows), dim3(kSelThreads), lds, (hipStream_t)stream, scores, noise, len, desc->capacity,
                           budget, protect_recent, n_candidates, lds_keys, keep_idx);
        return launch_status();
    }
    hipLaunchKernelGGL(select_keep_sampled_kernel, dim3(rows), dim3(kSelThreads), 0, (hipStream_t)stream, scores,
                       noise, len, desc->capacity, budget, protect_recent, n_candidates, keep_idx);
    return launch_status();
}
