// Device helpers of the selection kernels: order-preserving score keys, a workgroup scan and the
// selections over a workgroup, by range and most significant digit first (used by fk_select_keep,
// fk_select_keep_sampled and the Golden Eviction trace).
#ifndef FK_SELECT_COMMON_H
#define FK_SELECT_COMMON_H
#include "fk_common.h"

namespace fk {

static constexpr int kSelThreads = 1024;
static constexpr int kSelWaves = kSelThreads / kWave;

__device__ __forceinline__ uint32_t score_key(float s) {
    uint32_t u = __float_as_uint(s);
    if ((u & 0x7fffffffu) > 0x7f800000u) return 0u;   // NaN: below everything
    if (u == 0x80000000u) u = 0u;                     // -0 == +0
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Inclusive prefix sum over the 64 lanes of a wavefront with data-parallel-primitive moves (a handful of cycles per
// step; the same scan through LDS permutes costs about a hundred per step): shifts by 1, 2, 4, 8 inside each row of 16
// lanes, then the last lane of rows 0 / 2 is added to rows 1 / 3, then lane 31 to the upper half.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROW_MASK, 0xF, false);  // lanes without a source get 0
}
__device__ __forceinline__ uint32_t wave_scan_incl(uint32_t v) {
    v += dpp_u32<0x111, 0xF>(v);  // row_shr:1
    v += dpp_u32<0x112, 0xF>(v);  // row_shr:2
    v += dpp_u32<0x114, 0xF>(v);  // row_shr:4
    v += dpp_u32<0x118, 0xF>(v);  // row_shr:8
    v += dpp_u32<0x142, 0xA>(v);  // row_bcast:15 into rows 1 and 3
    v += dpp_u32<0x143, 0xC>(v);  // row_bcast:31 into rows 2 and 3
    return v;
}

// inclusive scan of a 64-bit value over the workgroup, in thread order; returns the inclusive
// value and the workgroup total.  s_part must hold kSelWaves entries.
__device__ __forceinline__ unsigned long long block_scan_incl(unsigned long long v,
                                                              unsigned long long* s_part,
                                                              unsigned long long* total) {
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const unsigned long long o = __shfl_up(v, off);
        if (lane >= off) v += o;
    }
    __syncthreads();  // s_part free for reuse
    if (lane == kWave - 1) s_part[wave] = v;
    __syncthreads();
    unsigned long long before = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kSelWaves; ++w) {
        const unsigned long long x = s_part[w];
        if (w < wave) before += x;
        tot += x;
    }
    *total = tot;
    return v + before;
}

// MSB-first radix select over slots [0, nslots): finds T and `want` such that the k best valid
// slots are those with key > T plus the first `want` (in slot order) with key == T.  k >= 1 and at
// least k valid slots.  key_of(i, valid) returns the slot's key and whether it takes part.
template <typename KeyFn>
__device__ __forceinline__ void radix_threshold(int nslots, uint32_t k, KeyFn key_of, uint32_t* s_hist,
                                                uint32_t* s_sel, uint32_t* T, uint32_t* want_out) {
    uint32_t prefix = 0, mask = 0, want = k;
    for (int shift = 24; shift >= 0; shift -= 8) {
        for (int i = threadIdx.x; i < 256; i += kSelThreads) s_hist[i] = 0;
        __syncthreads();
        for (int i = threadIdx.x; i < nslots; i += kSelThreads) {
            bool valid;
            const uint32_t key = key_of(i, valid);
            if (valid && (key & mask) == prefix) atomicAdd(&s_hist[(key >> shift) & 0xffu], 1u);
        }
        __syncthreads();
        if (threadIdx.x < kWave) {
            const int lane = threadIdx.x;
            uint32_t c[4], tot = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                c[j] = s_hist[255 - 4 * lane - j];
                tot += c[j];
            }
            uint32_t incl = tot;
#pragma unroll
            for (int off = 1; off < kWave; off <<= 1) {
                const uint32_t o = __shfl_up(incl, off);
                if (lane >= off) incl += o;
            }
            const uint32_t excl = incl - tot;
            if (excl < want && want <= incl) {
                uint32_t run = excl;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (run < want && want <= run + c[j]) {
                        s_sel[0] = 255 - 4 * lane - j;
                        s_sel[1] = run;
                    }
                    run += c[j];
                }
            }
        }
        __syncthreads();
        prefix |= s_sel[0] << shift;
        mask |= 0xffu << shift;
        want -= s_sel[1];
        __syncthreads();
    }
    *T = prefix;
    *want_out = want;
}

// minimum and maximum over the wavefront (results in every lane)
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp_keep_u32(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, ROW_MASK, 0xF, false);  // lanes without a source keep theirs
}
__device__ __forceinline__ void wave_min_max(uint32_t& lo, uint32_t& hi) {
#define FK_MIN_MAX_STEP(CTRL, MASK)                 \
    lo = min(lo, dpp_keep_u32<CTRL, MASK>(lo));     \
    hi = max(hi, dpp_keep_u32<CTRL, MASK>(hi));
    FK_MIN_MAX_STEP(0x111, 0xF)  // row_shr:1
    FK_MIN_MAX_STEP(0x112, 0xF)  // row_shr:2
    FK_MIN_MAX_STEP(0x114, 0xF)  // row_shr:4
    FK_MIN_MAX_STEP(0x118, 0xF)  // row_shr:8
    FK_MIN_MAX_STEP(0x142, 0xA)  // row_bcast:15 into rows 1 and 3
    FK_MIN_MAX_STEP(0x143, 0xC)  // row_bcast:31 into rows 2 and 3
#undef FK_MIN_MAX_STEP
    lo = (uint32_t)__builtin_amdgcn_readlane((int)lo, kWave - 1);
    hi = (uint32_t)__builtin_amdgcn_readlane((int)hi, kWave - 1);
}

// Most-significant-digit-first passes (8-bit digits, at most four) over the slots [0, nslots) whose key_of(i, valid)
// reports valid: finds the key T of the k-th best valid slot and the number `want` of valid slots equal to T that
// still belong to the k best (1 <= k <= number of valid slots).  hist: [4][256] in LDS, zero on entry, dirty on return
// (one histogram per pass, one barrier per pass).  U keys per thread are fetched before the first of them is used.
// Every thread of the workgroup must call this, with the same arguments.
//
// base, diff: what the caller knows about the keys' spread: every valid key agrees with `base` in every bit that is
// clear in `diff` (base = any valid key, diff = OR over the valid keys of key ^ base; base 0, diff ~0 if unknown).  The
// first digit starts at the highest bit set in diff: scores of one row share their sign and most of their exponent,
// so that the 256 bins of the first pass divide the range the keys really cover, not the whole float range.
//
// Early finish: once the digit's bin holds at most 64 slots, no further histogram is built.  One sweep appends the
// remaining bits of those slots to a list (in the last pass's histogram, which is then never needed), and every
// wavefront ranks the list by itself, one entry per lane: entries are made distinct by their list index, the entry of
// rank want - 1 carries the threshold.  The list's order depends on the order of the atomics; the threshold and the
// count above it do not.  With the spread known, 2000 distinct scores mostly take one histogram and the list; rows of
// equal scores take none (diff 0) or, if a few differ, up to four.
template <int THREADS, int U, typename KeyFn>
__device__ __forceinline__ void msd_select(KeyFn key_of, int nslots, uint32_t k, uint32_t* hist4, uint32_t base,
                                           uint32_t diff, uint32_t* T_out, uint32_t* want_out) {
    const int lane = threadIdx.x & (kWave - 1);
    if (diff == 0) {   // every valid key is `base`
        *T_out = base;
        *want_out = k;
        return;
    }
    int open = 32 - __clz(diff);   // bits [0, open) are still undecided
    uint32_t mask = open >= 32 ? 0u : ~0u << open, prefix = base & mask, want = k;
    for (int pass = 0; pass < 4; ++pass) {   // open <= 32 - 8 * pass
        const int shift = max(open - 8, 0);
        const uint32_t dmask = (1u << (open - shift)) - 1u;   // eight bits; fewer in a last, short digit
        uint32_t* hist = hist4 + pass * 256;
        for (int i0 = 0; i0 < nslots; i0 += U * THREADS) {   // uniform trip count: the wavefront votes below
            uint32_t kv[U];
            bool ok[U];
#pragma unroll
            for (int u = 0; u < U; ++u) kv[u] = key_of(min(i0 + u * THREADS + (int)threadIdx.x, nslots - 1), ok[u]);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const bool todo = ok[u] && i0 + u * THREADS + (int)threadIdx.x < nslots && (kv[u] & mask) == prefix;
                const uint32_t dg = (kv[u] >> shift) & dmask;
                // Scores of one row share their sign and most of their exponent: in the first pass a wavefront's keys
                // usually all carry one digit, and atomics of many lanes on one LDS word are served one per cycle (2000
                // keys on one word: 2000 cycles).  One vote: if every pending lane has the first one's digit, one lane
                // adds the count; otherwise one atomic per lane.  (Measured and dropped: counting the first lane's digit
                // by vote also when the wavefront is not unanimous, and peeling several digits off it one vote each;
                // the votes' scalar round trips cost what the shorter queues save, or more.)
                const unsigned long long act = __ballot(todo);
                if (act != 0) {
                    const int first = __ffsll((long long)act) - 1;
                    const uint32_t lead = __builtin_amdgcn_readlane(dg, first);
                    if (__ballot(todo && dg == lead) == act) {
                        if (lane == first) atomicAdd(&hist[lead], (uint32_t)__popcll(act));
                    } else if (todo) {
                        atomicAdd(&hist[dg], 1u);
                    }
                }
            }
        }
        __syncthreads();
        // Every wavefront finds the digit for itself (no broadcast through LDS, one barrier per pass): lane l owns
        // digits 255-4l .. 252-4l (descending); the digit where the running count from the top reaches `want`.
        const uint4 h4 = *reinterpret_cast<const uint4*>(hist + 252 - 4 * lane);
        const uint32_t c[4] = {h4.w, h4.z, h4.y, h4.x};
        const uint32_t tot = c[0] + c[1] + c[2] + c[3];
        const uint32_t incl = wave_scan_incl(tot), excl = incl - tot;
        uint32_t digit = 0, above = 0, inbin = 0;
        const bool mine = excl < want && want <= incl;  // exactly one lane
        if (mine) {
            uint32_t run = excl;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (run < want && want <= run + c[j]) {
                    digit = 255 - 4 * lane - j;
                    above = run;
                    inbin = c[j];
                }
                run += c[j];
            }
        }
        const int src = __ffsll((long long)__ballot(mine)) - 1;
        digit = __builtin_amdgcn_readlane(digit, src);
        above = __builtin_amdgcn_readlane(above, src);
        inbin = __builtin_amdgcn_readlane(inbin, src);
        prefix |= digit << shift;
        mask |= dmask << shift;
        want -= above;   // 1 <= want <= inbin
        open = shift;
        if (open == 0) break;   // every bit is decided (after the fourth pass at the latest)
        if (inbin <= (uint32_t)kWave) {   // the same for every wavefront: all read the same histogram; pass <= 2 here
            // the last pass's histogram, still zero: [0] entries so far, [4 + i] entry i as a tag: the open bits of the
            // key above six bits that tell equal keys apart, plus one (0 = no entry)
            uint32_t* fill = hist4 + 3 * 256;
            for (int i0 = 0; i0 < nslots; i0 += U * THREADS) {
                uint32_t kv[U];
                bool ok[U];
#pragma unroll
                for (int u = 0; u < U; ++u) kv[u] = key_of(min(i0 + u * THREADS + (int)threadIdx.x, nslots - 1), ok[u]);
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (ok[u] && i0 + u * THREADS + (int)threadIdx.x < nslots && (kv[u] & mask) == prefix) {
                        const uint32_t idx = atomicAdd(fill, 1u);
                        fill[4 + idx] = (((kv[u] & ~mask) << 6) | (63u - idx)) + 1u;   // at most 24 open bits
                    }
                }
            }
            __syncthreads();
            const bool have = (uint32_t)lane < inbin;
            const uint32_t tag = fill[4 + lane];   // 0 beyond the list
            const uint32_t low = (tag - 1u) >> 6;
            // rank = entries with a larger tag; the list is read 16 entries at a time, every lane the same words
            uint32_t rank = 0;
            for (uint32_t c = 0; c < inbin; c += 16) {
                uint4 e[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) e[q] = *reinterpret_cast<const uint4*>(fill + 4 + c + 4 * q);
#pragma unroll
                for (int q = 0; q < 4; ++q) rank += (e[q].x > tag) + (e[q].y > tag) + (e[q].z > tag) + (e[q].w > tag);
            }
            const int at = __ffsll((long long)__ballot(have && rank == want - 1)) - 1;   // exactly one lane
            const uint32_t tlow = __builtin_amdgcn_readlane(low, at);
            *T_out = prefix | tlow;
            *want_out = want - (uint32_t)__popcll(__ballot(have && low > tlow));
            return;
        }
    }
    *T_out = prefix;
    *want_out = want;
}

// ---- selection by range ------------------------------------------------------------------------------------------
// The k-th best of the keys by ONE histogram over their range: kRangeBins equal bins from the smallest to the largest key
// (keys of one sign: of the bit pattern, that is of the logarithm; of both signs: of the value, since most bit patterns between
// them are numbers near 0 that no score takes), then the list of the keys in the cut's bin, ranked as in msd_select.  Digits of
// the bit pattern put the scores of a row, whose exponents span a few octaves, into a handful of bins: every LDS atomic of a
// wavefront then waits for the others on its word (15360 keys between 1.2 and 4.5: 12 us in the first pass, 2984 keys left),
// and a second pass follows.  More than 64 keys in the bin (256 of long rows): msd_select on them, which ends at once where
// they are equal (ties).  Values that a few bins would hold (outliers, heavy tails: some wavefronts found a range far smaller
// than that of all) or that bins cannot divide (infinities, NaN among negative and positive ones): msd_select from the start.
// Measured, us, 128 rows of 2176 and 32 of 30000 keys: normal 6.3 and 28 (by digits 6.9 and 36), quotients of normal numbers 7.3
// and 34 (by digits 6.8 and 33: the range is what they pay for; by range 10.6).
static constexpr int kRangeBins = 1024;
static constexpr int kRangeList = 256, kRangeListRows = 8192;   // long rows list up to this many
// LDS words: histogram | list: count, threshold, how many of it, unused, kRangeList keys.  Zero on entry; dirty on return.
static constexpr int kRangeWords = kRangeBins + 4 + kRangeList;

__device__ __forceinline__ float key_score(uint32_t key) { return __uint_as_float((key & 0x80000000u) ? key ^ 0x80000000u : ~key); }

// Smallest and largest of the valid keys, gathered while they are formed: add() every key, then every thread calls plan().
// One wavefront puts the sixteen wavefronts' ranges together and works out how to divide them, and the others wait: sixteen
// doing it each for itself cost four turns on every SIMD.
enum { kRangeDigits = -1, kRangeValue = -2, kRangeEqual = -3 };   // or, by bit pattern, the shift
struct RangePlan {
    uint32_t kmin, kmax;
    float scale;
    int how;
};
// crowded: some wavefronts found a far smaller range than all of them together
__device__ __forceinline__ RangePlan range_plan(uint32_t kmin, uint32_t kmax, bool crowded = false) {
    const float scale = 1023.9f / (key_score(kmax) - key_score(kmin));
    int how = max(22 - __clz((int)(kmax - kmin)), 0);   // (kmax - kmin) >> how < 1024
    // by value: a finite, positive scale: kmin and kmax are numbers and their difference is a normal one
    if ((kmin ^ kmax) >> 31) how = !crowded && scale > 0.f && scale < 3.4e38f ? kRangeValue : kRangeDigits;
    if (kmin == kmax) how = kRangeEqual;
    return {kmin, kmax, scale, how};
}
static constexpr int kRangePart = 2 * kSelWaves + 4;   // LDS words, sixteen-byte aligned
struct KeyRange {
    uint32_t lo = 0xffffffffu, hi = 0;
    __device__ __forceinline__ void add(uint32_t key) {
        lo = min(lo, key);
        hi = max(hi, key);
    }
    // two barriers; dense: some sixteen keys or more to a wavefront that has any (fewer have a narrow range by chance)
    __device__ __forceinline__ RangePlan plan(uint32_t* part, bool dense = true) {
        static_assert(kSelWaves == 16, "one lane of a row per wavefront");
        const int lane = threadIdx.x & (kWave - 1);
        wave_min_max(lo, hi);
        if (lane == 0) *reinterpret_cast<uint2*>(part + 2 * (threadIdx.x / kWave)) = make_uint2(lo, hi);
        __syncthreads();
        if (threadIdx.x < kWave) {
            const uint2 r = *reinterpret_cast<const uint2*>(part + 2 * (lane & 15));
            uint32_t mn = r.x, mx = r.y;
#define FK_RANGE_STEP(CTRL)                          \
    mn = min(mn, dpp_keep_u32<CTRL, 0xF>(mn));       \
    mx = max(mx, dpp_keep_u32<CTRL, 0xF>(mx));
            FK_RANGE_STEP(DPP_QUAD_XOR1)
            FK_RANGE_STEP(DPP_QUAD_XOR2)
            FK_RANGE_STEP(DPP_ROW_HALF_MIRROR)
            FK_RANGE_STEP(DPP_ROW_MIRROR)
#undef FK_RANGE_STEP
            // Two of them, because one may have few keys; one where few have any.  (One without has NaN here.)
            const bool narrow = lane < kSelWaves && 5.f * (key_score(r.y) - key_score(r.x)) < key_score(mx) - key_score(mn);
            const int few = __popcll(__ballot(lane < kSelWaves && r.x <= r.y)) < 5;
            const RangePlan rp = range_plan(mn, mx, dense && __popcll(__ballot(narrow)) + few >= 2);
            if (lane == 0) *reinterpret_cast<uint4*>(part + 2 * kSelWaves) = make_uint4(mn, mx, __float_as_uint(rp.scale), (uint32_t)rp.how);
        }
        __syncthreads();
        const uint4 p = *reinterpret_cast<const uint4*>(part + 2 * kSelWaves);
        return {p.x, p.y, __uint_as_float(p.z), (int)p.w};
    }
};

// rp: of the valid keys; tid: threadIdx.x.  LOOP: for a caller with a loop round this, where code costs registers: no long list.
// hist4: [4][256] words for msd_select, contents undefined; part: 2 * THREADS / 64 words.
// The other conditions are those of msd_select (every thread calls, 1 <= k <= number of valid slots).
template <int THREADS, int U, bool LOOP = false, typename KeyFn>
__device__ __forceinline__ void range_select(KeyFn key_of, int nslots, uint32_t k, uint32_t* range, uint32_t* hist4, uint32_t* part,
                                             const RangePlan rp, int tid, uint32_t* T_out, uint32_t* want_out) {
    const int lane = tid & (kWave - 1);
    const int how = __builtin_amdgcn_readfirstlane(rp.how);
    if (how == kRangeEqual) {
        *T_out = rp.kmin;
        *want_out = k;
        return;
    }
    const float lo = key_score(rp.kmin);
    auto bin_of = [&](uint32_t key) -> uint32_t {
        if (how == kRangeValue) return (uint32_t)min(max((int)((key_score(key) - lo) * rp.scale), 0), kRangeBins - 1);   // monotone: so is every step
        return (key - rp.kmin) >> how;
    };
    uint32_t bin = 0, want = k, inbin = 0xffffffffu;
    if (how != kRangeDigits) {
        for (int i0 = 0; i0 < nslots; i0 += U * THREADS) {   // uniform trip count: the wavefront votes below
            uint32_t kv[U];
            bool ok[U];
#pragma unroll
            for (int u = 0; u < U; ++u) kv[u] = key_of(min(i0 + u * THREADS + tid, nslots - 1), ok[u]);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const bool todo = ok[u] && i0 + u * THREADS + tid < nslots;
                const uint32_t dg = bin_of(kv[u]);
                const unsigned long long act = __ballot(todo);
                if (act != 0) {   // one vote: a wavefront of equal bins adds its count once
                    const int first = __ffsll((long long)act) - 1;
                    const uint32_t lead = __builtin_amdgcn_readlane(dg, first);
                    if (__ballot(todo && dg == lead) == act) {
                        if (lane == first) atomicAdd(&range[lead], (uint32_t)__popcll(act));
                    } else if (todo) {
                        atomicAdd(&range[dg], 1u);
                    }
                }
            }
        }
        __syncthreads();
        // One wavefront finds the bin, as in KeyRange::plan: four blocks of 256 bins from the top, lane l owns the bins
        // 255 - 4 l .. 252 - 4 l of each.
        if (tid < kWave) {
            uint4 h[4];
            uint32_t tot[4], incl[4];
#pragma unroll
            for (int b = 0; b < 4; ++b) h[b] = *reinterpret_cast<const uint4*>(range + 256 * (3 - b) + 252 - 4 * lane);
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                tot[b] = h[b].x + h[b].y + h[b].z + h[b].w;
                incl[b] = wave_scan_incl(tot[b]);
            }
            uint32_t before = 0;   // keys in the blocks above
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const uint32_t excl = before + incl[b] - tot[b];
                if (excl < k && k <= excl + tot[b]) {   // one lane, one block
                    const uint32_t c[4] = {h[b].w, h[b].z, h[b].y, h[b].x};
                    uint32_t run = excl;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        if (run < k && k <= run + c[j]) {
                            part[0] = 256 * (3 - b) + 255 - 4 * lane - j;
                            part[1] = k - run;
                            part[2] = c[j];
                        }
                        run += c[j];
                    }
                }
                before += __builtin_amdgcn_readlane(incl[b], kWave - 1);
            }
        }
        __syncthreads();
        bin = part[0];
        want = part[1];
        inbin = part[2];   // 1 <= want <= inbin
        if (inbin <= (uint32_t)kWave) {
            uint32_t* list = range + kRangeBins;
            for (int i0 = 0; i0 < nslots; i0 += U * THREADS) {
                uint32_t kv[U];
                bool ok[U];
#pragma unroll
                for (int u = 0; u < U; ++u) kv[u] = key_of(min(i0 + u * THREADS + tid, nslots - 1), ok[u]);
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (ok[u] && i0 + u * THREADS + tid < nslots && bin_of(kv[u]) == bin) list[4 + atomicAdd(list, 1u)] = kv[u];
            }
            __syncthreads();
            // One entry per lane of one wavefront; rank = entries before it under (key descending, place in the list), which depends on
            // the list's order only among equal keys; an unused place holds 0 and is after every entry it is compared with.
            if (tid < kWave) {
                const bool have = (uint32_t)lane < inbin;
                const uint32_t key = list[4 + lane];
                uint32_t rank = 0;
                for (uint32_t q = 0; q < inbin; q += 4) {
                    const uint4 e = *reinterpret_cast<const uint4*>(list + 4 + q);
                    rank += (e.x > key || (e.x == key && q < (uint32_t)lane)) + (e.y > key || (e.y == key && q + 1 < (uint32_t)lane)) +
                            (e.z > key || (e.z == key && q + 2 < (uint32_t)lane)) + (e.w > key || (e.w == key && q + 3 < (uint32_t)lane));
                }
                const int at = __ffsll((long long)__ballot(have && rank == want - 1)) - 1;   // exactly one lane
                const uint32_t T = __builtin_amdgcn_readlane(key, at);
                const uint32_t over = (uint32_t)__popcll(__ballot(have && key > T));
                if (lane == 0) {
                    list[1] = T;
                    list[2] = want - over;
                }
            }
            __syncthreads();
            *T_out = list[1];
            *want_out = list[2];
            return;
        }
        if (!LOOP && inbin <= (uint32_t)kRangeList && nslots >= kRangeListRows) {   // the same with one entry per lane of up to four wavefronts
            uint32_t* list = range + kRangeBins;
            for (int i = tid; i < nslots; i += THREADS) {
                bool ok;
                const uint32_t key = key_of(i, ok);
                if (ok && bin_of(key) == bin) list[4 + atomicAdd(list, 1u)] = key;
            }
            __syncthreads();
            const uint4 quad = *reinterpret_cast<const uint4*>(list + 4 + 4 * lane);   // four entries a lane
            const uint32_t one = list[4], at = 4 * (uint32_t)lane;
            if (__all((at >= inbin || quad.x == one) && (at + 1 >= inbin || quad.y == one) && (at + 2 >= inbin || quad.z == one) &&
                      (at + 3 >= inbin || quad.w == one))) {   // equal scores: nothing to rank (8320 keys, 200 of them 16.0 -> 11.6 us)
                *T_out = one;
                *want_out = want;
                return;
            }
            if ((uint32_t)tid < inbin) {
                const uint32_t key = list[4 + tid];
                uint32_t above = 0, ties = 0;   // entries with a larger key; equal ones at earlier places
#pragma unroll 4
                for (uint32_t q = 0; q < inbin; q += 4) {
                    const uint4 e = *reinterpret_cast<const uint4*>(list + 4 + q);
                    above += (e.x > key) + (e.y > key) + (e.z > key) + (e.w > key);
                    ties += (e.x == key && q < (uint32_t)tid) + (e.y == key && q + 1 < (uint32_t)tid) + (e.z == key && q + 2 < (uint32_t)tid) +
                            (e.w == key && q + 3 < (uint32_t)tid);
                }
                if (above + ties == want - 1) {   // exactly one thread
                    list[1] = key;
                    list[2] = want - above;
                }
            }
            __syncthreads();
            *T_out = list[1];
            *want_out = list[2];
            return;
        }
    }
    // digit by digit: all keys, or those of the bin, from the highest bit in which any two differ (one msd_select for both: a copy is 6 KB
    // of instructions)
    uint32_t mn = rp.kmin, mx = rp.kmax;
    auto left = [&](int i, bool& valid) {
        const uint32_t key = key_of(i, valid);
        valid = valid && (how == kRangeDigits || bin_of(key) == bin);
        return key;
    };
    __syncthreads();   // part has been read
    for (int i = tid; i < 4 * 256; i += THREADS) hist4[i] = 0;
    if (how != kRangeDigits) {
        mn = 0xffffffffu;
        mx = 0;
        for (int i = tid; i < nslots; i += THREADS) {
            bool valid;
            const uint32_t key = left(i, valid);
            if (valid) {
                mn = min(mn, key);
                mx = max(mx, key);
            }
        }
        wave_min_max(mn, mx);
        if (lane == 0) {
            part[2 * (tid / kWave)] = mn;
            part[2 * (tid / kWave) + 1] = mx;
        }
        __syncthreads();
        for (int w = 0; w < THREADS / kWave; ++w) {
            mn = min(mn, part[2 * w]);
            mx = max(mx, part[2 * w + 1]);
        }
    }
    __syncthreads();   // the histograms are clear; part is the caller's again
    msd_select<THREADS, U>(left, nslots, want, hist4, mn, mn ^ mx, T_out, want_out);
}

}  // namespace fk
#endif
