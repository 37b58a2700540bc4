// fk_append, fk_compact and fk_compact_feat: the calls that rewrite the cache (and the attention-feature state).
#include "fk_common.h"

namespace fk {

// ---------------------------------------------------------------------------------------
// append (Section 3.1: each generated token adds one pair to every KV-head row)
// one workgroup per row; 16-byte chunks of the new K and V rows
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(64) void append_kernel(uint4* __restrict__ K, uint4* __restrict__ V,
                                                    int32_t* __restrict__ pos, int32_t* __restrict__ len,
                                                    const uint4* __restrict__ k_new,
                                                    const uint4* __restrict__ v_new,
                                                    const int32_t* __restrict__ pos_new, int n_kv,
                                                    int cap, int chunks /* 16-byte chunks per row */) {
    const int row = blockIdx.x;
    const int n = len[row];
    if (n < 0 || n >= cap) return;
    const size_t dst = ((size_t)row * cap + n) * chunks;
    for (int c = threadIdx.x; c < chunks; c += blockDim.x) {
        K[dst + c] = k_new[(size_t)row * chunks + c];
        V[dst + c] = v_new[(size_t)row * chunks + c];
    }
    if (threadIdx.x == 0) {
        pos[(size_t)row * cap + n] = pos_new[row / n_kv];
        len[row] = n + 1;  // only this workgroup reads or writes len[row]
    }
}

static constexpr int kCompactThreads = 1024;

// ---------------------------------------------------------------------------------------
// close a chunk of the attention features (Appendix B.1) and compact them with the cache
//
// feat [rows][6][cap][GP]: planes w8, w16, w32, wL (sums of this chunk's attention weights over
// the last 8 / 16 / 32 queries and over the whole chunk), cum, dec (sums carried over earlier
// chunks, plain and decayed by 0.9 per chunk).  At the end of a chunk cum += wL, dec = 0.9 dec
// + wL and the four chunk planes restart from zero; rows over budget move slot keep[j] to slot
// j in the same pass (ascending tiles, all sources of a tile read before it is written: the
// argument of compact_kernel).  One workgroup per row; a thread owns 4 heads of a slot.  The workgroups of compact_kernel's launch that run
// it come first in its grid: 128 rows of 2176 pairs, four heads, 8.6 us in a launch of its own before the compaction's 42; in one launch
// 46.4. (Two workgroups a CU, with four registers spilled, take 53: more rows in flight make the compaction slower, 42 -> 48.)
// ---------------------------------------------------------------------------------------

template <int Q4 /* float4 units per slot */>
__device__ __forceinline__ void feat_roll(float4* __restrict__ feat, int row, int n /* length before the compaction */,
                                          const int32_t* __restrict__ keep, int cap, int budget) {
    if (n <= 0) return;
    const size_t pl4 = (size_t)cap * Q4;
    float4* f = feat + (size_t)row * 6 * pl4;
    float4 *wl = f + 3 * pl4, *cum = f + 4 * pl4, *dec = f + 5 * pl4;
    const bool gather = n > budget;
    const int32_t* kp = keep + (size_t)row * budget;
    const int n_out = gather ? budget : n;
    constexpr int tile = kCompactThreads / Q4;  // slots per pass
    const int sl = threadIdx.x / Q4, q = threadIdx.x % Q4;
    for (int base = 0; base < n_out; base += tile) {
        const int j = base + sl;
        int src = -1;
        if (j < n_out) src = gather ? kp[j] : j;
        const bool ok = src >= 0 && src < n;
        float4 c = make_float4(0.f, 0.f, 0.f, 0.f), d = c, w = c;
        if (ok) {
            c = cum[(size_t)src * Q4 + q];
            d = dec[(size_t)src * Q4 + q];
            w = wl[(size_t)src * Q4 + q];
        }
        __syncthreads();
        if (ok) {
            cum[(size_t)j * Q4 + q] = make_float4(c.x + w.x, c.y + w.y, c.z + w.z, c.w + w.w);
            dec[(size_t)j * Q4 + q] = make_float4(fmaf(kFeatDecay, d.x, w.x), fmaf(kFeatDecay, d.y, w.y),
                                                  fmaf(kFeatDecay, d.z, w.z), fmaf(kFeatDecay, d.w, w.w));
        }
    }
    __syncthreads();  // every wL source has been read
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int t = threadIdx.x; t < n * Q4; t += kCompactThreads) {
        f[t] = zero;
        f[pl4 + t] = zero;
        f[2 * pl4 + t] = zero;
        f[3 * pl4 + t] = zero;
    }
}

// ---------------------------------------------------------------------------------------
// compact (stable in-place gather)
//
// keep[] is ascending with keep[j] >= j.  A workgroup owns one 128-byte column slice of one
// tensor of one row (bytes of different slices never alias, so slices are independent; 128
// bytes = two whole 64-byte memory requests per slot, narrower slices fetch and write partial
// lines and cost 1.5x the time) and walks the destination slots in ascending tiles of 512 (256)
// slots: all sources of a tile are loaded into registers, a barrier, then the tile is stored.  A store of tile t lands in slots
// [tT, (t+1)T); a source of any later tile is >= (t+1)T, and every source of tile t or of an
// earlier tile has already been read, so no live source is overwritten.  What does not move is neither
// read nor written, but for slot 0 in its place where there are few workgroups.
// grid.x = row, grid.y = tensor * slices + slice (K slices, then V slices), last y = pos; Q4 > 0: the attention features before them
// ---------------------------------------------------------------------------------------
static constexpr int kSliceChunks = 8;  // 16-byte chunks per column slice
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

// The workgroup that moves the positions (Q4 > 0: the features, which go by the length) also sets len[row] = min(len[row], budget) (no
// second launch).  No other workgroup may then read len[row]: what moves is decided by keep alone (rows at or under budget carry the
// identity, entries with keep[j] == j or outside [0, cap) move nothing).
enum CompactWalk { WALK_ONE, WALK_TURNS, WALK_MOVED };
template <int Q4 /* float4 units of a feature plane per slot; 0: no features */, int U /* 16-byte loads of a tile per thread */, int WALK,
          bool ALONE /* one workgroup to a CU */>
__global__ __launch_bounds__(kCompactThreads) __attribute__((amdgpu_waves_per_eu(4, (ALONE ? 4 : 8)))) void compact_kernel(uint4* __restrict__ K, uint4* __restrict__ V,
                                                                  int32_t* __restrict__ pos, float4* __restrict__ feat,
                                                                  int32_t* __restrict__ len,
                                                                  const int32_t* __restrict__ keep,
                                                                  int cap, int budget, int chunks) {
    const int row = blockIdx.x, part = (int)blockIdx.y - (Q4 > 0);
    if constexpr (Q4 > 0) {
        if (part < 0) {
            const int old = len[row];
            __syncthreads();   // every wavefront has it
            if (threadIdx.x == 0 && old > budget) len[row] = budget;
            feat_roll<Q4>(feat, row, min(old, cap), keep, cap, budget);
            return;
        }
    }
    const int n = cap;
    const int32_t* kp = keep + (size_t)row * budget;
    const int slices = chunks / kSliceChunks;
    if (part == 2 * slices) {
        if (Q4 == 0 && threadIdx.x == 0 && len[row] > budget) len[row] = budget;
        int32_t* p = pos + (size_t)row * cap;
        for (int base = 0; base < budget; base += kCompactThreads * U) {
            int32_t val[U];
            int src[U];
#pragma unroll
            for (int u = 0; u < U; ++u) src[u] = kp[min(base + u * kCompactThreads + (int)threadIdx.x, budget - 1)];
#pragma unroll
            for (int u = 0; u < U; ++u) val[u] = p[src[u] >= 0 && src[u] < n ? src[u] : 0];
#pragma unroll
            for (int u = 0; u < U; ++u) asm volatile("" : "+v"(val[u]));   // here before any slot is written
            __syncthreads();
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int j = base + u * kCompactThreads + threadIdx.x;
                if (j < budget && src[u] >= 0 && src[u] < n && src[u] != j) p[j] = val[u];
            }
        }
        return;
    }
    const int tensor = part / slices, slice = part % slices;
    uint4* X = (tensor == 0 ? K : V) + (size_t)row * cap * chunks + slice * kSliceChunks;
    constexpr int spi = kCompactThreads / kSliceChunks;  // slots per load instruction of the workgroup
    constexpr int tile = spi * U;
    const int sl = threadIdx.x / kSliceChunks;           // slot within that group
    const int c = threadIdx.x % kSliceChunks;            // 16-byte chunk inside the slice
    // One tile's rows and another tile's indices are in flight while a tile is stored (128 rows of 2048 kept pairs, 265 MB read and
    // written: 49 us with a round trip to memory per tile, 41.5 us, 6.4 TB/s, so).  The rows of tile t + 1 may be
    // read before tile t is stored: they lie at or behind their own destinations, past the slots of tile t.
    if constexpr (WALK != WALK_MOVED) {
        // Few workgroups: the loads are under no condition and two tiles take turns in their registers.  Behind conditions, or with a tile moved
        // from one set of registers to the other, the compiler waits for everything in flight before every store.  Figures: compact_kernel_for.
        auto load_idx = [&](int base, int (&src)[U]) {
#pragma unroll
            for (int u = 0; u < U; ++u) src[u] = kp[min(base + u * spi + sl, budget - 1)];
        };
        auto load_rows = [&](int base, const int (&src)[U], u32x4_t (&val)[U]) {   // a bit for every row that moves
            uint32_t moves = 0;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int j = base + u * spi + sl, s = src[u];
                const bool m = j < budget && s >= 0 && s < n && s != j;
                val[u] = *reinterpret_cast<const u32x4_t*>(X + (size_t)(m ? s : 0) * chunks + c);   // (the others: slot 0, not used)
                moves |= (uint32_t)m << u;
            }
            return moves;
        };
        auto store_rows = [&](int base, u32x4_t (&val)[U], uint32_t moves) {
#pragma unroll
            for (int u = 0; u < U; ++u) asm volatile("" : "+v"(val[u]));   // every row of the tile is here before any of its slots is written
            __syncthreads();
#pragma unroll
            for (int u = 0; u < U; ++u)
                if ((moves >> u) & 1) *reinterpret_cast<u32x4_t*>(X + (size_t)(base + u * spi + sl) * chunks + c) = val[u];
        };
        if constexpr (WALK == WALK_ONE) {   // the whole row is one tile
            int src[U];
            u32x4_t val[U];
            load_idx(0, src);
            const uint32_t moves = load_rows(0, src, val);
            store_rows(0, val, moves);
            return;
        }
        // ALONE: a slot that moves nothing costs this walk a load all the same.  Where the first two tiles have none that moves, the first one that
        // does is looked for in the indices alone, and the walk starts again there (32 rows of 8192 of which nothing moves 14.1 us, so 4.4; moved
        // from the third quarter on 19.0 and 13.1; 2048 at random as before).  The second copy of the loop takes the registers of a second workgroup.
        constexpr int WAVES = kCompactThreads / kWave, LOOK = 4;
        __shared__ int s_first[2][WAVES];   // a wavefront's first slot that moves; budget: none
        auto put_first = [&](int turn, int slot) {
            if (threadIdx.x % kWave == 0) s_first[turn][threadIdx.x / kWave] = slot;
        };
        auto get_first = [&](int turn) {
            int first = budget;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) first = min(first, s_first[turn][w]);
            return __builtin_amdgcn_readfirstlane(first);
        };
        auto walk = [&](int start, auto looking) {   // true: done; false: nothing moves in the first two tiles
            int src0[U], src1[U];
            u32x4_t val0[U], val1[U];
            load_idx(start, src0);
            load_idx(start + tile, src1);
            uint32_t moves0 = load_rows(start, src0, val0), moves1;
            for (int base = start; base < budget; base += 2 * tile) {
                load_idx(base + 2 * tile, src0);
                moves1 = load_rows(base + tile, src1, val1);
                if constexpr (looking) {
                    if (base == start) put_first(0, __any(moves0 | moves1) ? 0 : budget);
                }
                store_rows(base, val0, moves0);
                if constexpr (looking) {
                    if (base == start && get_first(0) == budget) return false;
                }
                if (base + tile >= budget) break;
                load_idx(base + 3 * tile, src1);
                moves0 = load_rows(base + 2 * tile, src0, val0);
                store_rows(base + tile, val1, moves1);
            }
            return true;
        };
        if (walk(0, std::integral_constant<bool, ALONE>())) return;
        int first = budget;
        for (int base = 2 * tile, turn = 1; first == budget && base < budget; base += LOOK * kCompactThreads, turn ^= 1) {
            int s[LOOK], mine = budget;
#pragma unroll
            for (int u = 0; u < LOOK; ++u) s[u] = kp[min(base + u * kCompactThreads + (int)threadIdx.x, budget - 1)];
#pragma unroll
            for (int u = LOOK - 1; u >= 0; --u) {
                const int j = base + u * kCompactThreads + (int)threadIdx.x;
                const unsigned long long m = __ballot(j < budget && s[u] >= 0 && s[u] < n && s[u] != j);
                if (m) mine = j - (int)(threadIdx.x % kWave) + __ffsll((long long)m) - 1;
            }
            put_first(turn, mine);
            __syncthreads();
            first = get_first(turn);
        }
        if (first < budget) walk(first / tile * tile, std::false_type());
    } else {
        auto load_idx = [&](int base, int (&src)[U]) {   // -1: nothing to move
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int j = base + u * spi + sl;
                const int s = j < budget ? kp[j] : -1;
                src[u] = s >= 0 && s < n && s != j ? s : -1;
            }
        };
        auto load_rows = [&](const int (&src)[U], u32x4_t (&val)[U]) {
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (src[u] >= 0) val[u] = *reinterpret_cast<const u32x4_t*>(X + (size_t)src[u] * chunks + c);
        };
        int now[U], next[U], after[U];
        u32x4_t val[U], val_next[U];
        load_idx(0, now);
        load_idx(tile, next);
        load_rows(now, val);
        for (int base = 0; base < budget; base += tile) {
            load_idx(base + 2 * tile, after);
            load_rows(next, val_next);
            __syncthreads();
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (now[u] >= 0) *reinterpret_cast<u32x4_t*>(X + (size_t)(base + u * spi + sl) * chunks + c) = val[u];
                now[u] = next[u];
                next[u] = after[u];
                val[u] = val_next[u];
            }
        }
    }
}

// By the workgroups that move rows (128 bytes of a slot each).  us, from the Infinity Cache / from HBM, WALK_MOVED and the form taken; rows of
// head_dim 128 in bf16 where nothing else is said:
//   one tile             32 rows of 512 of 640 pairs 4.7 / 6.6 and 4.2 / 6.5, 64 rows 6.6 / 11.2 and 5.5 / 10.5; tiles of 256 slots for up to 256
//                        pairs, 64 rows 5.2 / 7.6 and 4.0 / 6.4
//   two tiles in turns   4 rows of 20000 70.6 and 62.4; 32 rows of 2048 of 2176 11.3 / 19.0 and 10.0 / 18.2, out of 32768 13.5 / 15.5 and 12.1 /
//                        14.6; 64 rows of 2048 of 2176 19.6 / 31.1 and 18.1 / 30.9; head_dim 64, 96 rows of 2048 16.0 / 25.0 and 14.9 / 24.2
// Where they do not pay: kept bytes beyond the Infinity Cache (64 rows of 8192 80.7 and 84.4 from the cache, 32 of 16384 126 and 128), from 129
// workgroups on already half of it (48 rows of 8192, nothing of which moves, 11.7 and 14.3); scattered rows of more than 160 workgroups (head_dim
// 64, 96 rows of 2048 out of 32768 20.2 and 22.7); more than 256, which fill the chip twice (128 rows of 2048 with features 79.4 and 80.3 from
// HBM, fp32 88.5 and 89.9).  Up to 200, those of the features among them, a workgroup has a CU for itself: with two on some and none on others 16
// rows of 2048 take 14.4 us from HBM, so 14.0; beyond, a second round would begin (64 rows of 1024 8.7 and 9.4; with features, 48 of 2048 26.5
// and 26.9, head_dim 64, 96 of 2048 19.1 and 20.1).
template <int Q4> static auto compact_kernel_for(long long workgroups, int rows, int budget, int cap) {
    const bool alone = workgroups + (Q4 > 0 ? rows : 0) <= 200;
    if (workgroups <= 256 && budget <= 256) return alone ? compact_kernel<Q4, 2, WALK_ONE, true> : compact_kernel<Q4, 2, WALK_ONE, false>;
    if (workgroups <= 256 && budget <= 512) return alone ? compact_kernel<Q4, 4, WALK_ONE, true> : compact_kernel<Q4, 4, WALK_ONE, false>;
    const bool turns = workgroups <= 128 ? workgroups * budget < (1 << 21)
                                         : workgroups <= 256 && workgroups * budget <= (1 << 20) && (workgroups <= 160 || cap <= 4ll * budget);
    if (turns)
        return alone ? compact_kernel<Q4, 4, WALK_TURNS, true> : compact_kernel<Q4, 4, WALK_TURNS, false>;
    return compact_kernel<Q4, 4, WALK_MOVED, false>;
}

}  // namespace fk

using namespace fk;

extern "C" fk_status fk_append(const fk_cache_desc* desc, void* K, void* V, int32_t* pos, int32_t* len,
                               const void* k_new, const void* v_new, const int32_t* pos_new, void* stream) {
    fk_status s = check_desc(desc);
    if (s != FK_OK) return s;
    if (!K || !V || !pos || !len || !k_new || !v_new || !pos_new) return FK_ERR_INVALID_ARG;
    if (!aligned16(K) || !aligned16(V) || !aligned16(k_new) || !aligned16(v_new)) return FK_ERR_INVALID_ARG;
    const int chunks = desc->head_dim * (desc->dtype == FK_F32 ? 4 : 2) / 16;
    hipLaunchKernelGGL(append_kernel, dim3(desc->batch * desc->n_kv_heads), dim3(64), 0, (hipStream_t)stream, (uint4*)K,
                       (uint4*)V, pos, len, (const uint4*)k_new, (const uint4*)v_new, pos_new,
                       desc->n_kv_heads, desc->capacity, chunks);
    return launch_status();
}

extern "C" fk_status fk_compact(const fk_cache_desc* desc, void* K, void* V, int32_t* pos, int32_t* len,
                                const int32_t* keep_idx, int32_t budget, void* stream) {
    fk_status s = check_desc(desc);
    if (s != FK_OK) return s;
    if (!K || !V || !pos || !len || !keep_idx) return FK_ERR_INVALID_ARG;
    if (budget <= 0 || budget > desc->capacity) return FK_ERR_INVALID_ARG;
    if (!aligned16(K) || !aligned16(V)) return FK_ERR_INVALID_ARG;
    const int chunks = desc->head_dim * (desc->dtype == FK_F32 ? 4 : 2) / 16;
    const int rows = desc->batch * desc->n_kv_heads;
    hipStream_t st = (hipStream_t)stream;
    hipLaunchKernelGGL(compact_kernel_for<0>(rows * 2ll * (chunks / kSliceChunks), rows, budget, desc->capacity), dim3(rows, 2 * (chunks / kSliceChunks) + 1), dim3(kCompactThreads), 0, st, (uint4*)K, (uint4*)V,
                       pos, nullptr, len, keep_idx, desc->capacity, budget, chunks);
    return launch_status();
}

extern "C" fk_status fk_compact_feat(const fk_cache_desc* desc, void* K, void* V, int32_t* pos, float* feat,
                                     int32_t* len, const int32_t* keep_idx, int32_t budget, void* stream) {
    fk_status s = check_desc(desc);
    if (s != FK_OK) return s;
    if (!K || !V || !pos || !feat || !len || !keep_idx) return FK_ERR_INVALID_ARG;
    if (budget <= 0 || budget > desc->capacity) return FK_ERR_INVALID_ARG;
    if (!aligned16(K) || !aligned16(V) || !aligned16(feat)) return FK_ERR_INVALID_ARG;
    const int chunks = desc->head_dim * (desc->dtype == FK_F32 ? 4 : 2) / 16;
    const int rows = desc->batch * desc->n_kv_heads;
    const int g = desc->n_q_heads / desc->n_kv_heads;
    hipStream_t st = (hipStream_t)stream;
    const long long workgroups = rows * 2ll * (chunks / kSliceChunks);
    const auto kern = g <= 4 ? compact_kernel_for<1>(workgroups, rows, budget, desc->capacity) : compact_kernel_for<2>(workgroups, rows, budget, desc->capacity);
    hipLaunchKernelGGL(kern, dim3(rows, 2 * (chunks / kSliceChunks) + 2), dim3(kCompactThreads), 0, st, (uint4*)K, (uint4*)V, pos,
                       (float4*)feat, len, keep_idx, desc->capacity, budget, chunks);
    return launch_status();
}
