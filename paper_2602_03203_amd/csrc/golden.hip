// Golden Eviction label builder (Section 3.2 Eq. 3-5) on dense causal attention matrices.
//
//   pool   a~[h'][t][i] = 1/(g L) * sum over the g heads of group h' and the queries q of block t
//                         (B + tL <= q < min(B + (t+1)L, T)) of A[h][q][i]          (Eq. 3, 4)
//   future alpha[h'][t][i] = max_{j >= t} a~[h'][j][i]                               (Eq. 5, first half)
//   trace  step t keeps the L newest pairs and, of the other B the cache holds, the B - L with
//          the largest alpha[.][t] (ties: lower position), evicted pairs never return  (Eq. 5, second half)
//
// pool is the only kernel that touches the O(T^2) input and is HBM bound: a workgroup owns one
// (key tile, block, group) and streams g * L row segments of 256 bytes (16 lanes x 16 bytes, 16 rows per workgroup
// instruction, eight loads in flight per thread); chunks wholly above the diagonal are never read (A is causal), so
// the traffic is the lower triangle below query B + L.  future is a
// running maximum down the block axis; trace is sequential by nature: one workgroup per group walks the
// M steps with the selection of fk_select_keep on keys in LDS (the next step's are loaded while a step selects).
#include "select_common.h"

namespace fk {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
static constexpr int kPoolThreads = 256;
static constexpr int kPoolU = 8;   // loads in flight per thread

// 32 heads of 8192 tokens, bf16: 2.0 GB of causal entries in 341 us, 5.9 TB/s (354 us with a division per load to find the load's
// head and query, four loads in flight).  Wider segments are no faster, 512 bytes 343 us, 1 KB 370 us: the fewer and longer
// workgroups leave CUs idle at the end.
// FEW: blocks of fewer than 64 queries.
template <typename T, bool FEW>
__global__ __launch_bounds__(kPoolThreads) void golden_pool_kernel(const T* __restrict__ A, int g, int Tn, size_t ld,
                                                                   int budget, int L, int M,
                                                                   float* __restrict__ a_tilde) {
    constexpr int EPC = Vec16<T>::N;   // elements per 16-byte chunk
    constexpr int LPR = 16;            // lanes of a row segment
    constexpr int KT = LPR * EPC;      // keys per tile
    constexpr int RG = kPoolThreads / LPR;   // row groups of the workgroup
    const int i0 = blockIdx.x * KT, t = blockIdx.y + 1, hp = blockIdx.z;
    const int q0 = budget + t * L, q1 = min(q0 + L, Tn);
    const int c = threadIdx.x % LPR, rg = threadIdx.x / LPR;
    const int i_mine = i0 + c * EPC;   // this lane's first key; queries before it see none of its keys and are not read
    float acc[EPC];
#pragma unroll
    for (int e = 0; e < EPC; ++e) acc[e] = 0.f;
    const int qs = max(q0, i0), rows = q1 - qs;   // rows <= 0: above the diagonal for the whole block
    if (i_mine < q1 && (size_t)i_mine < ld) {
        // read once, never again: non-temporal, so the lines do not push anything out of the caches
        auto load = [](const T* p) { return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p)); };
        if constexpr (!FEW) {   // head by head
            for (int h = 0; h < g; ++h) {
                const T* head = A + (size_t)(hp * g + h) * Tn * ld + i_mine;
                for (int q = qs + rg; q < q1; q += RG * kPoolU) {
                    u32x4 v[kPoolU];
#pragma unroll
                    for (int u = 0; u < kPoolU; ++u) {
                        const int qu = q + u * RG;
                        v[u] = (u32x4){0, 0, 0, 0};
                        if (qu < q1 && qu >= i_mine) v[u] = load(head + (size_t)qu * ld);
                    }
                    float x[kPoolU][EPC];
#pragma unroll
                    for (int u = 0; u < kPoolU; ++u) Vec16<T>::unpack(make_uint4(v[u].x, v[u].y, v[u].z, v[u].w), x[u]);
#pragma unroll
                    for (int e = 0; e < EPC; ++e)
                        acc[e] += ((x[0][e] + x[1][e]) + (x[2][e] + x[3][e])) + ((x[4][e] + x[5][e]) + (x[6][e] + x[7][e]));
                }
            }
        } else {
            // A head has less than the loads in flight take, so they go on into the next ones.  (Head by head, 32 heads of 4096 tokens, L = 16:
            // 226 us, so 131; 32 heads of 2000 tokens in 4 groups, L = 8: 107 and 55.  From 64 queries on, head by head is 1 to 3 % the
            // faster; a kernel of its own, because the other one's registers cost these short workgroups their number on a CU, 8 heads of 4096 tokens
            // without pooling, L = 32: 52 us in one kernel, 42 so.)  This row group takes pairs (head, query) rg, rg + RG, ...: dh heads and dq queries on, one head
            // more where that leaves the block.
            constexpr int U = kPoolU / 2;
            const int total = rows * g, dh = RG / rows, dq = RG % rows;
            const size_t step = ((size_t)dh * Tn + dq) * ld, wrap = (size_t)(Tn - rows) * ld;
            int q = rg % rows;
            const T* p = A + ((size_t)(hp * g + rg / rows) * Tn + qs + q) * ld + i_mine;
            for (int r = rg; r < total; r += RG * U) {
                u32x4 v[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    v[u] = (u32x4){0, 0, 0, 0};
                    if (r + u * RG < total && qs + q >= i_mine) v[u] = load(p);
                    p += step;
                    q += dq;
                    if (q >= rows) {
                        q -= rows;
                        p += wrap;
                    }
                }
                float x[U][EPC];
#pragma unroll
                for (int u = 0; u < U; ++u) Vec16<T>::unpack(make_uint4(v[u].x, v[u].y, v[u].z, v[u].w), x[u]);
#pragma unroll
                for (int e = 0; e < EPC; ++e) acc[e] += (x[0][e] + x[1][e]) + (x[2][e] + x[3][e]);
            }
        }
    }
    __shared__ float s_acc[RG][KT + 4];
#pragma unroll
    for (int e = 0; e < EPC; ++e) s_acc[rg][c * EPC + e] = acc[e];
    __syncthreads();
    for (int k = threadIdx.x; k < KT && i0 + k < Tn; k += kPoolThreads) {
        float s = 0.f;
#pragma unroll
        for (int r = 0; r < RG; ++r) s += s_acc[r][k];
        a_tilde[((size_t)hp * M + (t - 1)) * Tn + i0 + k] = s / ((float)g * (float)L);
    }
}

// alpha[t] = max(a~[t], alpha[t + 1]), walking the blocks from the last to the first; one thread per key,
// eight blocks' loads in flight
__global__ void golden_future_kernel(const float* __restrict__ a_tilde, int Tn, int M, float* __restrict__ alpha) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x, hp = blockIdx.y;
    if (i >= Tn) return;
    const size_t o0 = (size_t)hp * M * Tn + i;
    float run = 0.f;
    for (int t = M; t >= 1; t -= 8) {
        float a[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) a[u] = t - u >= 1 ? a_tilde[o0 + (size_t)(t - u - 1) * Tn] : 0.f;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (t - u >= 1) {
                run = t - u == M ? a[u] : fmaxf(run, a[u]);
                alpha[o0 + (size_t)(t - u - 1) * Tn] = run;
            }
        }
    }
}

static constexpr int kTraceMaxCache = 12288;  // B + L positions and B keys in LDS (96 KB)

// One workgroup per KV group.  LDS holds the cache's positions (ascending; B + L of them: the B of this step and the
// L that are generated before the next one) and the keys of its first B entries under this step's future scores.
// A step: (1) the loads of the NEXT step's future scores at every position that can still be a candidate then are
// issued (they land while the step selects); (2) range_select finds the key of the (B - L)-th best candidate;
// (3) every wavefront walks its own contiguous stretch of the candidates, first to count its survivors, then, with
// the counts of the stretches before it, to move them (position and next key) to the front in order.  Sources are
// in registers before the barrier that precedes the moves, so the compaction is safe in place.
// PER_LANE: candidates one lane holds (stretch of a wavefront / 64) and newest pairs one thread holds (L / 1024), at most.
template <int PER_LANE>
__global__ __launch_bounds__(kSelThreads) void golden_trace_kernel(const float* __restrict__ alpha, int Tn, int M,
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
    if (dtype == FK_F32) {
        const int KT = 64;
        hipLaunchKernelGGL((interval < 64 ? golden_pool_kernel<float, true> : golden_pool_kernel<float, false>), dim3((T + KT - 1) / KT, M, n_kv_heads), dim3(kPoolThreads), 0, st,
                           (const float*)A, g, T, (size_t)ld, budget, interval, M, block_scores);
    } else {
        const int KT = 128;
        hipLaunchKernelGGL((interval < 64 ? golden_pool_kernel<bf16_t, true> : golden_pool_kernel<bf16_t, false>), dim3((T + KT - 1) / KT, M, n_kv_heads), dim3(kPoolThreads), 0, st,
                           (const bf16_t*)A, g, T, (size_t)ld, budget, interval, M, block_scores);
    }
    hipLaunchKernelGGL(golden_future_kernel, dim3((T + 255) / 256, n_kv_heads), dim3(256), 0, st, block_scores, T, M, alpha);
    return launch_status();
}

extern "C" fk_status fk_golden_trace(const float* alpha, int32_t n_kv_heads, int32_t T, int32_t budget, int32_t interval,
                                     int32_t* kept, void* stream) {
    if (!alpha || !kept) return FK_ERR_INVALID_ARG;
    if (n_kv_heads <= 0 || T <= 0 || budget <= 0 || interval <= 0 || interval > budget) return FK_ERR_INVALID_ARG;
    if (budget + interval > kTraceMaxCache) return FK_ERR_UNSUPPORTED;
    const int M = golden_steps(T, budget, interval);
    if (M == 0) return FK_OK;
    const size_t lds = sizeof(int32_t) * ((size_t)budget + interval) + sizeof(uint32_t) * (size_t)budget;
    // candidates per lane: a wavefront's stretch is the budget over the 16 wavefronts, rounded up to whole 64s
    const int per_lane = ((budget + kSelWaves - 1) / kSelWaves + kWave - 1) / kWave;
    auto launch = [&](auto kern, bool (&lds_ok)[kMaxDevices]) -> fk_status {
        if (!allow_dynamic_lds((const void*)kern, sizeof(int32_t) * 2 * kTraceMaxCache, lds_ok)) return FK_ERR_LAUNCH;
        hipLaunchKernelGGL(kern, dim3(n_kv_heads), dim3(kSelThreads), lds, (hipStream_t)stream, alpha, T, M, budget, interval,
                           kept);
        return launch_status();
    };
    static bool ok2[kMaxDevices] = {}, ok4[kMaxDevices] = {}, ok12[kMaxDevices] = {};
    if (per_lane <= 2) return launch(golden_trace_kernel<2>, ok2);
    if (per_lane <= 4) return launch(golden_trace_kernel<4>, ok4);
    return launch(golden_trace_kernel<12>, ok12);   // budget + interval <= kTraceMaxCache: at most 12
}
