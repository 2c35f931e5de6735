// The order in which the exact KNN of Sec. 3.2 streams a head's keys.
//
// The top-knn selection is exact whatever the order, but its cost is not: a key goes through the
// selection's slow path whenever its score reaches the query's current threshold, and over a
// stream in storage order that happens about knn * ln(N / knn) times per query. Queries of one
// attention head share a large common component (they are out of distribution with respect to
// the keys, Sec. 2.4), so the keys that score high for the head's MEAN query score high for most
// of its queries. Streaming the keys by descending inner product with that mean raises every
// threshold within the first few stages, and the rest of the stream seldom reaches it.
//
// Three steps per head, none of which can change a result:
//   ko_meanq_kernel   sum of a strided sample of the head's prefill queries (fixed order)
//   ko_proxy_kernel   64-bit sort keys [~ordered(<mean, k_i>):32][i:32], all ones beyond N
//   ko_sort_*         ascending sort: chunks by score in LDS, then a bitonic network over them, its wider exchanges
//                     in memory
// so entry p is the key of p-th largest inner product (lower id first among equals) and the KNN
// kernel reads the id of stream position p as the low word of entry p, ready to use.
#include "common.h"

typedef unsigned long long u64;

#define KO_SAMPLE 4096            // prefill queries summed per head (at most)
#define KO_CHUNK 8192             // sort keys a workgroup holds in LDS (64 KB)
#define KO_THREADS 1024
#define KO_FLY 4                  // key rows in flight per 16 lanes
#define KO_MEAN_T 256             // 64 groups of 4 lanes
#define KO_BINS 2048              // of a chunk's scores
#define KO_BIN_MOST 96            // keys in one bin that are still ordered by comparing them with each other

template <int DT>
__device__ __forceinline__ void ko_row8(const void* base, size_t at, float (&v)[8]) {
    if constexpr (DT == RA_BF16) {
        const uint4 u = *reinterpret_cast<const uint4*>(reinterpret_cast<const uint16_t*>(base) + at);
        v[0] = bf16_lo(u.x); v[1] = bf16_hi(u.x); v[2] = bf16_lo(u.y); v[3] = bf16_hi(u.y);
        v[4] = bf16_lo(u.z); v[5] = bf16_hi(u.z); v[6] = bf16_lo(u.w); v[7] = bf16_hi(u.w);
    } else {
        const float4 a = *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(base) + at);
        const float4 b = *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(base) + at + 4);
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
    }
}

// grid: x = head, y = quarter of the dimensions (64 heads x 4096 rows: 19 us with one workgroup per head, now 14). 4 lanes per
// row; lane group s sums samples s, s + 64, ... sixteen rows in flight
// (a serial sum of rows, one at a time, was 265 us of latency whatever the size of the input).
template <int DT>
__global__ __launch_bounds__(KO_MEAN_T) void ko_meanq_kernel(const void* __restrict__ Q, int64_t M,
                                                             float* __restrict__ mq) {
    constexpr int GROUPS = KO_MEAN_T / 4, FLY = 16, DIMS = RA_D / 4;
    __shared__ float part[GROUPS][DIMS];
    const int graph = blockIdx.x, d0 = blockIdx.y * DIMS, l4 = threadIdx.x & 3, s = threadIdx.x / 4;
    const int n_s = M < KO_SAMPLE ? (int)M : KO_SAMPLE;
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int k0 = s; k0 < n_s; k0 += FLY * GROUPS) {
        float v[FLY][8];
#pragma unroll
        for (int u = 0; u < FLY; ++u) {
            const int k = k0 + u * GROUPS < n_s ? k0 + u * GROUPS : k0;
            const int64_t j = M <= KO_SAMPLE ? k : (int64_t)k * M / KO_SAMPLE;
            ko_row8<DT>(Q, ((size_t)graph * M + j) * RA_D + d0 + 8 * l4, v[u]);
        }
#pragma unroll
        for (int u = 0; u < FLY; ++u)
            if (k0 + u * GROUPS < n_s)
#pragma unroll
                for (int c = 0; c < 8; ++c) acc[c] += v[u][c];
    }
#pragma unroll
    for (int c = 0; c < 8; ++c) part[s][8 * l4 + c] = acc[c];
    __syncthreads();
    if (threadIdx.x < DIMS) {
        float t = 0.f;
        for (int i = 0; i < GROUPS; ++i) t += part[i][threadIdx.x];
        mq[(size_t)graph * RA_D + d0 + threadIdx.x] = t;
    }
}

// grid: x = block of 64 * KO_FLY stream slots, y = HEADS query heads of a KV head. 16 lanes per key row, KO_FLY rows in flight, each
// read once for all HEADS. (One row and one head at a time, a key row went through a compute unit once per query head with nothing
// else on its way: 64 heads x 5003 keys 26.5 us, 32 x 128K 220; now 12 and 79.)
template <int DT, int HEADS>
__global__ __launch_bounds__(KO_THREADS) void ko_proxy_kernel(const void* __restrict__ K,
                                                              const float* __restrict__ mq, int n_q,
                                                              int n_kv, int64_t N, int64_t N_pad,
                                                              u64* __restrict__ keys) {
    const int graph0 = blockIdx.y * HEADS, seq = graph0 / n_q, h0 = graph0 % n_q, kvh = h0 / (n_q / n_kv);
    const int l16 = threadIdx.x & 15, lane = threadIdx.x % RA_WAVE;
    const int64_t i0 = (int64_t)blockIdx.x * (KO_THREADS / 16 * KO_FLY) + threadIdx.x / 16;
    if (i0 >= N_pad) return;                    // whole 16-lane groups leave together
    float k[KO_FLY][8];
#pragma unroll
    for (int u = 0; u < KO_FLY; ++u) {
        const int64_t i = i0 + u * (KO_THREADS / 16), row = i < N ? i : N - 1;
        ko_row8<DT>(K, (((size_t)seq * n_kv + kvh) * N + row) * RA_D + 8 * l16, k[u]);
    }
#pragma unroll
    for (int g = 0; g < HEADS; ++g) {
        const float* m = mq + (size_t)(graph0 + g) * RA_D + 8 * l16;
        const float4 ma = *reinterpret_cast<const float4*>(m), mb = *reinterpret_cast<const float4*>(m + 4);
        const float mv[8] = {ma.x, ma.y, ma.z, ma.w, mb.x, mb.y, mb.z, mb.w};
#pragma unroll
        for (int u = 0; u < KO_FLY; ++u) {
            const int64_t i = i0 + u * (KO_THREADS / 16);
            float p = 0.f;
#pragma unroll
            for (int c = 0; c < 8; ++c) p += k[u][c] * mv[c];
            p += __uint_as_float(lane_xor32<1>(__float_as_uint(p), lane));
            p += __uint_as_float(lane_xor32<2>(__float_as_uint(p), lane));
            p += __uint_as_float(lane_xor32<4>(__float_as_uint(p), lane));
            p += __uint_as_float(lane_xor32<8>(__float_as_uint(p), lane));
            if (p != p) p = 0.f;                // an order is all that is wanted: any place will do
            // ids stay below 2^31, so the all-ones entries beyond N sort behind every key
            if (l16 == 0 && i < N_pad)
                keys[(size_t)(graph0 + g) * N_pad + i] = i < N ? ((u64)(~f32_ordered(p)) << 32) | (u64)(uint32_t)i : ~0ull;
        }
    }
}

// One exchange of the bitonic network on a chunk in LDS: element e and e ^ j, ascending overall
// (the run that holds global index g descends when g & k is set).
__device__ __forceinline__ void ko_exchange(u64* s, int e, int j, bool ascending) {
    const u64 a = s[e], b = s[e | j];
    if ((a > b) == ascending) { s[e] = b; s[e | j] = a; }
}

// How many keys of array y there are to sort: `counts` (one int every count_stride) or all N_pad. The
// network runs over the smallest power of two of them; what it would do beyond is skipped, and the
// first pass over a chunk takes places beyond the count for all-ones keys.
__device__ __forceinline__ int64_t ko_count(const int32_t* counts, size_t count_stride, int64_t N_pad) {
    return counts ? counts[(size_t)blockIdx.y * count_stride] : N_pad;
}
__device__ __forceinline__ int64_t ko_run(int64_t n) {
    return n <= 1 ? 1 : (int64_t)1 << (64 - __clzll((long long)(n - 1)));
}

// Stage k of the network, from distance half a chunk at most, on the chunk in LDS (filled, with a barrier after).
__device__ __forceinline__ void ko_stage(u64* s, int chunk, int64_t base, int64_t k) {
    const int j_top = k > chunk ? chunk / 2 : (int)(k / 2);
    for (int j = j_top; j >= 1; j >>= 1) {
        for (int t = threadIdx.x; t < chunk / 2; t += KO_THREADS) {
            const int e = ((t & ~(j - 1)) << 1) | (t & (j - 1));      // bit j clear
            ko_exchange(s, e, j, ((base + e) & k) == 0);
        }
        __syncthreads();
    }
}

// grid: x = chunk, y = array of score keys (ko_proxy_kernel). Sorts each chunk, ascending or descending as the network over the
// chunks wants it. The network's 91 exchanges of 8192 keys are 91 round trips through LDS and barriers (73 us for 64
// arrays of 5003, now 13); here keys are dealt to 2048 equal-width bins of their score, and a key's place is the keys in earlier bins
// plus the smaller keys of its own, of which there are about ten where scores are densest. A chunk
// with a crowded bin (equal scores, a wide outlier), or whose scores' width is not finite, takes the network.
__global__ __launch_bounds__(KO_THREADS) void ko_sort_scores_kernel(u64* __restrict__ keys, size_t stride, int chunk) {
    extern __shared__ __align__(16) unsigned char ko_lds[];
    constexpr int PER = KO_CHUNK / KO_THREADS, OWN = KO_BINS / KO_THREADS, WAVES = KO_THREADS / RA_WAVE;
    u64* s = reinterpret_cast<u64*>(ko_lds);
    int* start = reinterpret_cast<int*>(s + chunk);               // [KO_BINS + 1] counts, then first places
    int* wave_sum = start + KO_BINS + 1;
    unsigned* ends = reinterpret_cast<unsigned*>(wave_sum + WAVES);       // smallest and largest upper half; [2] a bin is crowded
    const int tid = threadIdx.x, lane = tid % RA_WAVE, wv = tid / RA_WAVE;
    const int64_t base = (int64_t)blockIdx.x * chunk;
    u64* g = keys + (size_t)blockIdx.y * stride + base;
    u64 k[PER];
#pragma unroll
    for (int r = 0; r < PER; ++r) k[r] = r * KO_THREADS + tid < chunk ? g[r * KO_THREADS + tid] : ~0ull;
    for (int b = tid; b < KO_BINS; b += KO_THREADS) start[b] = 0;
    if (tid < 3) ends[tid] = tid == 0 ? 0xffffffffu : 0u;
    __syncthreads();
    unsigned lo = 0xffffffffu, hi = 0u;
#pragma unroll
    for (int r = 0; r < PER; ++r)
        if (k[r] != ~0ull) {                                      // (places beyond N)
            lo = min(lo, (unsigned)(k[r] >> 32));
            hi = max(hi, (unsigned)(k[r] >> 32));
        }
    for (int d = RA_WAVE / 2; d >= 1; d >>= 1) {
        lo = min(lo, (unsigned)__shfl_xor((int)lo, d));
        hi = max(hi, (unsigned)__shfl_xor((int)hi, d));
    }
    if (lane == 0) {
        atomicMin(&ends[0], lo);
        atomicMax(&ends[1], hi);
    }
    __syncthreads();
    if (ends[0] > ends[1]) return;                                // nothing but places beyond N
    // the upper halves are complements: the smallest is the largest score. Every operation is monotone in the score, so a
    // larger score is never in a later bin.
    const float top = f32_from_ordered(~ends[0]), width = top - f32_from_ordered(~ends[1]);
    const float to_bin = width > 0.f && width < INFINITY ? (float)(KO_BINS - 1) / width : 0.f;
    int bin[PER], at[PER];
#pragma unroll
    for (int r = 0; r < PER; ++r) {
        const float b = (top - f32_from_ordered(~(uint32_t)(k[r] >> 32))) * to_bin;
        bin[r] = b >= (float)(KO_BINS - 1) ? KO_BINS - 1 : b > 0.f ? (int)b : 0;
        at[r] = k[r] != ~0ull ? atomicAdd(&start[bin[r]], 1) : 0;
    }
    __syncthreads();
    int own[OWN], sum = 0;
    bool crowded = false;
#pragma unroll
    for (int b = 0; b < OWN; ++b) {
        own[b] = start[OWN * tid + b];
        crowded = crowded || own[b] > KO_BIN_MOST;
        sum += own[b];
    }
    int incl = sum;
    for (int d = 1; d < RA_WAVE; d <<= 1) {
        const int v = __shfl_up(incl, d);
        if (lane >= d) incl += v;
    }
    if (lane == RA_WAVE - 1) wave_sum[wv] = incl;
    if (crowded) ends[2] = 1u;
    __syncthreads();
    if (ends[2]) {                                                // (uniform)
#pragma unroll
        for (int r = 0; r < PER; ++r)
            if (r * KO_THREADS + tid < chunk) s[r * KO_THREADS + tid] = k[r];
        __syncthreads();
        for (int64_t size = 2; size <= chunk; size <<= 1) ko_stage(s, chunk, base, size);
        for (int e = tid; e < chunk; e += KO_THREADS) g[e] = s[e];
        return;
    }
    int before = incl - sum;
    for (int w = 0; w < wv; ++w) before += wave_sum[w];
#pragma unroll
    for (int b = 0; b < OWN; ++b) {
        start[OWN * tid + b] = before;
        before += own[b];
    }
    if (tid == KO_THREADS - 1) start[KO_BINS] = before;           // the chunk's keys
    __syncthreads();
#pragma unroll
    for (int r = 0; r < PER; ++r)
        if (k[r] != ~0ull) s[start[bin[r]] + at[r]] = k[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < PER; ++r) {
        const int b0 = start[bin[r]], b1 = start[bin[r] + 1];
        at[r] = b0;
        for (int j = b0; j < b1; ++j) at[r] += s[j] < k[r] ? 1 : 0;
    }
    const int n = start[KO_BINS];
    const bool descending = (base & chunk) != 0;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < PER; ++r)
        if (k[r] != ~0ull) s[descending ? chunk - 1 - at[r] : at[r]] = k[r];
    for (int e = n + tid; e < chunk; e += KO_THREADS) s[descending ? chunk - 1 - e : e] = ~0ull;
    __syncthreads();
    for (int e = tid; e < chunk; e += KO_THREADS) g[e] = s[e];
}

// grid: x = chunk, y = array. k_first == 0: sorts the chunk (all k up to its length); otherwise
// finishes stage k_first of the global network (j from half a chunk down to 1).
__global__ __launch_bounds__(KO_THREADS) void ko_sort_chunk_kernel(u64* __restrict__ keys, size_t stride,
                                                                   int64_t N_pad, int chunk, int64_t k_first,
                                                                   const int32_t* __restrict__ counts,
                                                                   size_t count_stride) {
    extern __shared__ __align__(16) unsigned char ko_lds[];
    u64* s = reinterpret_cast<u64*>(ko_lds);
    const int64_t base = (int64_t)blockIdx.x * chunk;
    const int64_t n = ko_count(counts, count_stride, N_pad), run = ko_run(n);
    if (base >= run || k_first > run) return;            // (the whole workgroup)
    if (chunk > run) chunk = (int)run;
    u64* g = keys + (size_t)blockIdx.y * stride + base;
    for (int e = threadIdx.x; e < chunk; e += KO_THREADS) s[e] = k_first || base + e < n ? g[e] : ~0ull;
    __syncthreads();
    for (int64_t k = k_first ? k_first : 2; k_first ? k == k_first : k <= chunk; k <<= 1) ko_stage(s, chunk, base, k);
    for (int e = threadIdx.x; e < chunk; e += KO_THREADS) g[e] = s[e];
}

// grid: x = block of KO_THREADS pairs, y = array: the exchange at distance j >= chunk of stage k.
__global__ __launch_bounds__(KO_THREADS) void ko_sort_far_kernel(u64* __restrict__ keys, size_t stride,
                                                                 int64_t N_pad, int64_t k, int64_t j,
                                                                 const int32_t* __restrict__ counts,
                                                                 size_t count_stride) {
    const int64_t t = (int64_t)blockIdx.x * KO_THREADS + threadIdx.x;
    const int64_t run = ko_run(ko_count(counts, count_stride, N_pad));
    if (k > run || t >= run / 2) return;
    const int64_t e = ((t & ~(j - 1)) << 1) | (t & (j - 1));
    u64* g = keys + (size_t)blockIdx.y * stride;
    const u64 a = g[e], b = g[e | j];
    const bool ascending = (e & k) == 0;
    if ((a > b) == ascending) { g[e] = b; g[e | j] = a; }
}

// Ascending sort of n_arrays arrays of 64-bit keys, `stride` keys apart, of N_pad (a power of two)
// places each; `counts` (device, one int every count_stride): how many keys each holds, or null: N_pad, and the keys'
// upper halves are scores (ko_proxy_kernel). Chunks of keys with counts, popularities with few values each, take the network.
ra_status ra_launch_sort(void* keys, size_t stride, int n_arrays, int64_t N_pad, const int32_t* counts,
                         size_t count_stride, hipStream_t st) {
    u64* k64 = reinterpret_cast<u64*>(keys);
    const int chunk = (int)(N_pad < KO_CHUNK ? N_pad : KO_CHUNK);
    const size_t lds = (size_t)chunk * sizeof(u64);
    const dim3 cgrid((unsigned)(N_pad / chunk), (unsigned)n_arrays);
    const dim3 fgrid((unsigned)((N_pad / 2 + KO_THREADS - 1) / KO_THREADS), (unsigned)n_arrays);
    RA_LDS_OPT_IN(ko_sort_chunk_kernel, lds);
    if (counts) {
        hipLaunchKernelGGL(ko_sort_chunk_kernel, cgrid, dim3(KO_THREADS), lds, st, k64, stride, N_pad, chunk, (int64_t)0,
                           counts, count_stride);
    } else {
        const size_t lds_scores = lds + (KO_BINS + 1 + KO_THREADS / RA_WAVE + 3) * sizeof(int);
        RA_LDS_OPT_IN(ko_sort_scores_kernel, lds_scores);
        hipLaunchKernelGGL(ko_sort_scores_kernel, cgrid, dim3(KO_THREADS), lds_scores, st, k64, stride, chunk);
    }
    for (int64_t k = 2 * (int64_t)chunk; k <= N_pad; k <<= 1) {
        for (int64_t j = k / 2; j >= chunk; j >>= 1)
            hipLaunchKernelGGL(ko_sort_far_kernel, fgrid, dim3(KO_THREADS), 0, st, k64, stride, N_pad, k, j, counts,
                               count_stride);
        hipLaunchKernelGGL(ko_sort_chunk_kernel, cgrid, dim3(KO_THREADS), lds, st, k64, stride, N_pad, chunk, k,
                           counts, count_stride);
    }
    RA_HIP(hipGetLastError());
    return RA_OK;
}

int64_t ra_sort_padded(int64_t N) {
    int64_t p = 2;
    while (p < N) p <<= 1;
    return p;
}

// [n_graphs][N_pad] sort keys, then [n_graphs][RA_D] query sums
size_t ra_knn_order_bytes(int n_graphs, int64_t N) {
    return (size_t)n_graphs * ((size_t)ra_sort_padded(N) * sizeof(u64) + RA_D * sizeof(float));
}

int64_t ra_knn_order_stride(int64_t N) { return ra_sort_padded(N); }

const float* ra_knn_order_mean(const void* workspace, int graphs, int64_t N, int64_t M, int* samples) {
    *samples = M < KO_SAMPLE ? (int)M : KO_SAMPLE;
    return reinterpret_cast<const float*>(reinterpret_cast<const u64*>(workspace) + (size_t)graphs * ra_sort_padded(N));
}

// Fills workspace with the stream order of every head: entry p of head g, at
// workspace[g * ra_knn_order_stride(N) + p], holds the id of the key streamed p-th in its low word.
ra_status ra_launch_knn_order(const void* K, const void* Q, ra_dtype dt, int n_seq, int n_q, int n_kv,
                              int64_t N, int64_t M, void* workspace, hipStream_t st) {
    const int graphs = n_seq * n_q;
    if (graphs > 65535) RA_FAIL(RA_EUNSUP, "more than 65535 (sequence, query head) pairs");
    const int64_t N_pad = ra_sort_padded(N);
    u64* keys = reinterpret_cast<u64*>(workspace);
    float* mq = reinterpret_cast<float*>(keys + (size_t)graphs * N_pad);
    const int group = n_q / n_kv, heads = group % 4 == 0 ? 4 : group % 2 == 0 ? 2 : 1;
    const int64_t per = KO_THREADS / 16 * KO_FLY;
    const dim3 mgrid(graphs, 4), pgrid((unsigned)((N_pad + per - 1) / per), (unsigned)(graphs / heads));
#define KO_GO(DTV)                                                                                                       \
    do {                                                                                                                 \
        hipLaunchKernelGGL(ko_meanq_kernel<DTV>, mgrid, dim3(KO_MEAN_T), 0, st, Q, M, mq);                               \
        if (heads == 4)                                                                                                  \
            hipLaunchKernelGGL((ko_proxy_kernel<DTV, 4>), pgrid, dim3(KO_THREADS), 0, st, K, mq, n_q, n_kv, N, N_pad, keys); \
        else if (heads == 2)                                                                                             \
            hipLaunchKernelGGL((ko_proxy_kernel<DTV, 2>), pgrid, dim3(KO_THREADS), 0, st, K, mq, n_q, n_kv, N, N_pad, keys); \
        else                                                                                                             \
            hipLaunchKernelGGL((ko_proxy_kernel<DTV, 1>), pgrid, dim3(KO_THREADS), 0, st, K, mq, n_q, n_kv, N, N_pad, keys); \
    } while (0)
    if (dt == RA_BF16) KO_GO(RA_BF16); else KO_GO(RA_F32);
#undef KO_GO
    RA_HIP(hipGetLastError());
    return ra_launch_sort(keys, (size_t)N_pad, graphs, N_pad, nullptr, 0, st);
}
