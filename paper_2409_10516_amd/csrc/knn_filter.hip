// The long part of the exact KNN's key stream (Sec. 3.2), at the integer rate of the matrix cores.
//
// knn.hip multiplies a head's prefill queries with the first keys of the stream order and leaves
// every query its best knn keys so far with their scores. From there on nearly every key is below
// every threshold (stream order puts the keys that matter first: knn_order.hip), and proving that a
// score stays below a threshold does not take the score itself. This file streams the remaining
// keys through an 8-bit copy of keys and queries and an error bound that holds for every pair; only
// keys that the bound cannot rule out are scored, with the same instructions on the same inputs in
// the same order as in knn.hip, so the lists are the same bits as without the filter.
//
// The bound. With m the head's mean query (its sum, knn_order.hip) and a = <q, m> / <m, m>, a score is
// a <m, k> + <r, k>, r = q - a m. The first term is known: the keys come by descending <m, k>, so in a
// segment of the stream it is at most a times the first key's (or the last one's, for negative a). The second
// is small where the queries of a head share a large common component. Per KV head and dimension,
// c_d = max_i |k_id| / 127 and k_id = c_d (x_id + e_id) with x_id the nearest integer; per query
// r'_d = r_d c_d = s (y_d + f_d) with s = max_d |r'_d| / 127 and y_d the nearest integer. Then
//     <r, k> = s <y, x> + s <f, x> + <r', e>,   |<r, k> - s <y, x>| <= s |f| |x| + |r'| |e|,
// where <y, x> is an exact integer (at most 128 x 127 x 127) from v_mfma_i32_32x32x32_i8 and the
// largest |x| and |e| over a segment's keys are taken when the copy is made. Every norm is taken relative to
// a power of two or to s (|r'| = s |y + f|), so none of them loses its terms where squares of the
// inputs leave the range of float32, and every norm is widened by 0.1 % and a little more for its own rounding.
// What the floating point sum of the exact path can be off by is added: 2^-15 |q| |k|, several times what
// 128 additions in float32 can lose (and what r, r' and the differences here do: |a m| <= |q|); 2^-19 |a m| |k|
// for the rounding of <m, k> (thirteen operations deep); and, should the matrix cores take denormal numbers
// for zero, 2^-126 sqrt(128) (|q| + |k|) for the inputs and 256 x 2^-126 for products and partial sums. So a key
// whose score could reach a query's threshold tau has <y, x> >= (tau - a <m, k> - bound) / s: one integer per
// query and segment, compared with the largest of a lane's 16 accumulators. Where that does not hold nothing is ruled out
// (an infinite bound: the integer is the smallest there is): non-finite inputs, norms whose product could
// overflow a score (10^38), and s below 2^-100, where the quotients above would round in the denormal range.
// (a is zero where <m, m> or the first term could leave that range.)
//
// Most keys take a part of the product. The dimensions go through the matrix cores in the order of
// what they carry (c_d^2 times the variance of the queries there, kf_rank_kernel), 32 at a time, and <y, x> is
// at most the sum over the dimensions done plus |y'| |x'| over the rest. A block of 32 keys that this
// rules out after 32 or 64 dimensions is done. Whether a wavefront looks that early is decided by how the
// first blocks of its last segments fared, which are looked at after 32, 64 and all 128 dimensions; the
// instructions a look takes (8 per 16 scores) are as long as a step of the product, so a look that mostly fails
// is not worth taking.
//
// What it buys: the copy is half as many bytes and twice the multiply rate, and a wavefront holds
// the 8-bit queries of four sets of 32 in the registers that one set of bf16 queries took, so a key
// operand read from LDS feeds four chains.
#include "common.h"

typedef unsigned long long u64;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x16 __attribute__((ext_vector_type(16)));

#define KF_WAVES 8
#define KF_THREADS (KF_WAVES * RA_WAVE)
#define KF_SEG KN_FILTER_SEGMENT   // keys that share one bound
#define KF_SEG_BLOCKS (KF_SEG / 32)
#define KF_OPERAND (RA_WAVE * 16)  // bytes of one step's operand of 32 keys
#define KF_RING 8                  // operands a wavefront has in LDS or on their way there
#define KF_RUN 3                   // scored keys a lane can hold for its query's list
#define KF_RUNS (2 * KF_RUN)       // ... and the two lanes of a query together
#define KF_PENDING 64              // keys a query set can have waiting to be scored (a batch is 32; a block may add to 31)
#define KF_MEET 4                  // segments between two meetings of a workgroup's wavefronts
#define KF_HOLD 16                 // segments at most between two trials of an earlier look
#define KF_LINE_FIRST(dt) ((dt) == RA_BF16 ? 3 : 8)      // keys of 32 kept above which a workgroup gives up, in the first launch
#define KF_LINE_LAST 12                                  // ... and in a second
#define KF_RANK_SAMPLE 512         // queries whose variance ranks the dimensions (at most)

template <int V> struct kf_int { static constexpr int value = V; };      // a compile-time number as an argument

// memory that one lane of a wavefront wrote and another reads: the hardware keeps the wavefront's order,
// this keeps the compiler's
__device__ __forceinline__ void kf_wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// ---- column maxima of |k| per KV head (bits of a non-negative float order like the float; NaN and
//      infinity come out above every finite value) ------------------------------------------------
template <int DT>
__device__ __forceinline__ void kf_row8(const void* K, size_t at, float (&v)[8]) {
    if constexpr (DT == RA_BF16) {
        const uint4 u = *reinterpret_cast<const uint4*>(reinterpret_cast<const uint16_t*>(K) + at);
        v[0] = bf16_lo(u.x); v[1] = bf16_hi(u.x); v[2] = bf16_lo(u.y); v[3] = bf16_hi(u.y);
        v[4] = bf16_lo(u.z); v[5] = bf16_hi(u.z); v[6] = bf16_lo(u.w); v[7] = bf16_hi(u.w);
    } else {
        const float4 a = *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(K) + at);
        const float4 b = *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(K) + at + 4);
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
    }
}

// grid (blocks, KV heads); 16 lanes per row, 16 rows per pass of a workgroup
__global__ __launch_bounds__(256) void kf_zero_kernel(uint32_t* p, int n) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = 0u;
}
template <int DT>
__global__ __launch_bounds__(256) void kf_maxabs_kernel(const void* __restrict__ K, int64_t N,
                                                        uint32_t* __restrict__ maxabs) {
    __shared__ uint32_t m[RA_D];
    const int tid = threadIdx.x, l16 = tid & 15;
    const size_t base = (size_t)blockIdx.y * N;
    if (tid < RA_D) m[tid] = 0u;
    __syncthreads();
    uint32_t mx[8] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};
    for (int64_t r = (int64_t)blockIdx.x * 16 + tid / 16; r < N; r += (int64_t)gridDim.x * 16) {
        float v[8];
        kf_row8<DT>(K, (base + r) * RA_D + 8 * l16, v);
#pragma unroll
        for (int c = 0; c < 8; ++c) mx[c] = max(mx[c], __float_as_uint(v[c]) & 0x7fffffffu);
    }
#pragma unroll
    for (int c = 0; c < 8; ++c) atomicMax(&m[8 * l16 + c], mx[c]);
    __syncthreads();
    if (tid < RA_D) atomicMax(&maxabs[(size_t)blockIdx.y * RA_D + tid], m[tid]);
}

// sum and maximum over the 16 lanes of a row
__device__ __forceinline__ float kf_sum16(float x, int lane) {
    x += __uint_as_float(lane_xor32<1>(__float_as_uint(x), lane));
    x += __uint_as_float(lane_xor32<2>(__float_as_uint(x), lane));
    x += __uint_as_float(lane_xor32<4>(__float_as_uint(x), lane));
    return x + __uint_as_float(lane_xor32<8>(__float_as_uint(x), lane));
}
__device__ __forceinline__ uint32_t kf_max16(uint32_t x, int lane) {
    x = max(x, lane_xor32<1>(x, lane));
    x = max(x, lane_xor32<2>(x, lane));
    x = max(x, lane_xor32<4>(x, lane));
    return max(x, lane_xor32<8>(x, lane));
}

__device__ __forceinline__ float kf_scale(uint32_t maxabs_bits) {
    return maxabs_bits == 0u ? 1.f : __uint_as_float(maxabs_bits) * (1.0f / 127.0f);
}
// Exponent of the largest |k| of a head, from its column maxima (16 lanes hold 8 of them each). Norms of keys
// are taken over k 2^-exponent: their squares neither overflow nor, for the largest of them, vanish.
__device__ __forceinline__ int kf_exponent(const uint32_t (&maxabs_bits)[8]) {
    uint32_t top = 0u;
#pragma unroll
    for (int c = 0; c < 8; ++c) top = max(top, maxabs_bits[c]);
    top = kf_max16(top, threadIdx.x % RA_WAVE);
    return __builtin_amdgcn_frexp_expf(__uint_as_float(top));       // (0 for zero, infinity and NaN)
}

// ---- the order of the dimensions ------------------------------------------------------------------
// A dimension of rank t (0: the one that carries most) has its byte at 64 ((t / 16) % 2) + 16 (t / 32) + t % 16 of a
// row: the 16-byte chunks t and t + 4 are what the two halves of a wavefront take in step t of the product.
// Any order gives the same lists.
__device__ __forceinline__ int kf_step_of(int byte) { return (byte >> 4) & 3; }

// grid: graph; 16 lanes per query, 64 queries at a time
template <int DT>
__global__ __launch_bounds__(1024) void kf_rank_kernel(const void* __restrict__ Q, const float* __restrict__ mq,
                                                       int mq_samples, const uint32_t* __restrict__ maxabs, int g0,
                                                       int n_q, int n_kv, int64_t M, unsigned char* __restrict__ place) {
    __shared__ float s_part[64][RA_D];
    __shared__ float s_carry[RA_D];
    const int gl = blockIdx.x, graph = g0 + gl, seq = graph / n_q, h = graph % n_q, kvh = h / (n_q / n_kv);
    const int tid = threadIdx.x, l16 = tid & 15, grp = tid / 16;
    const int n_s = M < KF_RANK_SAMPLE ? (int)M : KF_RANK_SAMPLE;
    float mean[8], acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < 8; ++c) mean[c] = mq[(size_t)graph * RA_D + 8 * l16 + c] / (float)mq_samples;
    for (int k = grp; k < n_s; k += 64) {
        float v[8];
        kf_row8<DT>(Q, ((size_t)graph * M + (int64_t)k * M / n_s) * RA_D + 8 * l16, v);
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[c] += (v[c] - mean[c]) * (v[c] - mean[c]);
    }
#pragma unroll
    for (int c = 0; c < 8; ++c) s_part[grp][8 * l16 + c] = acc[c];
    __syncthreads();
    if (tid < RA_D) {
        float t = 0.f;
        for (int i = 0; i < 64; ++i) t += s_part[i][tid];
        const float c = kf_scale(maxabs[((size_t)seq * n_kv + kvh) * RA_D + tid]);
        t = sqrtf(t) * c;
        s_carry[tid] = t < INFINITY ? t : 0.f;           // (also NaN)
    }
    __syncthreads();
    if (tid < RA_D) {
        const float mine = s_carry[tid];
        int t = 0;
        for (int d = 0; d < RA_D; ++d) t += s_carry[d] > mine || (s_carry[d] == mine && d < tid) ? 1 : 0;
        place[(size_t)gl * RA_D + tid] = (unsigned char)(64 * ((t >> 4) & 1) + 16 * (t >> 5) + (t & 15));
    }
}

// ---- the 8-bit copy of a head's keys in stream order ----------------------------------------------
// The keys are stored as operands, in stream order after the first part: per graph and step of the product, for
// each 32 keys the 16 bytes of lane 0, of lane 1 and so on (row lane % 32, chunk step + 4 (lane / 32) of it), a
// linear kilobyte for a wavefront to load. Rows beyond the stream are zero. seg[graph][segment]: what the
// bound takes from the segment's keys. k_top[graph]: bits of the largest |k 2^-kf_exponent|^2 of the graph's keys.
struct KfSegment {
    float x, e;            // largest |x| and |e|
    float b_max, b_min;    // <m, k> of the first and the last key
    float x1, x2, x3;      // largest |x| over the dimensions of steps 1, 2 and 3 of the product
    float pad;
};
// grid (segments, graphs); 16 lanes per row
template <int DT>
__global__ __launch_bounds__(1024) void kf_pack_kernel(const void* __restrict__ K, const u64* __restrict__ order,
                                                       int64_t order_stride, const uint32_t* __restrict__ maxabs,
                                                       const unsigned char* __restrict__ place, int g0, int n_q,
                                                       int n_kv, int64_t N, int64_t first, int64_t rows8, int nseg,
                                                       uint2* __restrict__ K8, KfSegment* __restrict__ seg,
                                                       uint32_t* __restrict__ k_top) {
    __shared__ uint32_t s_top[6];
    __shared__ float s_b[2];
    __shared__ __align__(16) unsigned char s_row[64][RA_D];
    const int gl = blockIdx.y, graph = g0 + gl, seq = graph / n_q, h = graph % n_q, kvh = h / (n_q / n_kv);
    const int tid = threadIdx.x, l16 = tid & 15;
    const size_t kv = (size_t)seq * n_kv + kvh;
    float sc[8], inv[8];
    uint32_t mx[8];
    int at[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        mx[c] = maxabs[kv * RA_D + 8 * l16 + c];
        sc[c] = kf_scale(mx[c]);
        inv[c] = 1.0f / sc[c];
        at[c] = place[(size_t)gl * RA_D + 8 * l16 + c];
    }
    const int k_exp = kf_exponent(mx);
    const u64* ord = order + (size_t)graph * order_stride;
    for (int sg = blockIdx.x; sg < nseg; sg += gridDim.x) {
        if (tid < 6) s_top[tid] = 0u;
        __syncthreads();
        uint32_t top[6] = {0u, 0u, 0u, 0u, 0u, 0u};      // of the rows of these 16 lanes: |e|^2, |x|^2, |k|^2, |x|^2 by step
        for (int64_t p = (int64_t)sg * KF_SEG + tid / 16; p < (int64_t)(sg + 1) * KF_SEG; p += 64) {
            uint2 w = make_uint2(0u, 0u);
            if (first + p < N) {
                const u64 entry = ord[first + p];
                float v[8], sum[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                kf_row8<DT>(K, (kv * N + (int64_t)(uint32_t)entry) * RA_D + 8 * l16, v);
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    float x = rintf(v[c] * inv[c]);
                    x = fminf(fmaxf(x, -127.f), 127.f);
                    const float e = __fmaf_rn(-x, sc[c], v[c]) * inv[c];
                    const float k = __builtin_amdgcn_ldexpf(v[c], -k_exp);
                    sum[0] += e * e;
                    sum[1] += x * x;
                    sum[2] += k * k;
#pragma unroll
                    for (int t = 0; t < 3; ++t) sum[3 + t] += kf_step_of(at[c]) == t + 1 ? x * x : 0.f;
                    s_row[tid / 16][at[c]] = (unsigned char)((uint32_t)(int)x & 255u);
                }
                if (l16 == 0) {
                    const float b = f32_from_ordered(~(uint32_t)(entry >> 32));
                    if (p == (int64_t)sg * KF_SEG) s_b[0] = b;
                    if (p == (int64_t)(sg + 1) * KF_SEG - 1 || first + p == N - 1) s_b[1] = b;
                }
                // a NaN (from non-finite keys) has the largest bits of all
#pragma unroll
                for (int t = 0; t < 6; ++t) top[t] = max(top[t], __float_as_uint(kf_sum16(sum[t], tid % RA_WAVE)) & 0x7fffffffu);
                kf_wave_sync();                          // (a row is a wavefront's own)
                w = *reinterpret_cast<const uint2*>(&s_row[tid / 16][8 * l16]);
                kf_wave_sync();
            }
            if (p < rows8)
                K8[((size_t)gl * 4 + ((l16 >> 1) & 3)) * rows8 * 4 + (p >> 5) * 128 + ((int)(p & 31) + 32 * (l16 >> 3)) * 2 +
                   (l16 & 1)] = w;
        }
        if (l16 == 0)
#pragma unroll
            for (int t = 0; t < 6; ++t) atomicMax(&s_top[t], top[t]);
        __syncthreads();
        if (tid == 0) {
            // (finite whatever the keys are: where one is not, every query's bound is infinite, and nothing
            // may turn that into a NaN)
            auto finite = [](float x, float top) { return x < top ? x : x >= top ? top : 0.f; };
            KfSegment g;
            g.x = finite(1.001f * sqrtf(__uint_as_float(s_top[1])), 1e6f);
            g.e = finite(1.001f * sqrtf(__uint_as_float(s_top[0])) + 1e-3f, 1e6f);
            g.x1 = finite(1.001f * sqrtf(__uint_as_float(s_top[3])), 1e6f);
            g.x2 = finite(1.001f * sqrtf(__uint_as_float(s_top[4])), 1e6f);
            g.x3 = finite(1.001f * sqrtf(__uint_as_float(s_top[5])), 1e6f);
            g.b_max = fmaxf(finite(s_b[0], 1e37f), -1e37f);
            g.b_min = fmaxf(finite(s_b[1], 1e37f), -1e37f);
            g.pad = 0.f;
            seg[(size_t)gl * nseg + sg] = g;
            atomicMax(&k_top[gl], s_top[2]);
        }
        __syncthreads();
    }
}

// ---- scoring, as in knn.hip ---------------------------------------------------------------------------
// Operand of lane (row = lane % 32, half = lane / 32): dimensions [64 half, 64 half + 64) of the row;
// the same instructions in the same order as the first part of the stream.
template <int DT>
__device__ __forceinline__ f32x16 kf_scores(const void* K, size_t krow, const void* Q, size_t qrow, int half) {
    f32x16 c = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if constexpr (DT == RA_BF16) {
        const uint4* a = reinterpret_cast<const uint4*>(reinterpret_cast<const uint16_t*>(K) + krow * RA_D + 64 * half);
        const uint4* b = reinterpret_cast<const uint4*>(reinterpret_cast<const uint16_t*>(Q) + qrow * RA_D + 64 * half);
#pragma unroll
        for (int s0 = 0; s0 < 8; s0 += 4) {
            uint4 av[4], bv[4];
#pragma unroll
            for (int s = 0; s < 4; ++s) { av[s] = a[s0 + s]; bv[s] = b[s0 + s]; }
#pragma unroll
            for (int s = 0; s < 4; ++s)
                c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av[s]),
                                                            __builtin_bit_cast(bf16x8, bv[s]), c, 0, 0, 0);
        }
    } else {
        const float4* a = reinterpret_cast<const float4*>(reinterpret_cast<const float*>(K) + krow * RA_D + 64 * half);
        const float4* b = reinterpret_cast<const float4*>(reinterpret_cast<const float*>(Q) + qrow * RA_D + 64 * half);
#pragma unroll
        for (int s0 = 0; s0 < 16; s0 += 4) {
            float4 av[4], bv[4];
#pragma unroll
            for (int s = 0; s < 4; ++s) { av[s] = a[s0 + s]; bv[s] = b[s0 + s]; }
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                c = __builtin_amdgcn_mfma_f32_32x32x2f32(av[s].x, bv[s].x, c, 0, 0, 0);
                c = __builtin_amdgcn_mfma_f32_32x32x2f32(av[s].y, bv[s].y, c, 0, 0, 0);
                c = __builtin_amdgcn_mfma_f32_32x32x2f32(av[s].z, bv[s].z, c, 0, 0, 0);
                c = __builtin_amdgcn_mfma_f32_32x32x2f32(av[s].w, bv[s].w, c, 0, 0, 0);
            }
        }
    }
    return c;
}

__device__ __forceinline__ u64 kf_key(float score, int id) {
    return ((u64)f32_ordered(score) << 32) | (u64)(0xffffffffu - (uint32_t)id);
}
__device__ __forceinline__ u64 kf_readlane64(u64 x, int l) {
    return ((u64)(uint32_t)__builtin_amdgcn_readlane((int)(x >> 32), l) << 32) |
           (u64)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, l);
}

// Merge up to KF_RUNS new keys (lane k < KF_RUNS holds the k-th, zero for none) into a query's sorted
// list in device memory, whose entries the lanes below knn hold (v, zero for none). A list entry moves
// down by the number of new keys above it, a new key lands at the number of keys above it; what leaves
// the list is not written. Returns the new threshold. All 64 lanes cooperate; only this wavefront
// touches the list.
__device__ __forceinline__ float kf_fold(float* sc, int32_t* id, int knn, u64 v, u64 fresh, int lane) {
    int pos = lane, fpos = 0;
#pragma unroll
    for (int k = 0; k < KF_RUNS; ++k) {
        const u64 x = kf_readlane64(fresh, k);
        const int above = __popcll(__ballot(lane < knn && v > x));
        if (v < x) ++pos;
        if (lane == k) fpos += above;
        if (fresh < x) ++fpos;
    }
    const bool old = lane < knn && v != 0ull && pos < knn;
    if (old && pos != lane) {
        sc[pos] = f32_from_ordered((uint32_t)(v >> 32));
        id[pos] = (int)(0xffffffffu - (uint32_t)v);
    }
    const bool in = lane < KF_RUNS && fresh != 0ull && fpos < knn;
    if (in) {
        sc[fpos] = f32_from_ordered((uint32_t)(fresh >> 32));
        id[fpos] = (int)(0xffffffffu - (uint32_t)fresh);
    }
    const u64 old_end = __ballot(old && pos == knn - 1), new_end = __ballot(in && fpos == knn - 1);
    kf_wave_sync();
    if (new_end)
        return f32_from_ordered((uint32_t)__builtin_amdgcn_readlane((int)(fresh >> 32), __ffsll((long long)new_end) - 1));
    if (old_end)
        return f32_from_ordered((uint32_t)__builtin_amdgcn_readlane((int)(v >> 32), __ffsll((long long)old_end) - 1));
    return -INFINITY;
}

// smallest integer product that x leaves possible (no product is below -128 x 127^2: -10^9, also for NaN, rules out nothing)
__device__ __forceinline__ int kf_floor(float x) { return (int)floorf(fminf(fmaxf(x, -1.0e9f), 1.0e9f)) - 2; }

// What the filter keeps of a query. A threshold tau asks for <y, x> of at least
// (tau - slack - a b - f x - r e) * inv from a segment, b, x and e its own.
struct KfQuery {
    float a, f, r, inv;            // a; s |f|; |r'|; 1 / s
    float y1, y2, y3;              // |y| over the dimensions of steps 1, 2 and 3 of the product
    float tau, slack, pad[3];      // slack: the rest of the bound
};
#define KF_QUERY16 (sizeof(KfQuery) / 16)

// ---- the queries in 8 bits: y (128 bytes per query, dimensions in the order of `place`), and KfQuery
// grid (rows / 16, graphs); 16 lanes per row
template <int DT>
__global__ __launch_bounds__(256) void kf_queries_kernel(const void* __restrict__ Q, const float* __restrict__ mq,
                                                         const uint32_t* __restrict__ maxabs,
                                                         const unsigned char* __restrict__ place,
                                                         const uint32_t* __restrict__ k_top, int g0, int n_q,
                                                         int n_kv, int64_t M, int knn,
                                                         const float* __restrict__ scores, uint2* __restrict__ Q8,
                                                         float4* __restrict__ qinfo, int* __restrict__ resume, int waves,
                                                         int wave_queries) {
    __shared__ __align__(16) unsigned char s_row[16][RA_D];
    const int gl = blockIdx.y, graph = g0 + gl, seq = graph / n_q, h = graph % n_q, kvh = h / (n_q / n_kv);
    const int tid = threadIdx.x, l16 = tid & 15;
    const size_t kv = (size_t)seq * n_kv + kvh;
    // where the wavefronts of knn_filter_kernel begin: at the front, or, those without a query, at the end
    for (int i = blockIdx.x * 256 + tid; i < waves; i += gridDim.x * 256)
        resume[(size_t)gl * waves + i] = (int64_t)i * wave_queries < M ? 0 : 0x7fffffff;
    float sc[8], m[8], mm = 0.f;
    uint32_t mx[8];
    int at[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        mx[c] = maxabs[kv * RA_D + 8 * l16 + c];
        sc[c] = kf_scale(mx[c]);
        m[c] = mq[(size_t)graph * RA_D + 8 * l16 + c];
        at[c] = place[(size_t)gl * RA_D + 8 * l16 + c];
        mm += m[c] * m[c];
    }
    const int lane = tid % RA_WAVE;
    mm = kf_sum16(mm, lane);
    const float k_max = __builtin_amdgcn_ldexpf(1.001f * sqrtf(__uint_as_float(k_top[gl])), kf_exponent(mx));
    const float m_norm = 1.001f * sqrtf(mm);
    const bool mean = mm >= 1e-30f && mm <= 1e30f && m_norm * k_max < 1e36f;
    const int64_t rounds = (M + (int64_t)gridDim.x * 16 - 1) / ((int64_t)gridDim.x * 16);
    for (int64_t i = 0; i < rounds; ++i) {
        const int64_t row = (i * gridDim.x + blockIdx.x) * 16 + tid / 16, j = row < M ? row : M - 1;
        float v[8], p[8], top = 0.f, q_top = 0.f, qm = 0.f;
        kf_row8<DT>(Q, ((size_t)graph * M + j) * RA_D + 8 * l16, v);
#pragma unroll
        for (int c = 0; c < 8; ++c) qm += v[c] * m[c];
        qm = kf_sum16(qm, lane);
        float a = mean ? qm / mm : 0.f;
        if (!(fabsf(a) < 1e30f)) a = 0.f;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            p[c] = (a == 0.f ? v[c] : __fmaf_rn(-a, m[c], v[c])) * sc[c];
            top = fmaxf(top, fabsf(p[c]));
            q_top = fmaxf(q_top, fabsf(v[c]));
        }
        top = __uint_as_float(kf_max16(__float_as_uint(top), lane));          // (not negative: the bits order like the numbers)
        q_top = __uint_as_float(kf_max16(__float_as_uint(q_top), lane));
        const float s = top > 0.f ? top * (1.0f / 127.0f) : 1.f, inv = 1.0f / s;
        const int q_exp = __builtin_amdgcn_frexp_expf(q_top);
        float f2 = 0.f, n2 = 0.f, q2 = 0.f, ys[3] = {0.f, 0.f, 0.f};      // |f|^2, |r' / s|^2, |q 2^-q_exp|^2, parts of |y|^2
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const float r = p[c] * inv;
            float y = rintf(r);
            y = fminf(fmaxf(y, -127.f), 127.f);
            const float f = __fmaf_rn(-y, s, p[c]) * inv;
            const float q = __builtin_amdgcn_ldexpf(v[c], -q_exp);
            f2 += f * f;
            n2 += r * r;
            q2 += q * q;
#pragma unroll
            for (int t = 0; t < 3; ++t) ys[t] += kf_step_of(at[c]) == t + 1 ? y * y : 0.f;
            s_row[tid / 16][at[c]] = (unsigned char)((uint32_t)(int)y & 255u);
        }
        f2 = kf_sum16(f2, lane);
        n2 = kf_sum16(n2, lane);
        q2 = kf_sum16(q2, lane);
#pragma unroll
        for (int t = 0; t < 3; ++t) ys[t] = kf_sum16(ys[t], lane);
        kf_wave_sync();                                  // (a row is a wavefront's own)
        if (row < M) {
            Q8[((size_t)gl * M + j) * 16 + l16] = *reinterpret_cast<const uint2*>(&s_row[tid / 16][8 * l16]);
            if (l16 == 0) {
                const float q_norm = __builtin_amdgcn_ldexpf(1.001f * sqrtf(q2), q_exp), norms = q_norm * k_max;
                float slack = 3.1e-5f * norms + 2e-6f * fabsf(a) * m_norm * k_max + 1.4e-37f * (q_norm + k_max) + 1e-35f;
                float f = 1.002f * s * (1.001f * sqrtf(f2) + 1e-3f), r = 1.002f * s * (1.001f * sqrtf(n2));
                if (!(s >= 0x1p-100f && norms < 1e38f && slack < INFINITY && f < INFINITY && r < INFINITY)) {
                    slack = INFINITY;
                    a = f = r = 0.f;
                }
                float4* out = qinfo + KF_QUERY16 * ((size_t)gl * M + j);
                out[0] = make_float4(a, f, r, inv);
                out[1] = make_float4(1.001f * sqrtf(ys[0]), 1.001f * sqrtf(ys[1]), 1.001f * sqrtf(ys[2]),
                                     scores[((size_t)gl * M + j) * knn + knn - 1]);
                out[2] = make_float4(slack, 0.f, 0.f, 0.f);
            }
        }
        kf_wave_sync();
    }
}

// grid: x = block of KF_WAVES * NQ * 32 queries, y = graph of the launch. A wavefront owns NQ sets
// of 32 queries. What only the rare path needs (a query's bound, scale and threshold, the waiting keys)
// sits in LDS; a lane keeps its queries' 8-bit operands and integer floors.
template <int DT, int NQ>
__global__ __launch_bounds__(KF_THREADS, 2) void knn_filter_kernel(
    const void* __restrict__ K, const void* __restrict__ Q, const u64* __restrict__ order, int64_t order_stride,
    const unsigned char* __restrict__ K8, int64_t rows8, const unsigned char* __restrict__ Q8,
    const float4* __restrict__ qinfo, const KfSegment* __restrict__ seg, int nseg, int g0, int n_q, int n_kv, int64_t N,
    int64_t M, int knn, int first, int from, int end, int line, float* scores, int32_t* L, int* resume) {
    __shared__ int s_pend[KF_WAVES][NQ][KF_PENDING];
    __shared__ int s_count[KF_WAVES][NQ];
    __shared__ u64 s_run[KF_WAVES][NQ][KF_RUN][RA_WAVE];
    __shared__ unsigned char s_fill[KF_WAVES][NQ][RA_WAVE];
    // What is copied to LDS has to lie in its first 64 KB (16 bits of m0). The compiler lays a kernel's arrays out by alignment, the
    // largest first: no other may ask for as much. (In one struct with the rings first, or looked at when the kernel starts, the
    // rare path's registers go to memory and 1M keys x 4 heads take 1.5 to 2 % longer.)
    static_assert(KF_WAVES * KF_RING * KF_OPERAND <= 1 << 16, "the rings fit the first 64 KB of LDS");
    __shared__ __align__(1024) unsigned char s_ring[KF_WAVES][KF_RING * KF_OPERAND];
    __shared__ __align__(16) float4 s_query[KF_WAVES][NQ][2][32];      // of KfQuery: [a, f, r, inv], [y1, y2, y3, tau]
    __shared__ float s_slack[KF_WAVES][NQ][32];
    __shared__ int s_kept, s_seen;                     // of the workgroup's sets: keys not ruled out, blocks looked at
    const int tid = threadIdx.x, wv = tid / RA_WAVE, lane = tid % RA_WAVE;
    const int col = lane & 31, half = lane >> 5;
    const int gl = blockIdx.y, graph = g0 + gl, seq = graph / n_q, h = graph % n_q, kvh = h / (n_q / n_kv);
    const size_t esz = DT == RA_BF16 ? 2 : 4;
    const char* Kh = reinterpret_cast<const char*>(K) + ((size_t)seq * n_kv + kvh) * N * RA_D * esz;
    const char* Qh = reinterpret_cast<const char*>(Q) + (size_t)graph * M * RA_D * esz;
    const int64_t q0 = (int64_t)blockIdx.x * (KF_WAVES * NQ * 32) + wv * NQ * 32;
    const int* ord = reinterpret_cast<const int*>(order + (size_t)graph * order_stride);
    float* sc_g = scores + (size_t)gl * M * knn;
    int32_t* L_g = L + (size_t)graph * M * knn;

    // the stream position this wavefront goes on from: `from`, or where it gave up behind that (knn.hip has
    // multiplied what lies between); nothing is left where it came to the end in a launch before, or has no query
    int* my_resume = resume + ((size_t)gl * gridDim.x + blockIdx.x) * KF_WAVES + wv;
    int begin = __builtin_amdgcn_readfirstlane(*my_resume);
    if (begin < from) begin = from;
    if (begin >= end) begin = -1;
    if (tid == 0) s_kept = s_seen = 0;
    __syncthreads();
    if (begin < 0) return;                             // (a barrier waits for no wavefront that has ended)
    i32x4 b[NQ][4];
#pragma unroll
    for (int s = 0; s < NQ; ++s) {
        int64_t qr = q0 + 32 * s + col;
        if (qr >= M) qr = M - 1;                       // such columns are never written
        const i32x4* src = reinterpret_cast<const i32x4*>(Q8 + ((size_t)gl * M + qr) * RA_D + 64 * half);
#pragma unroll
        for (int c = 0; c < 4; ++c) b[s][c] = src[c];
        float4 qi = qinfo[KF_QUERY16 * ((size_t)gl * M + qr) + half];
        if (half == 1) qi.w = sc_g[(size_t)qr * knn + knn - 1];        // the threshold as it is now
        s_query[wv][s][half][col] = qi;
        if (half == 0) s_slack[wv][s][col] = qinfo[KF_QUERY16 * ((size_t)gl * M + qr) + 2].x;
        s_count[wv][s] = 0;
        s_fill[wv][s][lane] = 0;
        // (complete here: a load that the compiler took for outstanding in the loop would be waited for there,
        // and with it the operands on their way to LDS, which it does not count)
        asm volatile("; queries loaded" ::"v"(b[s][0]), "v"(b[s][1]), "v"(b[s][2]), "v"(b[s][3]));
    }
    // (A column without a query keeps no key: its threshold is infinity. With the last query's and no way to raise it, such columns,
    // and wavefronts without a query, kept ever more keys and made their workgroup give up: 4 heads of the mixture law, 256K
    // keys x 65537 queries 20.7 ms, now 19.7, 1M x 16385 29.7 and 29.2, float32 64K x 8193 4.25 and 3.91.)
    if (q0 + 32 * NQ > M)
        for (int s = 0; s < NQ; ++s)
            if (half == 1 && q0 + 32 * s + col >= M) s_query[wv][s][1][col].w = INFINITY;
    kf_wave_sync();
    int kept = 0;                                      // keys that were not ruled out

    // the waiting scored keys of the queries in `mask` of set s go into their lists (the next query's
    // list is on its way while one is merged)
    auto fold = [&](int s, uint32_t mask, float& tau, int& fill) __attribute__((always_inline)) {
        if (!mask) return;
        auto list_of = [&](int jq, u64& v) __attribute__((always_inline)) {
            const size_t at = (size_t)(q0 + 32 * s + jq) * knn;
            const float sc = sc_g[at + (lane < knn ? lane : 0)];
            const int id = L_g[at + (lane < knn ? lane : 0)];
            v = lane < knn && sc > -INFINITY ? kf_key(sc, id) : 0ull;
        };
        int jq = __ffs((int)mask) - 1;
        u64 v, nv;
        list_of(jq, v);
        while (true) {
            mask &= mask - 1;
            const int jn = mask ? __ffs((int)mask) - 1 : jq;
            if (mask) list_of(jn, nv);
            const int f_lo = __builtin_amdgcn_readlane(fill, jq), f_hi = __builtin_amdgcn_readlane(fill, jq + 32);
            u64 fresh = 0ull;
            if (lane < f_lo) fresh = s_run[wv][s][lane][jq];
            if (lane >= KF_RUN && lane - KF_RUN < f_hi) fresh = s_run[wv][s][lane - KF_RUN][jq + 32];
            const size_t at = (size_t)(q0 + 32 * s + jq) * knn;
            const float nt = kf_fold(sc_g + at, L_g + at, knn, v, fresh, lane);
            if (col == jq) { tau = nt; fill = 0; }
            if (!mask) break;
            jq = jn;
            v = nv;
        }
    };
    // exact scores of n waiting keys of set s, from place `at` on; those that reach a threshold join their
    // query's run
    auto score_pending = [&](int s, int at, int n) __attribute__((always_inline)) {
        const int p = s_pend[wv][s][at + (col < n ? col : 0)];
        const int id = ord[2 * (size_t)(unsigned)p];
        int64_t qr = q0 + 32 * s + col;
        const bool mine = qr < M;
        if (!mine) qr = M - 1;
        float tau = s_query[wv][s][1][col].w;
        int fill = s_fill[wv][s][lane];
        const f32x16 c = kf_scores<DT>(Kh, (size_t)id, Qh, (size_t)qr, half);
        uint32_t some = 0u;                            // rows of which a score reaches its threshold
#pragma unroll
        for (int r = 0; r < 16; ++r)
            if (__ballot(c[r] >= tau) != 0ull) some |= 1u << r;
        while (some) {
            const int r = __ffs((int)some) - 1;
            some &= some - 1;
            const int row = (r / 4) * 8 + half * 4 + (r % 4);
            const float sc = c[r];
            const bool ok = mine && row < n && sc > -INFINITY;
            const u64 full = __ballot(ok && sc >= tau && fill == KF_RUN);
            if (full) fold(s, (uint32_t)full | (uint32_t)(full >> 32), tau, fill);
            const int lo = __builtin_amdgcn_readlane(id, (r / 4) * 8 + (r % 4));
            const int hi = __builtin_amdgcn_readlane(id, (r / 4) * 8 + 4 + (r % 4));
            if (ok && sc >= tau) s_run[wv][s][fill++][lane] = kf_key(sc, half ? hi : lo);
            kf_wave_sync();
        }
        kf_wave_sync();
        s_query[wv][s][1][col].w = tau;
        s_fill[wv][s][lane] = (unsigned char)fill;
    };
    // the keys of block `pos` (stream position of its first row) that set s cannot rule out join its
    // waiting keys; true when a full batch waits
    auto keep = [&](int s, const i32x16& c, int floor_s, int pos) __attribute__((always_inline)) -> bool {
        uint32_t rows = 0u;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int gm = max(max(c[4 * g], c[4 * g + 1]), max(c[4 * g + 2], c[4 * g + 3]));
            if (__ballot(gm >= floor_s) == 0ull) continue;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const u64 m = __ballot(c[4 * g + r] >= floor_s);
                if ((uint32_t)m) rows |= 1u << (8 * g + r);
                if ((uint32_t)(m >> 32)) rows |= 1u << (8 * g + 4 + r);
            }
        }
        if (pos + 32 > N) rows &= N > pos ? (1u << (int)(N - pos)) - 1u : 0u;
        rows = __builtin_amdgcn_readfirstlane(rows);
        const int have = __builtin_amdgcn_readfirstlane(s_count[wv][s]);
        if (lane < 32 && ((rows >> lane) & 1u))
            s_pend[wv][s][have + __popc(rows & ((1u << lane) - 1u))] = pos + lane;
        s_count[wv][s] = have + __popc(rows);
        kept += __popc(rows);
        return have + __popc(rows) >= 32;
    };
    // what a segment's keys need so that their scores can reach the thresholds: the whole product, and its
    // first 32 and 64 dimensions
    const float4* seg_g = reinterpret_cast<const float4*>(seg + (size_t)gl * nseg);
    float sg_x = 0.f, sg_e = 0.f, sg_b_max = 0.f, sg_b_min = 0.f, sg_x1 = 0.f, sg_x2 = 0.f, sg_x3 = 0.f;
    int floor_[NQ], floor1[NQ], floor2[NQ];
    // (false where no product of the segment can reach any threshold: |y| |x| is below them all; |y| <= |r'| / s + |f|)
    auto set_floors = [&]() __attribute__((always_inline)) -> bool {
        bool reach = false;
#pragma unroll
        for (int s = 0; s < NQ; ++s) {
            const float4 q0 = s_query[wv][s][0][col], q1 = s_query[wv][s][1][col];
            const float a = q0.x, f = q0.y, r = q0.z, inv = q0.w, tau = q1.w;
            const float x = (tau - s_slack[wv][s][col] - a * (a >= 0.f ? sg_b_max : sg_b_min) - f * sg_x - r * sg_e) * inv;
            const float rest2 = 1.001f * (q1.y * sg_x2 + q1.z * sg_x3);
            floor_[s] = kf_floor(x);
            floor1[s] = kf_floor(x - rest2 - 1.001f * (q1.x * sg_x1));
            floor2[s] = kf_floor(x - rest2);
            reach = reach || kf_floor(x - (r + f) * inv * sg_x) <= 0;
        }
        return __ballot(reach) != 0ull;
    };
    // sets with a full batch waiting (or, at the end, any key) are scored; their floors follow
    auto score_full = [&](bool all) __attribute__((always_inline)) {
        kf_wave_sync();
        for (int s = 0; s < NQ; ++s) {
            int have = __builtin_amdgcn_readfirstlane(s_count[wv][s]);
            while (have >= 32 || (all && have)) {
                const int n = have < 32 ? have : 32;
                have -= n;
                score_pending(s, have, n);
            }
            s_count[wv][s] = have;
        }
        kf_wave_sync();
        (void)set_floors();
    };

    // ---- the stream. Every wavefront copies its operands to a ring of its own in LDS, eight of them ahead, straight
    //      from memory (no register holds them on the way), and waits for the others only where they meet. 128K keys x 32 heads, when it was made: 33 ms;
    //      with stages of 128 keys that the workgroup shares in LDS 34 ms, loads to registers instead of the ring 42 ms.
    //      1M keys x 4 heads, where wavefronts have keys to score at different times: 36, 41 and 35 ms. Before
    //      (stages, whole products, no mean taken off): 51 and 41 ms.
    const unsigned char* K8g = K8 + (size_t)gl * rows8 * RA_D;
    const int nblocks = (end - first + 31) / 32;
    const uint32_t ring_at = __builtin_amdgcn_readfirstlane(
        (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)s_ring + wv * (KF_RING * KF_OPERAND));
    const unsigned char* ring = s_ring[wv];
    const int lane_at = lane * 16;
    auto operand_of = [&](int blk, int c) __attribute__((always_inline)) {       // (past the end: the last block's, unused)
        const unsigned at = __builtin_amdgcn_readfirstlane(blk < nblocks ? blk : nblocks - 1);
        return K8g + (size_t)c * rows8 * 32 + (size_t)at * KF_OPERAND;
    };
    auto fetch = [&](int blk, int c, int slot) __attribute__((always_inline)) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(__builtin_amdgcn_readfirstlane(ring_at + slot * KF_OPERAND)),
                     "v"(lane_at), "s"(operand_of(blk, c)) : "m0", "memory");
    };
    auto operand = [&](int blk, int c) __attribute__((always_inline)) {          // (without the ring: seldom)
        return *reinterpret_cast<const i32x4*>(operand_of(blk, c) + lane_at);
    };
    // The sets of a wavefront go in two halves (one, where there is one set): while the products of one half
    // run, the other half's are looked at, so that neither waits for the other's latency.
    constexpr int H = NQ >= 2 ? 2 : 1, HQ = NQ / H;
    // largest product of a lane's 16 against the floors of half h: whether any set has a key left, and which
    auto left = [&](auto h_c, const i32x16 (&acc)[HQ], const int (&floors)[NQ], bool (&yes)[HQ])
        __attribute__((always_inline)) -> bool {
        constexpr int h = decltype(h_c)::value;
        int m[HQ];
#pragma unroll
        for (int s = 0; s < HQ; ++s) m[s] = max(acc[s][0], acc[s][1]);
#pragma unroll
        for (int r = 2; r < 16; r += 2)
#pragma unroll
            for (int s = 0; s < HQ; ++s) m[s] = max(max(m[s], acc[s][r]), acc[s][r + 1]);
        bool any = false;
#pragma unroll
        for (int s = 0; s < HQ; ++s) {
            yes[s] = m[s] >= floors[h * HQ + s];
            any = any || yes[s];
        }
        return __ballot(any) != 0ull;
    };
    auto products = [&](auto h_c, i32x16 (&acc)[HQ], const i32x4& a, auto c_c) __attribute__((always_inline)) {
        constexpr int h = decltype(h_c)::value, c = decltype(c_c)::value;
        const i32x16 z = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < HQ; ++s)
            acc[s] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b[h * HQ + s][c], c == 0 ? z : acc[s], 0, 0, 0);
    };
    // ---- how early to look. What a look in the lower steps fails to rule out costs the rest of the product and
    //      another look, so a wavefront looks early only while at most two in five of those looks fail, and, where
    //      it does not, tries again every so often (thresholds are the further away the later in the stream).
    // (The wavefront's own scalars; the compiler does not see that they are, through the loops of the rare path.)
    auto uniform = [](int x) __attribute__((always_inline)) { return __builtin_amdgcn_readfirstlane(x); };
    int blk = uniform((begin - first) / 32), look = 4, fails = 0, hold = 1, wait = 1, counted = blk;
    // at the end of a segment: true when the wavefront goes on as it did
    auto same_look = [&]() __attribute__((always_inline)) -> bool {
        const int was = look = uniform(look);
        fails = uniform(fails);
        wait = uniform(wait);
        hold = uniform(hold);
        if (look < 4 && 5 * fails > 2 * H * KF_SEG_BLOCKS) {
            look *= 2;
            wait = hold = min(2 * hold, KF_HOLD);
        } else if (look > 1 && --wait <= 0) {
            look /= 2;
            wait = 1;
            if (look == 1 && was == 2 && fails == 0) hold = 1;
        }
        fails = 0;
        return look == was;
    };
    // Scoring a kept key costs about ten times what ruling it out does. Where the bound cannot tell the keys apart (at the
    // start of a stream whose queries have little in common, or all along: ties, a few dimensions that dwarf the
    // others) they are better off in knn.hip's loop: when a workgroup's wavefronts have kept more than `line` keys in 32, each stops
    // at the end of its segment and leaves its queries' keys up to `end` there. All of them, because that loop costs a workgroup's
    // whole stream however few of its queries are left. The line is three (in float32, whose products cost sixteen times
    // as much, eight) up to an eighth of the stream, or where there is one launch, and twelve behind, where thresholds are near
    // final and giving up means exact products to the end. Whole calls, 4 heads of the mixture law, lists of 48, lines at 1 / 2 / 3 / 4 in 32,
    // ms: 64K keys x 64K queries 7.8 / 7.8 / 8.0 / 9.8, 128K 12.5 / 13.7 / 10.4 / 10.5, 256K 20.0 / 14.9 / 14.8 / 15.0; float32, 64K
    // keys x 8K queries, 4 / 8 / 16 / 24 in 32: 7.7 / 3.2 / 5.6 / 3.4; behind the eighth 3 and 12: 81008 keys x 64K queries 13.1 and 7.5; one launch
    // of 30000 keys x 30000 queries 3 / 8 / 16: 2.2 / 3.1 / 2.6.
    auto keeps_too_much = [&]() __attribute__((always_inline)) -> bool {
        const int seen = (blk - counted) * NQ;           // (blocks of 32 keys)
        int all_kept = 0, all_seen = 0;
        if (lane == 0) {
            all_kept = atomicAdd(&s_kept, kept) + kept;
            all_seen = atomicAdd(&s_seen, seen) + seen;
        }
        kept = 0;
        counted = blk;
        all_kept = uniform(all_kept);
        all_seen = uniform(all_seen);
        return all_seen >= KF_WAVES / 2 * KF_SEG_BLOCKS * NQ && (int64_t)all_kept > (int64_t)all_seen * line;
    };
    // the floors of the segment that opens at block blk; false when none of its keys can reach a threshold
    auto open_segment = [&]() __attribute__((always_inline)) -> bool {
        // The wavefronts meet every 2048 keys, so that they stay in reach of each other's lines in the caches (whole
        // calls, 1M keys x 4 heads of 64K queries: 43.4 -> 40.6 ms, of 16K queries, one set per wavefront: 30.1 -> 17.0; a meeting
        // every 512 keys: 43.3 and 17.9). A barrier waits for no wavefront that has ended. One that comes out of run() because nothing of a
        // segment can reach a threshold opens that segment again, and where that is a meeting, takes its part in the next one, too:
        // with others it is then a meeting ahead. (Opening it once: 128K keys x 32 heads 39.1 -> 39.8 ms, more registers in
        // memory; 1M keys x 4 heads of 64K queries 39.1 -> 39.4, of 16385 29.1 -> 28.8.)
        if ((blk / KF_SEG_BLOCKS) % KF_MEET == 0) __builtin_amdgcn_s_barrier();
        const float4 g0 = seg_g[2 * (blk / KF_SEG_BLOCKS)], g1 = seg_g[2 * (blk / KF_SEG_BLOCKS) + 1];
        sg_x = g0.x; sg_e = g0.y; sg_b_max = g0.z; sg_b_min = g0.w; sg_x1 = g1.x; sg_x2 = g1.y; sg_x3 = g1.z;
        return set_floors();
    };
    // blocks from blk, the first of a segment whose floors are set, until the look changes, nothing of a segment can
    // reach a threshold or the stream ends; E: steps of 32 dimensions before the first look (1, 2 or 4: all of them)
    auto run = [&](auto e_c) __attribute__((always_inline)) {
        constexpr int E = decltype(e_c)::value;
        // an early look that fails goes on with the next step at once: where that may be often, its operand is in the ring
        constexpr int C = E == 1 ? 2 : E;              // operands of a block in the ring
        constexpr int AHEAD = KF_RING / C;             // blocks in the ring
        i32x16 acc[H][HQ];
        i32x4 a[E];
        bool batch = false;                            // some set has 32 keys waiting
        auto from_ring = [&](int at, int c) __attribute__((always_inline)) {
            return *reinterpret_cast<const i32x4*>(ring + ((unsigned)at % AHEAD * C + c) * KF_OPERAND + lane_at);
        };
        auto first_steps = [&](auto h_c) __attribute__((always_inline)) {
            constexpr int h = decltype(h_c)::value;
            products(h_c, acc[h], a[0], kf_int<0>{});
            if constexpr (E >= 2) products(h_c, acc[h], a[1], kf_int<1>{});
            if constexpr (E == 4) {
                products(h_c, acc[h], a[2], kf_int<2>{});
                products(h_c, acc[h], a[3], kf_int<3>{});
            }
        };
        auto look_at = [&](auto h_c) __attribute__((always_inline)) {
            constexpr int h = decltype(h_c)::value;
            bool yes[HQ];
            if (__builtin_expect(!left(h_c, acc[h], E == 1 ? floor1 : E == 2 ? floor2 : floor_, yes), 1)) return;
            ++fails;
            if constexpr (E == 1) {
                products(h_c, acc[h], from_ring(blk, 1), kf_int<1>{});
                if (!left(h_c, acc[h], floor2, yes)) return;
            }
            if constexpr (E < 4) {
                const i32x4 a2 = operand(blk, 2), a3 = operand(blk, 3);
                products(h_c, acc[h], a2, kf_int<2>{});
                products(h_c, acc[h], a3, kf_int<3>{});
                if (!left(h_c, acc[h], floor_, yes)) return;
            }
#pragma unroll
            for (int s = 0; s < HQ; ++s)
                if (__ballot(yes[s])) batch = keep(h * HQ + s, acc[h][s], floor_[h * HQ + s], first + blk * 32) || batch;
        };
        auto copy_ahead = [&](int at) __attribute__((always_inline)) {          // block `at` to its place in the ring
#pragma unroll
            for (int c = 0; c < C; ++c) fetch(at, c, (unsigned)at % AHEAD * C + c);
        };
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // (nothing of another ring is on its way)
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) copy_ahead(blk + u);
        asm volatile("s_waitcnt vmcnt(%0)" ::"i"((AHEAD - 1) * C) : "memory");
#pragma unroll
        for (int c = 0; c < E; ++c) a[c] = from_ring(blk, c);
        first_steps(kf_int<0>{});
        if constexpr (H == 2) first_steps(kf_int<H - 1>{});
#pragma unroll 1
        while (true) {
            // Whole products: block blk's operands have been multiplied, block blk + AHEAD takes their place now;
            // early looks may come back for them, so its copy starts when they have been taken.
            if constexpr (E == 4) copy_ahead(blk + AHEAD);
            asm volatile("s_waitcnt vmcnt(%0)" ::"i"((E == 4 ? AHEAD - 1 : AHEAD - 2) * C) : "memory");      // block blk + 1 has come
#pragma unroll
            for (int c = 0; c < E; ++c) a[c] = from_ring(blk + 1, c);
            look_at(kf_int<0>{});
            first_steps(kf_int<0>{});
            if constexpr (H == 2) {
                look_at(kf_int<H - 1>{});
                first_steps(kf_int<H - 1>{});
            }
            if constexpr (E < 4) copy_ahead(blk + AHEAD);
            if (__builtin_expect(uniform(batch), 0)) {
                score_full(false);
                batch = false;
            }
            blk = uniform(blk + 1);
            if (__builtin_expect(blk == nblocks, 0)) return;
            if (__builtin_expect(blk % KF_SEG_BLOCKS == 0, 0)) {
                if (!same_look() || keeps_too_much() || !open_segment()) return;
            }
        }
    };
    int stop = nblocks;
    while (blk < nblocks) {
        if (keeps_too_much()) { stop = blk; break; }
        if (!open_segment()) {                         // nothing to multiply
            blk = uniform(min(blk + KF_SEG_BLOCKS, nblocks));
            continue;
        }
        look = uniform(look);
        if (look == 1) run(kf_int<1>{});
        else if (look == 2) run(kf_int<2>{});
        else run(kf_int<4>{});
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // nothing is left on its way to LDS
    score_full(true);
    for (int s = 0; s < NQ; ++s) {
        float tau = s_query[wv][s][1][col].w;
        int fill = s_fill[wv][s][lane];
        const u64 some = __ballot(fill > 0);
        fold(s, (uint32_t)some | (uint32_t)(some >> 32), tau, fill);
    }
    if (lane == 0) *my_resume = stop < nblocks ? first + stop * 32 : end < N ? end : 0x7fffffff;
}

static int64_t kf_rows(int64_t N) { return (N + 31) & ~(int64_t)31; }

// workspace of one ra_launch_knn_filter call over `graphs` graphs
struct KfLayout { size_t top, place, resume, seg, k8, q8, info, scores, total; };
static KfLayout kf_layout(int graphs, int64_t N, int64_t M, int knn) {
    KfLayout l;
    size_t o = 0;
    auto take = [&](size_t bytes) { const size_t at = o; o += (bytes + 255) & ~(size_t)255; return at; };
    l.top = take((size_t)graphs * 4);
    l.place = take((size_t)graphs * RA_D);
    l.resume = take((size_t)graphs * ((M + KF_WAVES * 32 - 1) / (KF_WAVES * 32)) * KF_WAVES * sizeof(int));
    l.seg = take((size_t)graphs * ((N + KF_SEG - 1) / KF_SEG) * sizeof(KfSegment));
    l.k8 = take((size_t)graphs * kf_rows(N) * RA_D);
    l.q8 = take((size_t)graphs * M * RA_D);
    l.info = take((size_t)graphs * M * sizeof(KfQuery));
    l.scores = take((size_t)graphs * M * knn * sizeof(float));
    l.total = o;
    return l;
}
size_t ra_knn_filter_bytes(int graphs, int64_t N, int64_t M, int knn) { return kf_layout(graphs, N, M, knn).total; }
float* ra_knn_filter_scores(void* workspace, int graphs, int64_t N, int64_t M, int knn) {
    return reinterpret_cast<float*>(reinterpret_cast<char*>(workspace) + kf_layout(graphs, N, M, knn).scores);
}

// column maxima of every KV head, once per build
ra_status ra_launch_knn_filter_scales(const void* K, ra_dtype dt, int n_seq_kv, int64_t N, uint32_t* maxabs,
                                      hipStream_t st) {
    hipLaunchKernelGGL(kf_zero_kernel, dim3((n_seq_kv * RA_D + 255) / 256), dim3(256), 0, st, maxabs, n_seq_kv * RA_D);
    int blocks = (int)((N + 255) / 256);                 // at least 16 rows per thread group
    const int most = n_seq_kv >= 512 ? 4 : 2048 / n_seq_kv;
    if (blocks > most) blocks = most;
    const dim3 grid((unsigned)blocks, (unsigned)n_seq_kv);
    if (dt == RA_BF16) hipLaunchKernelGGL(kf_maxabs_kernel<RA_BF16>, grid, dim3(256), 0, st, K, N, maxabs);
    else hipLaunchKernelGGL(kf_maxabs_kernel<RA_F32>, grid, dim3(256), 0, st, K, N, maxabs);
    RA_HIP(hipGetLastError());
    return RA_OK;
}

// Graphs [g0, g0 + n_graphs) of the `graphs` that `order` holds: the rest of their streams from position
// `from` on. L holds the lists of what came before, ra_knn_filter_scores(workspace, ...) their scores. The first
// launch of a group of graphs (from == first) makes the 8-bit copies. Every launch ends at stream position `end`, a whole number of
// segments on or N; what gives up before (resume: where) is knn.hip's up to there, and the next launch goes on from `end`.
ra_status ra_launch_knn_filter(const void* K, const void* Q, ra_dtype dt, const void* order, int graphs, int g0,
                               int n_graphs, int n_q, int n_kv, int64_t N, int64_t M, int knn, int64_t first, int64_t from,
                               int64_t end, const uint32_t* maxabs, void* workspace, hipStream_t st, int32_t* L,
                               const int** resume, int* resume_queries, int* resume_blocks) {
    const KfLayout l = kf_layout(n_graphs, N, M, knn);
    char* ws = reinterpret_cast<char*>(workspace);
    uint32_t* k_top = reinterpret_cast<uint32_t*>(ws + l.top);
    unsigned char* place = reinterpret_cast<unsigned char*>(ws + l.place);
    KfSegment* seg = reinterpret_cast<KfSegment*>(ws + l.seg);
    float* scores = reinterpret_cast<float*>(ws + l.scores);
    const int64_t rows8 = kf_rows(N - first);
    const int nseg = (int)((N - first + KF_SEG - 1) / KF_SEG);
    const u64* ord = reinterpret_cast<const u64*>(order);
    const int64_t stride = ra_knn_order_stride(N);
    int mq_samples;
    const float* mq = ra_knn_order_mean(order, graphs, N, M, &mq_samples);
    if (from == first)
        hipLaunchKernelGGL(kf_zero_kernel, dim3((n_graphs + 255) / 256), dim3(256), 0, st, k_top, n_graphs);
    const dim3 pgrid((unsigned)(nseg < 128 ? nseg : 128), (unsigned)n_graphs);
    const dim3 qgrid((unsigned)(M / 16 < 255 ? M / 16 + 1 : 256), (unsigned)n_graphs);
    int* res = reinterpret_cast<int*>(ws + l.resume);
    const int line = from == first ? KF_LINE_FIRST(dt) : KF_LINE_LAST;
    // four query sets per wavefront (a key operand feeds four chains: 39.9 ms against 47.1 with two and 69.9
    // with one, 128K keys x 32 heads; 4 heads 5.7, 6.2 and 9.0) unless that leaves compute units without a workgroup
    auto blocks = [&](int nq) { return (M + KF_WAVES * 32 * nq - 1) / (KF_WAVES * 32 * nq); };
    const int NQ = blocks(4) * n_graphs * KF_WAVES >= 2048 ? 4 : blocks(2) * n_graphs * KF_WAVES >= 2048 ? 2 : 1;
    const dim3 grid((unsigned)blocks(NQ), (unsigned)n_graphs);
#define KF_GO_N(DTV, NQV)                                                                                       \
    hipLaunchKernelGGL((knn_filter_kernel<DTV, NQV>), grid, dim3(KF_THREADS), 0, st, K, Q, ord, stride,         \
                       reinterpret_cast<unsigned char*>(ws + l.k8), rows8,                                      \
                       reinterpret_cast<unsigned char*>(ws + l.q8), reinterpret_cast<float4*>(ws + l.info),     \
                       seg, nseg, g0, n_q, n_kv, N, M, knn, (int)first, (int)from, (int)end, line, scores, L, res)
#define KF_GO(DTV)                                                                                              \
    do {                                                                                                        \
        if (from == first) {                                                                                    \
            hipLaunchKernelGGL(kf_rank_kernel<DTV>, dim3((unsigned)n_graphs), dim3(1024), 0, st, Q, mq,         \
                               mq_samples, maxabs, g0, n_q, n_kv, M, place);                                    \
            hipLaunchKernelGGL(kf_pack_kernel<DTV>, pgrid, dim3(1024), 0, st, K, ord, stride, maxabs, place,    \
                               g0, n_q, n_kv, N, first, rows8, nseg, reinterpret_cast<uint2*>(ws + l.k8), seg,  \
                               k_top);                                                                          \
            hipLaunchKernelGGL(kf_queries_kernel<DTV>, qgrid, dim3(256), 0, st, Q, mq, maxabs, place, k_top,    \
                               g0, n_q, n_kv, M, knn, scores, reinterpret_cast<uint2*>(ws + l.q8),              \
                               reinterpret_cast<float4*>(ws + l.info), res, (int)grid.x * KF_WAVES, 32 * NQ);   \
        }                                                                                                       \
        if (NQ == 4) KF_GO_N(DTV, 4); else if (NQ == 2) KF_GO_N(DTV, 2); else KF_GO_N(DTV, 1);                  \
    } while (0)
    if (dt == RA_BF16) KF_GO(RA_BF16); else KF_GO(RA_F32);
#undef KF_GO_N
#undef KF_GO
    *resume = res;
    *resume_queries = 32 * NQ;
    *resume_blocks = (int)grid.x * KF_WAVES;
    RA_HIP(hipGetLastError());
    return RA_OK;
}
