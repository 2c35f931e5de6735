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
// The bound. Per KV head and dimension, c_d = max_i |k_id| / 127 and k_id = c_d (x_id + e_id) with
// x_id the nearest integer; per query q'_d = q_d c_d = s (y_d + f_d) with s = max_d |q'_d| / 127
// and y_d the nearest integer. Then
//     <q, k> = s <y, x> + s <f, x> + <q', e>,   |<q, k> - s <y, x>| <= s |f| |x| + |q'| |e|,
// where <y, x> is an exact integer (at most 128 x 127 x 127) from v_mfma_i32_32x32x32_i8 and the
// largest |x| and |e| over the head's keys are taken when the copy is made. Every norm is taken relative to
// a power of two or to s (|q'| = s |y + f|), so none of them loses its terms where squares of the
// inputs leave the range of float32, and every norm is widened by 0.1 % and a little more for its own rounding.
// What the floating point sum of the exact path can be off by is added: 2^-15 |q| |k|, several times what
// 128 additions in float32 can lose; and, should the matrix cores take denormal numbers for zero, 2^-126
// sqrt(128) (|q| + |k|) for the inputs and 256 x 2^-126 for products and partial sums. So a key
// whose score could reach a query's threshold tau has <y, x> >= (tau - bound) / s: one integer per
// query, compared with the largest of a lane's 16 accumulators. Where that does not hold nothing is ruled out
// (an infinite bound: the integer is the smallest there is): non-finite inputs, norms whose product could
// overflow a score (10^38), and s below 2^-100, where the quotients above would round in the denormal range.
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
#define KF_SROWS (KF_WAVES * 16)    // keys per stage: 32 bytes per thread
#define KF_STAGE (KF_SROWS * RA_D)
#define KF_RUN 4                   // scored keys a lane can hold for its query's list
#define KF_RUNS (2 * KF_RUN)       // ... and the two lanes of a query together
#define KF_CHECK (1024 / KF_SROWS)                 // stages between two looks at how much the filter rules out
#define KF_PENDING 64              // keys a query set can have waiting to be scored (a batch is 32)

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

__device__ __forceinline__ float kf_scale(uint32_t maxabs_bits) {
    return maxabs_bits == 0u ? 1.f : __uint_as_float(maxabs_bits) * (1.0f / 127.0f);
}
// Exponent of the largest |k| of a head, from its column maxima (16 lanes hold 8 of them each). Norms of keys
// are taken over k 2^-exponent: their squares neither overflow nor, for the largest of them, vanish.
__device__ __forceinline__ int kf_exponent(const uint32_t (&maxabs_bits)[8]) {
    uint32_t top = 0u;
#pragma unroll
    for (int c = 0; c < 8; ++c) top = max(top, maxabs_bits[c]);
#pragma unroll
    for (int d = 1; d < 16; d <<= 1) top = max(top, (uint32_t)__shfl_xor((int)top, d));
    return __builtin_amdgcn_frexp_expf(__uint_as_float(top));       // (0 for zero, infinity and NaN)
}

// ---- the 8-bit copy of a head's keys in stream order ----------------------------------------------
// Row p of a graph (128 bytes) holds the key streamed p-th, its 16-byte chunks at chunk ^ (p / 2 % 8):
// the layout a stage has in LDS, so that a stage is one linear copy and operand reads (16 rows, the
// same chunk) cover all 64 banks. Rows beyond N are zero. bounds[graph]: bits of the largest |e|^2,
// |x|^2 and |k 2^-kf_exponent|^2 of the graph's keys.
// grid (rows / 64, graphs); 16 lanes per row
template <int DT>
__global__ __launch_bounds__(1024) void kf_pack_kernel(const void* __restrict__ K, const u64* __restrict__ order,
                                                       int64_t order_stride, const uint32_t* __restrict__ maxabs,
                                                       int g0, int n_q, int n_kv, int64_t N, int64_t rows8,
                                                       uint2* __restrict__ K8, uint32_t* __restrict__ bounds) {
    __shared__ uint32_t s_b[4];
    const int gl = blockIdx.y, graph = g0 + gl, seq = graph / n_q, h = graph % n_q, kvh = h / (n_q / n_kv);
    const int tid = threadIdx.x, l16 = tid & 15;
    const size_t kv = (size_t)seq * n_kv + kvh;
    if (tid < 4) s_b[tid] = 0u;
    __syncthreads();
    float sc[8], inv[8];
    uint32_t mx[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        mx[c] = maxabs[kv * RA_D + 8 * l16 + c];
        sc[c] = kf_scale(mx[c]);
        inv[c] = 1.0f / sc[c];
    }
    const int k_exp = kf_exponent(mx);
    const u64* ord = order + (size_t)graph * order_stride;
    for (int64_t p = (int64_t)blockIdx.x * 64 + tid / 16; p < rows8; p += (int64_t)gridDim.x * 64) {
        uint32_t w[2] = {0u, 0u};
        float e2 = 0.f, x2 = 0.f, k2 = 0.f;
        if (p < N) {
            const int64_t id = (int64_t)(uint32_t)ord[p];
            float v[8];
            kf_row8<DT>(K, (kv * N + id) * RA_D + 8 * l16, v);
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                float x = rintf(v[c] * inv[c]);
                x = fminf(fmaxf(x, -127.f), 127.f);
                const float e = __fmaf_rn(-x, sc[c], v[c]) * inv[c];
                e2 += e * e;
                x2 += x * x;
                const float k = __builtin_amdgcn_ldexpf(v[c], -k_exp);
                k2 += k * k;
                w[c / 4] |= ((uint32_t)(int)x & 255u) << (8 * (c % 4));
            }
        }
        const int chunk = (l16 >> 1) ^ (int)((p >> 1) & 7);
        K8[((size_t)gl * rows8 + p) * 16 + chunk * 2 + (l16 & 1)] = make_uint2(w[0], w[1]);
#pragma unroll
        for (int d = 1; d < 16; d <<= 1) {
            e2 += __shfl_xor(e2, d);
            x2 += __shfl_xor(x2, d);
            k2 += __shfl_xor(k2, d);
        }
        if (l16 == 0) {
            // a NaN (from non-finite keys) has the largest bits of all
            atomicMax(&s_b[0], __float_as_uint(e2) & 0x7fffffffu);
            atomicMax(&s_b[1], __float_as_uint(x2) & 0x7fffffffu);
            atomicMax(&s_b[2], __float_as_uint(k2) & 0x7fffffffu);
        }
    }
    __syncthreads();
    if (tid < 3) atomicMax(&bounds[gl * 4 + tid], s_b[tid]);
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

// smallest <y, x> a key needs so that its score can reach tau
__device__ __forceinline__ int kf_floor(float tau, float bound, float inv_s) {
    const float x = (tau - bound) * inv_s;
    if (!(x > -1.0e9f)) return (int)0x80000000;         // also NaN: nothing is ruled out
    return x > 1.0e9f ? 1000000000 : (int)floorf(x) - 2;
}

// ---- the queries in 8 bits: y (128 bytes per query, in order), and per query [bound, 1 / s, tau, 0]
// grid (rows / 16, graphs); 16 lanes per row
template <int DT>
__global__ __launch_bounds__(256) void kf_queries_kernel(const void* __restrict__ Q,
                                                         const uint32_t* __restrict__ maxabs,
                                                         const uint32_t* __restrict__ bounds, int g0, int n_q,
                                                         int n_kv, int64_t M, int knn,
                                                         const float* __restrict__ scores, uint2* __restrict__ Q8,
                                                         float4* __restrict__ qinfo) {
    const int gl = blockIdx.y, graph = g0 + gl, seq = graph / n_q, h = graph % n_q, kvh = h / (n_q / n_kv);
    const int tid = threadIdx.x, l16 = tid & 15;
    const size_t kv = (size_t)seq * n_kv + kvh;
    float sc[8];
    uint32_t mx[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        mx[c] = maxabs[kv * RA_D + 8 * l16 + c];
        sc[c] = kf_scale(mx[c]);
    }
    const float e_max = 1.001f * sqrtf(__uint_as_float(bounds[gl * 4])) + 1e-3f;
    const float x_max = 1.001f * sqrtf(__uint_as_float(bounds[gl * 4 + 1]));
    const float k_max = __builtin_amdgcn_ldexpf(1.001f * sqrtf(__uint_as_float(bounds[gl * 4 + 2])), kf_exponent(mx));
    for (int64_t j = (int64_t)blockIdx.x * 16 + tid / 16; j < M; j += (int64_t)gridDim.x * 16) {
        float v[8], p[8], top = 0.f, q_top = 0.f;
        kf_row8<DT>(Q, ((size_t)graph * M + j) * RA_D + 8 * l16, v);
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            p[c] = v[c] * sc[c];
            top = fmaxf(top, fabsf(p[c]));
            q_top = fmaxf(q_top, fabsf(v[c]));
        }
#pragma unroll
        for (int d = 1; d < 16; d <<= 1) {
            top = fmaxf(top, __shfl_xor(top, d));
            q_top = fmaxf(q_top, __shfl_xor(q_top, d));
        }
        const float s = top > 0.f ? top * (1.0f / 127.0f) : 1.f, inv = 1.0f / s;
        const int q_exp = __builtin_amdgcn_frexp_expf(q_top);
        float f2 = 0.f, n2 = 0.f, q2 = 0.f;              // |f|^2, |q' / s|^2, |q 2^-q_exp|^2
        uint32_t w[2] = {0u, 0u};
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
            w[c / 4] |= ((uint32_t)(int)y & 255u) << (8 * (c % 4));
        }
#pragma unroll
        for (int d = 1; d < 16; d <<= 1) {
            f2 += __shfl_xor(f2, d);
            n2 += __shfl_xor(n2, d);
            q2 += __shfl_xor(q2, d);
        }
        Q8[((size_t)gl * M + j) * 16 + l16] = make_uint2(w[0], w[1]);
        if (l16 == 0) {
            const float q_norm = __builtin_amdgcn_ldexpf(1.001f * sqrtf(q2), q_exp), norms = q_norm * k_max;
            float bound = 1.002f * s * ((1.001f * sqrtf(f2) + 1e-3f) * x_max + 1.001f * sqrtf(n2) * e_max) +
                          3.1e-5f * norms + 1.4e-37f * (q_norm + k_max) + 1e-35f;
            if (!(s >= 0x1p-100f && norms < 1e38f)) bound = INFINITY;
            qinfo[(size_t)gl * M + j] = make_float4(bound, inv, scores[((size_t)gl * M + j) * knn + knn - 1], 0.f);
        }
    }
}

// grid: x = block of KF_WAVES * NQ * 32 queries, y = graph of the launch. A wavefront owns NQ sets
// of 32 queries. What only the rare path needs (a query's bound, scale and threshold, the waiting keys)
// sits in LDS; a lane keeps its queries' 8-bit operands and integer floors.
template <int DT, int NQ>
__global__ __launch_bounds__(KF_THREADS, NQ <= 2 ? 4 : 2) void knn_filter_kernel(
    const void* __restrict__ K, const void* __restrict__ Q, const u64* __restrict__ order, int64_t order_stride,
    const unsigned char* __restrict__ K8, int64_t rows8, const unsigned char* __restrict__ Q8,
    const float4* __restrict__ qinfo, int g0, int n_q, int n_kv, int64_t N, int64_t M, int knn, int first_stage,
    float* scores, int32_t* L, int* __restrict__ resume) {
    __shared__ __align__(16) unsigned char stage_buf[2 * KF_STAGE];
    __shared__ int s_pend[KF_WAVES][NQ][KF_PENDING];
    __shared__ int s_count[KF_WAVES][NQ];
    __shared__ u64 s_run[KF_WAVES][NQ][KF_RUN][RA_WAVE];
    __shared__ int s_fill[KF_WAVES][NQ][RA_WAVE];
    __shared__ int s_kept;
    __shared__ float s_bound[KF_WAVES][NQ][32], s_inv[KF_WAVES][NQ][32], s_tau[KF_WAVES][NQ][32];
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

    i32x4 b[NQ][4];
    int floor_[NQ];
#pragma unroll
    for (int s = 0; s < NQ; ++s) {
        int64_t qr = q0 + 32 * s + col;
        if (qr >= M) qr = M - 1;                       // such columns are never written
        const i32x4* src = reinterpret_cast<const i32x4*>(Q8 + ((size_t)gl * M + qr) * RA_D + 64 * half);
#pragma unroll
        for (int c = 0; c < 4; ++c) b[s][c] = src[c];
        const float4 qi = qinfo[(size_t)gl * M + qr];
        floor_[s] = kf_floor(qi.z, qi.x, qi.y);
        s_bound[wv][s][col] = qi.x;
        s_inv[wv][s][col] = qi.y;
        s_tau[wv][s][col] = qi.z;
        s_count[wv][s] = 0;
        s_fill[wv][s][lane] = 0;
    }
    if (tid == 0) s_kept = 0;

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
    // exact scores of the first n waiting keys of set s; those that reach a threshold join their
    // query's run
    auto score_pending = [&](int s, int n) __attribute__((always_inline)) {
        const int p = s_pend[wv][s][col < n ? col : 0];
        const int id = ord[2 * (size_t)(unsigned)p];
        int64_t qr = q0 + 32 * s + col;
        const bool mine = qr < M;
        if (!mine) qr = M - 1;
        float tau = s_tau[wv][s][col];
        int fill = s_fill[wv][s][lane];
        const f32x16 c = kf_scores<DT>(Kh, (size_t)id, Qh, (size_t)qr, half);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int row = (r / 4) * 8 + half * 4 + (r % 4);
            const bool ok = mine && row < n && c[r] > -INFINITY;
            if (__ballot(ok && c[r] >= tau) == 0ull) continue;
            const u64 full = __ballot(ok && c[r] >= tau && fill == KF_RUN);
            if (full) fold(s, (uint32_t)full | (uint32_t)(full >> 32), tau, fill);
            const int lo = __builtin_amdgcn_readlane(id, (r / 4) * 8 + (r % 4));
            const int hi = __builtin_amdgcn_readlane(id, (r / 4) * 8 + 4 + (r % 4));
            if (ok && c[r] >= tau) s_run[wv][s][fill++][lane] = kf_key(c[r], half ? hi : lo);
            kf_wave_sync();
        }
        s_tau[wv][s][col] = tau;
        s_fill[wv][s][lane] = fill;
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
        const int have = __builtin_amdgcn_readfirstlane(s_count[wv][s]);
        if (lane < 32 && ((rows >> lane) & 1u))
            s_pend[wv][s][have + __popc(rows & ((1u << lane) - 1u))] = pos + lane;
        s_count[wv][s] = have + __popc(rows);
        if (lane == 0) atomicAdd(&s_kept, __popc(rows));
        return have + __popc(rows) >= 32;
    };
    // sets with a full batch waiting (or, at the end, any key) are scored; their floors follow
    auto score_full = [&](bool all) __attribute__((always_inline)) {
        kf_wave_sync();
        for (int s = 0; s < NQ; ++s) {
            const int have = __builtin_amdgcn_readfirstlane(s_count[wv][s]);
            if (have < 32 && !(all && have)) continue;
            const int n = have < 32 ? have : 32;
            score_pending(s, n);
            const int more = s_pend[wv][s][32 + col];
            kf_wave_sync();
            if (lane < have - n) s_pend[wv][s][lane] = more;
            s_count[wv][s] = have - n;
        }
#pragma unroll
        for (int s = 0; s < NQ; ++s) floor_[s] = kf_floor(s_tau[wv][s][col], s_bound[wv][s][col], s_inv[wv][s][col]);
    };

    // ---- the stream: a stage is requested two stages before it is multiplied, waits one stage in
    //      registers and one in its LDS buffer
    const unsigned char* K8g = K8 + (size_t)gl * rows8 * RA_D;
    const int nstage = (int)(rows8 / KF_SROWS);
    struct Held { uint4 c0, c1; };
    auto fetch = [&](Held& hd, int st) __attribute__((always_inline)) {
        if (st >= nstage) st = nstage - 1;             // past the end: the last stage again, unused
        const unsigned char* src = K8g + (size_t)st * KF_STAGE + tid * 16;
        hd.c0 = *reinterpret_cast<const uint4*>(src);
        hd.c1 = *reinterpret_cast<const uint4*>(src + KF_THREADS * 16);
    };
    auto store = [&](const Held& hd, unsigned char* buf) __attribute__((always_inline)) {
        *reinterpret_cast<uint4*>(buf + tid * 16) = hd.c0;
        *reinterpret_cast<uint4*>(buf + (KF_THREADS + tid) * 16) = hd.c1;
    };
    int at[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) at[c] = col * RA_D + (((4 * half + c) ^ ((col >> 1) & 7)) << 4);
    auto multiply = [&](const unsigned char* buf, int st) __attribute__((always_inline)) {
#pragma unroll
        for (int blk = 0; blk < KF_SROWS / 32; ++blk) {
            i32x4 a[4];
#pragma unroll
            for (int c = 0; c < 4; ++c)
                a[c] = *reinterpret_cast<const i32x4*>(buf + at[c] + blk * 32 * RA_D);
            i32x16 acc[NQ];
#pragma unroll
            for (int s = 0; s < NQ; ++s) {
                const i32x16 z = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
                acc[s] = z;
            }
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int s = 0; s < NQ; ++s)
                    acc[s] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[c], b[s][c], acc[s], 0, 0, 0);
            bool any = false, over[NQ];
#pragma unroll
            for (int s = 0; s < NQ; ++s) {
                int m = acc[s][0];
#pragma unroll
                for (int r = 1; r < 16; ++r) m = max(m, acc[s][r]);
                over[s] = m >= floor_[s];
                any = any || over[s];
            }
            if (__ballot(any) == 0ull) continue;
            const int pos = st * KF_SROWS + blk * 32;
            bool batch = false;
#pragma unroll
            for (int s = 0; s < NQ; ++s)
                if (__ballot(over[s])) batch = keep(s, acc[s], floor_[s], pos) || batch;
            if (batch) score_full(false);
        }
    };
    // Scoring a kept key costs about ten times what ruling it out does. Inputs whose scores the bound
    // cannot tell apart (most keys tied, a few dimensions that dwarf the others) are better off in
    // knn.hip's loop: when a workgroup has kept more than an eighth of what it has seen it stops and
    // leaves the rest of its stream there.
    auto keeps_too_much = [&](int seen) __attribute__((always_inline)) {
        return (int64_t)s_kept * 8 > (int64_t)seen * KF_SROWS * KF_WAVES * NQ;
    };
    Held ha, hb;
    fetch(ha, first_stage);
    store(ha, stage_buf);
    fetch(ha, first_stage + 1);
    fetch(hb, first_stage + 2);
    __syncthreads();
    int stop = nstage;
    for (int st = first_stage; st < nstage; st += 2) {
        multiply(stage_buf, st);
        store(ha, stage_buf + KF_STAGE);               // stage st + 1
        __syncthreads();
        fetch(ha, st + 3);
        if (st + 1 >= nstage) break;
        multiply(stage_buf + KF_STAGE, st + 1);
        store(hb, stage_buf);                          // stage st + 2
        const bool look = (st + 2 - first_stage) % KF_CHECK == 0 || st == first_stage;
        __syncthreads();
        if (look) {
            const bool quit = keeps_too_much(st + 2 - first_stage);
            __syncthreads();                           // (everyone has read the count before it moves on)
            if (quit) { stop = st + 2; break; }
        }
        fetch(hb, st + 4);
    }
    score_full(true);
    for (int s = 0; s < NQ; ++s) {
        float tau = s_tau[wv][s][col];
        int fill = s_fill[wv][s][lane];
        const u64 some = __ballot(fill > 0);
        fold(s, (uint32_t)some | (uint32_t)(some >> 32), tau, fill);
    }
    if (tid == 0) resume[(size_t)gl * gridDim.x + blockIdx.x] = stop < nstage ? stop * KF_SROWS : 0x7fffffff;
}

static int64_t kf_rows(int64_t N) { return (N + KF_SROWS - 1) / KF_SROWS * KF_SROWS; }

// workspace of one ra_launch_knn_filter call over `graphs` graphs
struct KfLayout { size_t bounds, resume, k8, q8, info, scores, total; };
static KfLayout kf_layout(int graphs, int64_t N, int64_t M, int knn) {
    KfLayout l;
    size_t o = 0;
    auto take = [&](size_t bytes) { const size_t at = o; o += (bytes + 255) & ~(size_t)255; return at; };
    l.bounds = take((size_t)graphs * 16);
    l.resume = take((size_t)graphs * ((M + KF_WAVES * 32 - 1) / (KF_WAVES * 32)) * sizeof(int));
    l.k8 = take((size_t)graphs * kf_rows(N) * RA_D);
    l.q8 = take((size_t)graphs * M * RA_D);
    l.info = take((size_t)graphs * M * sizeof(float4));
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

// Graphs [g0, g0 + n_graphs): the rest of their streams from position `first` (a multiple of
// KF_SROWS) on. L holds the lists of the first part, ra_knn_filter_scores(workspace, ...) their scores.
ra_status ra_launch_knn_filter(const void* K, const void* Q, ra_dtype dt, const void* order, int g0, int n_graphs,
                               int n_q, int n_kv, int64_t N, int64_t M, int knn, int64_t first,
                               const uint32_t* maxabs, void* workspace, hipStream_t st, int32_t* L,
                               const int** resume, int* resume_queries, int* resume_blocks) {
    const KfLayout l = kf_layout(n_graphs, N, M, knn);
    char* ws = reinterpret_cast<char*>(workspace);
    uint32_t* bounds = reinterpret_cast<uint32_t*>(ws + l.bounds);
    float* scores = reinterpret_cast<float*>(ws + l.scores);
    const int64_t rows8 = kf_rows(N);
    const u64* ord = reinterpret_cast<const u64*>(order);
    const int64_t stride = ra_knn_order_stride(N);
    hipLaunchKernelGGL(kf_zero_kernel, dim3((n_graphs * 4 + 255) / 256), dim3(256), 0, st, bounds, n_graphs * 4);
    const dim3 pgrid((unsigned)(rows8 / 64 < 128 ? rows8 / 64 : 128), (unsigned)n_graphs);
    const dim3 qgrid((unsigned)(M / 16 < 255 ? M / 16 + 1 : 256), (unsigned)n_graphs);
    int* res = reinterpret_cast<int*>(ws + l.resume);
    // four query sets per wavefront (a key operand feeds four chains: 64 ms against 71 with two and 103
    // with one, 128K keys x 32 heads) unless that leaves compute units without a workgroup
    auto blocks = [&](int nq) { return (M + KF_WAVES * 32 * nq - 1) / (KF_WAVES * 32 * nq); };
    const int NQ = blocks(4) * n_graphs >= 256 ? 4 : blocks(2) * n_graphs >= 256 ? 2 : 1;
    const dim3 grid((unsigned)blocks(NQ), (unsigned)n_graphs);
#define KF_GO_N(DTV, NQV)                                                                                       \
    hipLaunchKernelGGL((knn_filter_kernel<DTV, NQV>), grid, dim3(KF_THREADS), 0, st, K, Q, ord, stride,         \
                       reinterpret_cast<unsigned char*>(ws + l.k8), rows8,                                      \
                       reinterpret_cast<unsigned char*>(ws + l.q8), reinterpret_cast<float4*>(ws + l.info),     \
                       g0, n_q, n_kv, N, M, knn, (int)(first / KF_SROWS), scores, L, res)
#define KF_GO(DTV)                                                                                              \
    do {                                                                                                        \
        hipLaunchKernelGGL(kf_pack_kernel<DTV>, pgrid, dim3(1024), 0, st, K, ord, stride, maxabs, g0, n_q, n_kv, \
                           N, rows8, reinterpret_cast<uint2*>(ws + l.k8), bounds);                              \
        hipLaunchKernelGGL(kf_queries_kernel<DTV>, qgrid, dim3(256), 0, st, Q, maxabs, bounds, g0, n_q, n_kv, M, \
                           knn, scores, reinterpret_cast<uint2*>(ws + l.q8),                                    \
                           reinterpret_cast<float4*>(ws + l.info));                                             \
        if (NQ == 4) KF_GO_N(DTV, 4); else if (NQ == 2) KF_GO_N(DTV, 2); else KF_GO_N(DTV, 1);                  \
    } while (0)
    if (dt == RA_BF16) KF_GO(RA_BF16); else KF_GO(RA_F32);
#undef KF_GO_N
#undef KF_GO
    *resume = res;
    *resume_queries = KF_WAVES * 32 * NQ;
    *resume_blocks = (int)grid.x;
    RA_HIP(hipGetLastError());
    return RA_OK;
}
