// 8-bit copy of the keys for the graph search. Appendix C of the paper names 8-bit scalar
// quantisation of the KV vectors as the next step without giving a scheme; the one here is
// symmetric, linear, per (sequence, KV head) and per dimension:
//     scale[d] = max_i |k[i][d]| / 127   (1 for an all-zero column)
//     k8[i][d] = clamp(round_half_even(k[i][d] / scale[d]), -127, 127)
// in float32, every division rounded once, so the bytes are reproducible on a CPU. Only the
// search reads the copy; attention uses the original keys.
#include "common.h"

// Both passes read the keys once, 16 bytes (float32: 32) per lane, 16 lanes per row: bound by memory. (A key per load, two
// rows per pass of a workgroup: 8 heads of 64K keys 137 us for the maxima and 70 for the copy, now 37 and 39; 16 heads of 5003
// keys 14.5 and 16.6, now 6.1 and 9.1. Keys that are not 16-byte aligned are still loaded one by one.)
#define QZ_THREADS 256
#define QZ_ROWS (QZ_THREADS / 16)  // rows per pass of a workgroup
#define QZ_FLY 4                   // passes in flight

// dimensions [8 l16, 8 l16 + 8) of row `row`; WIDE: K is 16-byte aligned (and the copy 8-byte)
template <int DT, bool WIDE>
__device__ __forceinline__ void qz_row8(const void* K, size_t row, int l16, float (&v)[8]) {
    const size_t at = row * RA_D + 8 * l16;
    if constexpr (!WIDE) {
#pragma unroll
        for (int c = 0; c < 8; ++c)
            v[c] = DT == RA_BF16 ? bf16_lo(reinterpret_cast<const uint16_t*>(K)[at + c]) : reinterpret_cast<const float*>(K)[at + c];
    } else if constexpr (DT == RA_BF16) {
        const uint4 u = *reinterpret_cast<const uint4*>(reinterpret_cast<const uint16_t*>(K) + at);
        v[0] = bf16_lo(u.x); v[1] = bf16_hi(u.x); v[2] = bf16_lo(u.y); v[3] = bf16_hi(u.y);
        v[4] = bf16_lo(u.z); v[5] = bf16_hi(u.z); v[6] = bf16_lo(u.w); v[7] = bf16_hi(u.w);
    } else {
        const float4 a = *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(K) + at);
        const float4 b = *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(K) + at + 4);
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
    }
}

// grid (workers, groups); |x| of a float is monotone in its bit pattern, so the column
// maxima are taken with integer atomic-max on the bits (maxabs zeroed beforehand)
template <int DT, bool WIDE>
__global__ __launch_bounds__(QZ_THREADS) void qz_maxabs_kernel(const void* __restrict__ K, int64_t N,
                                                               uint32_t* __restrict__ maxabs) {
    __shared__ uint32_t s_max[RA_D];
    const int tid = threadIdx.x, l16 = tid & 15;
    const size_t g = blockIdx.y;
    if (tid < RA_D) s_max[tid] = 0u;
    __syncthreads();
    uint32_t m[8] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};
    const int64_t step = (int64_t)gridDim.x * QZ_ROWS;
    for (int64_t r = (int64_t)blockIdx.x * QZ_ROWS + tid / 16; r < N; r += QZ_FLY * step) {
        float v[QZ_FLY][8];
#pragma unroll
        for (int u = 0; u < QZ_FLY; ++u) qz_row8<DT, WIDE>(K, g * N + (r + u * step < N ? r + u * step : r), l16, v[u]);
#pragma unroll
        for (int u = 0; u < QZ_FLY; ++u)
#pragma unroll
            for (int c = 0; c < 8; ++c) m[c] = max(m[c], __float_as_uint(v[u][c]) & 0x7fffffffu);
    }
#pragma unroll
    for (int c = 0; c < 8; ++c) atomicMax(&s_max[8 * l16 + c], m[c]);
    __syncthreads();
    if (tid < RA_D) atomicMax(&maxabs[g * RA_D + tid], s_max[tid]);
}

__global__ void qz_scale_kernel(float* __restrict__ scale, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float m = scale[i];                                               // the maximum's bits are its value
    scale[i] = m == 0.f ? 1.f : __fdiv_rn(m, 127.f);
}

template <int DT, bool WIDE>
__global__ __launch_bounds__(QZ_THREADS) void qz_write_kernel(const void* __restrict__ K, int64_t N,
                                                              const float* __restrict__ scale,
                                                              int8_t* __restrict__ K8) {
    const int tid = threadIdx.x, l16 = tid & 15;
    const size_t g = blockIdx.y;
    float s[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) s[c] = scale[g * RA_D + 8 * l16 + c];
    const int64_t step = (int64_t)gridDim.x * QZ_ROWS;
    for (int64_t r = (int64_t)blockIdx.x * QZ_ROWS + tid / 16; r < N; r += QZ_FLY * step) {
        float v[QZ_FLY][8];
#pragma unroll
        for (int u = 0; u < QZ_FLY; ++u) qz_row8<DT, WIDE>(K, g * N + (r + u * step < N ? r + u * step : r), l16, v[u]);
#pragma unroll
        for (int u = 0; u < QZ_FLY; ++u) {
            uint32_t w[2] = {0u, 0u};
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                float q = rintf(__fdiv_rn(v[u][c], s[c]));                  // rintf: half to even
                q = fminf(fmaxf(q, -127.f), 127.f);
                w[c / 4] |= ((uint32_t)(int)q & 255u) << (8 * (c & 3));
            }
            if (r + u * step >= N) continue;
            int8_t* out = K8 + (g * N + r + u * step) * RA_D + 8 * l16;
            if constexpr (WIDE) *reinterpret_cast<uint2*>(out) = make_uint2(w[0], w[1]);
            else
#pragma unroll
                for (int c = 0; c < 8; ++c) out[c] = (int8_t)(w[c / 4] >> (8 * (c & 3)));
        }
    }
}

__global__ void qz_zero_kernel(uint32_t* p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

// K [n_groups][N][128] -> K8 [n_groups][N][128], scale [n_groups][128]
ra_status ra_launch_quantize(const void* K, ra_dtype dt, int n_groups, int64_t N, hipStream_t st,
                             int8_t* K8, float* scale) {
    const int ns = n_groups * RA_D;
    hipLaunchKernelGGL(qz_zero_kernel, dim3((ns + 255) / 256), dim3(256), 0, st,
                       reinterpret_cast<uint32_t*>(scale), ns);
    // workgroups that fill the part a few times over, none without rows
    int64_t blocks = (N + QZ_ROWS * QZ_FLY - 1) / (QZ_ROWS * QZ_FLY);
    const int64_t most = n_groups >= 2048 ? 1 : 2048 / n_groups;
    if (blocks > most) blocks = most;
    const dim3 grid((unsigned)blocks, (unsigned)n_groups);
    const bool wide = (uintptr_t)K % 16 == 0 && (uintptr_t)K8 % 8 == 0;
#define QZ_GO(DTV, WIDEV)                                                                                    \
    do {                                                                                                     \
        hipLaunchKernelGGL((qz_maxabs_kernel<DTV, WIDEV>), grid, dim3(QZ_THREADS), 0, st, K, N,               \
                           reinterpret_cast<uint32_t*>(scale));                                              \
        hipLaunchKernelGGL(qz_scale_kernel, dim3((ns + 255) / 256), dim3(256), 0, st, scale, ns);            \
        hipLaunchKernelGGL((qz_write_kernel<DTV, WIDEV>), grid, dim3(QZ_THREADS), 0, st, K, N, scale, K8);    \
    } while (0)
    if (dt == RA_BF16) { if (wide) QZ_GO(RA_BF16, true); else QZ_GO(RA_BF16, false); }
    else { if (wide) QZ_GO(RA_F32, true); else QZ_GO(RA_F32, false); }
#undef QZ_GO
    RA_HIP(hipGetLastError());
    return RA_OK;
}
