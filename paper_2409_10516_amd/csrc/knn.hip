// Exact KNN from prefill queries to keys (Sec. 3.2, Fig. 2b): S = Q K^T on the matrix cores
// with the per-query top-knn selection fused behind it, so the M x N score matrix is never
// written anywhere.
//
// The product is computed transposed, one 32-key x 32-query block at a time:
//     C[key i][query j] += A[i][k] * B[k][j],  A = key rows, B = query rows,
// with v_mfma_f32_32x32x16_bf16 (bf16 inputs) or v_mfma_f32_32x32x2_f32 (fp32 inputs). In the
// 32x32 accumulator layout a lane holds ONE query column (lane % 32) and 16 key rows, so the
// selection threshold of a query is a single per-lane register: the common case is a
// max-tree over the lane's 16 scores and one compare. Only scores that reach the threshold go
// further (about knn * ln(N / knn) per query over a stream in storage order, a third of that in
// the order the keys are streamed in here: see knn_order.hip). The two lanes of a query hold its best keys so far in
// registers, sorted, half of the list each, and a run of pending slots in LDS each: a lane appends a score and an
// id to its own run with a single LDS write; when a run cannot take what a lane is about to append, the wavefront
// merges the runs of all its 32 queries into their lists at once, by sorting networks whose exchanges are one
// maximum and one minimum for 64 lanes, between the two lanes by half-wave swaps. (400 to 600 instructions for 32
// queries; one query at a time, its 64 slots sorted across the lanes by a bitonic network, took 200 for each. First
// 4096 keys of 32 heads x 128K queries, lists of 32: 12.5 -> 7.0 ms, of which writing scores and ids as they are, without
// a branch, instead of whole keys 0.8 ms. Lists of 64, by sorted insertion before, 3000 keys x 3000 queries x 32 heads:
// 2.0 -> 0.27 ms.)
// Between two merges a threshold is stale but valid (never above the true one), so nothing is
// lost.
//
// A wavefront owns 32 queries for the whole key stream (their B operands stay in registers); a
// workgroup is WAVES wavefronts. Lists hold
// 64-bit keys [0:1][ordered(score):32][2^31 - 1 - id:31], so "larger key" is "(score descending, id ascending)". The
// bits of a key are also those of a positive double of the same order (the scores that are numbers, and zero
// for an empty slot, give neither NaNs nor denormals), whose maximum and minimum are single instructions.
// The inner-product summation order is the hardware's; identical key rows still score
// identically for a given query because they go through the same instruction sequence.
//
// Key rows reach the matrix cores through LDS. In the operand layout a lane holds 16 bytes of
// its own row per step, so a load straight from memory touches 64 cache lines per instruction
// and the vector cache's line rate, not the matrix cores, sets the pace. Instead the workgroup
// copies the key stream in 16 KB stages straight to LDS (16 lanes per 256-byte row, each stage fetched once for all
// its wavefronts, two stages ahead of its use in bf16 and one in float32), a lane taking the chunk that belongs at its place
// with the 16-byte chunks of a row XOR-swizzled by the row number, and every wavefront
// reads its operands from there with conflict-free 16-byte LDS reads; one barrier per stage. What a stage of 64 keys costs 256
// queries: 1.1 us, of which the products alone with a barrier take 0.76 (two wavefronts per SIMD, 1.4 PFLOP/s); the first eight
// stages 26 instead of 9, for the merges of keys that are nearly all kept, and 9 us go before and after the stream. Through
// registers, with the loop unrolled twice and a merge in each of 16 places, whole calls took 2.5 to 4 % longer (32 heads: 2 x
// 5003 keys x 5003 queries 720 -> 697 us, 12000 x 12000 1415 -> 1366; float32 up to 11 %). No gain: the operands of two blocks
// read and multiplied before the first is looked at, half of the wavefronts a block behind, their priority raised, two stages per
// barrier; worse: workgroups of four wavefronts with stages of 8 KB (+8 to 16 %) or of two.

#include "common.h"

#define KN_PLACES 17              // places of a pending run: one more than it holds (see knn_kernel)
#define KN_PEND (KN_PLACES - 1)
#define KN_IDS 8                  // stages whose key ids are in LDS or on their way there, a power of two
#define KN_RUN_BYTES (KN_PLACES * RA_WAVE * 8)      // pending runs of a wavefront

typedef unsigned long long u64;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef u32x4 kn_any16 __attribute__((aligned(2)));       // 16 bytes at any element

__device__ __forceinline__ u64 knn_key(float score, int id) {
    return ((u64)f32_ordered(score) << 31) | (u64)(0x7fffffffu - (uint32_t)id);
}
__device__ __forceinline__ int knn_key_id(u64 k) { return k == 0ull ? -1 : (int)(0x7fffffffu - ((uint32_t)k & 0x7fffffffu)); }
// memory that one lane of a wavefront wrote and another reads: the hardware keeps the wavefront's order,
// this keeps the compiler's
__device__ __forceinline__ void kn_wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}
__device__ __forceinline__ float knn_key_score(u64 k) { return f32_from_ordered((uint32_t)(k >> 31)); }

// ---- merging pending keys into lists, all 32 queries of a wavefront at once ------------------------------
// Lane (col, half) holds a part of the keys of query col. In-lane exchanges work on registers of one lane, cross
// exchanges between the register of a lane and that of the query's other lane.
template <bool DESC>
__device__ __forceinline__ void kn_exchange(double& a, double& b) {
    const double lo = __builtin_fmin(a, b), hi = __builtin_fmax(a, b);
    a = DESC ? hi : lo;
    b = DESC ? lo : hi;
}
// Batcher's odd-even merge sort of N registers of each lane, descending
template <int N>
__device__ __forceinline__ void kn_sort(double (&v)[N]) {
#pragma unroll
    for (int p = 1; p < N; p *= 2)
#pragma unroll
        for (int k = p; k >= 1; k /= 2)
#pragma unroll
            for (int j = k % p; j + k < N; j += 2 * k)
#pragma unroll
                for (int i = 0; i < k; ++i)
                    if (i + j + k < N && (i + j) / (2 * p) == (i + j + k) / (2 * p)) kn_exchange<true>(v[i + j], v[i + j + k]);
}
// the in-lane part of a bitonic merge: distances N / 2 down to 1
template <int N, bool DESC>
__device__ __forceinline__ void kn_merge(double (&v)[N]) {
#pragma unroll
    for (int d = N / 2; d >= 1; d /= 2)
#pragma unroll
        for (int i = 0; i < N; ++i)
            if ((i & d) == 0) kn_exchange<DESC>(v[i], v[i | d]);
}
// Exchange between the two lanes of a query, register by register: the lower lane keeps the larger (DESC) or the
// smaller. Two registers at a time: after a swap of the one's upper with the other's lower half the pairs
// to compare sit in the same lane.
__device__ __forceinline__ void kn_swap_halves(double& a, double& b) {
    const u64 x = __builtin_bit_cast(u64, a), y = __builtin_bit_cast(u64, b);
    const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)y, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
    a = __builtin_bit_cast(double, ((u64)hi[0] << 32) | lo[0]);
    b = __builtin_bit_cast(double, ((u64)hi[1] << 32) | lo[1]);
}
template <int N, bool DESC>
__device__ __forceinline__ void kn_cross(double (&v)[N]) {
#pragma unroll
    for (int i = 0; i < N; i += 2) {
        kn_swap_halves(v[i], v[i + 1]);
        kn_exchange<DESC>(v[i], v[i + 1]);
        kn_swap_halves(v[i], v[i + 1]);
    }
}
// the pending keys of both lanes, sorted ascending over them (the lower lane holds the smaller ones)
template <int N>
__device__ __forceinline__ void kn_sort_pending(double (&v)[N], int half) {
    // the upper lane sorts negated keys: its own come out ascending, and both together are bitonic
    const u64 sign = (u64)half << 63;
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = __builtin_bit_cast(double, __builtin_bit_cast(u64, v[i]) ^ sign);
    kn_sort<N>(v);
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = __builtin_bit_cast(double, __builtin_bit_cast(u64, v[i]) ^ sign);
    kn_cross<N, false>(v);
    kn_merge<N, false>(v);
}

// Merges the pending keys (`fill` of this lane; place i of all lanes' runs is 64 scores, then 64 ids) of all 32 queries
// into their lists: the lower lane of a query holds its best LN keys, descending, the upper lane the next LN.
template <int LN>
__device__ __forceinline__ void knn_fold(double (&list)[LN], const uint32_t* run, int half, int fill) {
    static_assert(LN == 16 || LN == 32, "lists of up to 32 or up to 64 keys");
    double p[KN_PEND];
#pragma unroll
    for (int i = 0; i < KN_PEND; ++i) {
        const u64 k = knn_key(__uint_as_float(run[i * 128]), (int)run[i * 128 + 64]);
        p[i] = __builtin_bit_cast(double, i < fill ? k : 0ull);
    }
    kn_sort_pending<KN_PEND>(p, half);
    // list descending against pending ascending (none before its 32): the larger of each pair are the best 2 LN, a
    // bitonic sequence over the two lanes
    if constexpr (LN == 16) {
#pragma unroll
        for (int i = 0; i < 16; ++i) list[i] = __builtin_fmax(list[i], p[i]);
    } else {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            double low = p[i], own = p[i];
            kn_swap_halves(low, own);                 // low: the lower lane's value in both
            list[i] = __builtin_fmax(list[i], half ? low : 0.0);
            list[16 + i] = __builtin_fmax(list[16 + i], half ? p[i] : 0.0);
        }
    }
    kn_cross<LN, true>(list);
    kn_merge<LN, true>(list);
}
// The query's threshold, for both its lanes: the score of its knn-th key, or the next number below; the lowest
// number while there is none (what cannot be in a list, minus infinity and what is no number, stays below).
template <int LN>
__device__ __forceinline__ float knn_threshold(const double (&list)[LN], int knn, int half, int lane) {
    const int at = (knn - 1) & (LN - 1);
    uint32_t hi = 0u;
#pragma unroll
    for (int i = 0; i < LN; ++i) hi = i == at ? (uint32_t)(__builtin_bit_cast(u64, list[i]) >> 32) : hi;
    const uint32_t other = lane_xor32<32>(hi, lane);
    if (half != (knn - 1) / LN) hi = other;
    return hi == 0u ? -3.402823466e38f : f32_from_ordered(hi << 1);
}

template <int DT> struct Operand;
template <> struct Operand<RA_BF16> { bf16x8 v[8]; };     // 8 k-steps of 16
template <> struct Operand<RA_F32> { float v[64]; };      // 64 k-steps of 2

// The operand of lane (row = lane % 32, half = lane / 32): dimensions [64*half, 64*half+64)
// of the row. The same assignment is used for keys and queries, so any consistent split of
// the 128 dimensions over k-steps gives the same inner product.
template <int DT>
__device__ __forceinline__ void load_operand(const void* base, int64_t row, int half, Operand<DT>& o) {
    if constexpr (DT == RA_BF16) {
        const uint4* p = reinterpret_cast<const uint4*>(
            reinterpret_cast<const uint16_t*>(base) + row * RA_D + 64 * half);
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const uint4 u = p[s];
            o.v[s] = __builtin_bit_cast(bf16x8, u);
        }
    } else {
        const float4* p = reinterpret_cast<const float4*>(
            reinterpret_cast<const float*>(base) + row * RA_D + 64 * half);
#pragma unroll
        for (int s = 0; s < 16; ++s) {
            const float4 f = p[s];
            o.v[4 * s] = f.x; o.v[4 * s + 1] = f.y; o.v[4 * s + 2] = f.z; o.v[4 * s + 3] = f.w;
        }
    }
}

// A use of every register of an operand (an empty asm statement that only reads them): its loads
// are complete here and cannot sink below later ones. The key stream's waits count loads in
// flight, and an operand load still counted there would turn every one of them into a wait for
// the newest load.
template <int DT>
__device__ __forceinline__ void settle_operand(const Operand<DT>& o) {
    if constexpr (DT == RA_BF16) {
        asm volatile("; operand loaded" ::"v"(o.v[0]), "v"(o.v[1]), "v"(o.v[2]), "v"(o.v[3]), "v"(o.v[4]),
                     "v"(o.v[5]), "v"(o.v[6]), "v"(o.v[7]));
    } else {
#pragma unroll
        for (int s = 0; s < 64; s += 16)
            asm volatile("; operand loaded" ::"v"(o.v[s]), "v"(o.v[s + 1]), "v"(o.v[s + 2]), "v"(o.v[s + 3]),
                         "v"(o.v[s + 4]), "v"(o.v[s + 5]), "v"(o.v[s + 6]), "v"(o.v[s + 7]), "v"(o.v[s + 8]),
                         "v"(o.v[s + 9]), "v"(o.v[s + 10]), "v"(o.v[s + 11]), "v"(o.v[s + 12]),
                         "v"(o.v[s + 13]), "v"(o.v[s + 14]), "v"(o.v[s + 15]));
    }
}

template <int DT>
__device__ __forceinline__ f32x16 block_scores(const Operand<DT>& a, const Operand<DT>& b) {
    f32x16 c = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if constexpr (DT == RA_BF16) {
#pragma unroll
        for (int s = 0; s < 8; ++s)
            c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.v[s], b.v[s], c, 0, 0, 0);
    } else {
#pragma unroll
        for (int s = 0; s < 64; ++s)
            c = __builtin_amdgcn_mfma_f32_32x32x2f32(a.v[s], b.v[s], c, 0, 0, 0);
    }
    return c;
}

// A staged key row keeps its 16-byte chunks at (chunk ^ (row & 15)): the 16 lanes that write one
// row, and the 16 lanes that read the same chunk of 16 consecutive rows, both cover all 64 banks.
// A lane reads the same chunks of the same row (lane % 32, or 32 rows on: same swizzle) in every
// stage, so the byte offsets are computed once (operand_offsets) and a read is one instruction
// with the stage buffer and the block as a constant displacement.
template <int DT> struct OperandAt { int at[DT == RA_BF16 ? 8 : 16]; };
template <int DT>
__device__ __forceinline__ void operand_offsets(int base, int row, int half, OperandAt<DT>& o) {
    constexpr int ROWB = DT == RA_BF16 ? 256 : 512, CPH = ROWB / 32;   // chunks per half row
    const int sw = row & 15;
#pragma unroll
    for (int s = 0; s < CPH; ++s) o.at[s] = base + row * ROWB + (((half * CPH + s) ^ sw) << 4);
}
template <int DT>
__device__ __forceinline__ void read_operand(const unsigned char* lds, const OperandAt<DT>& at, int disp,
                                             Operand<DT>& o) {
    if constexpr (DT == RA_BF16) {
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const uint4 u = *reinterpret_cast<const uint4*>(lds + at.at[s] + disp);
            o.v[s] = __builtin_bit_cast(bf16x8, u);
        }
    } else {
#pragma unroll
        for (int s = 0; s < 16; ++s) {
            const float4 f = *reinterpret_cast<const float4*>(lds + at.at[s] + disp);
            o.v[4 * s] = f.x; o.v[4 * s + 1] = f.y; o.v[4 * s + 2] = f.z; o.v[4 * s + 3] = f.w;
        }
    }
}

// grid: x = block of 32 * WAVES queries, y = graph (seq * n_q + h) - g0. The keys are the first
// n_stream of the graph's stream order. With `scores` the lists' scores are written
// too, for knn_filter.hip, which takes the rest of the stream; with `resume` (first stream position not
// yet seen, per graph and block of resume_queries queries, a multiple of 32) the lists are read from L_out and scores and
// the stream goes on from there.
// LDS: the key ids of KN_IDS stages, then kn_ring stage buffers of STAGE bytes, then the pending runs of the wavefronts.
// LN: keys of its query's list that a lane holds (16 or 32).
// DIRECT: key rows are copied straight to LDS, which asks for 16-byte aligned rows. A caller's K that is not (a view at an odd
// offset) goes through registers, by loads that may be at any element, each waited for before the stage's products: 32 heads x 12000
// keys x 12000 queries 1.99 ms instead of 1.46, float32 4000 x 4000 0.60 instead of 0.57.
template <int DT> constexpr int kn_ring() { return DT == RA_BF16 ? 3 : 2; }      // stage buffers
template <int DT, int WAVES, int LN, int STAGE, bool DIRECT>
__global__ __launch_bounds__(WAVES * RA_WAVE) void knn_kernel(
    const void* __restrict__ K, const void* __restrict__ Q, const u64* __restrict__ order,
    int64_t order_stride, int g0, int n_q, int n_kv, int64_t N, int64_t n_stream, int64_t M, int knn,
    int32_t* __restrict__ L_out, float* __restrict__ scores, const int* __restrict__ resume, int resume_queries,
    int resume_blocks) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    constexpr int QPB = 32 * WAVES;
    constexpr int ROWB = DT == RA_BF16 ? 256 : 512;          // bytes of a key row
    constexpr int CPR = ROWB / 16;                            // 16-byte chunks per row
    constexpr int SROWS = STAGE / ROWB;              // key rows per stage
    constexpr int SBLK = SROWS / 32;                          // 32-key blocks per stage
    constexpr int ND = STAGE / 1024 / WAVES;         // copies of 64 chunks that a wavefront does per stage
    constexpr int RPD = 64 / CPR;                    // rows of one
    constexpr int RING = kn_ring<DT>(), D = RING - 1, IDS = KN_IDS;      // D: stages a copy is ahead
    static_assert(2 * D + 1 < IDS, "a stage's ids are there until it has been multiplied");
    static_assert(IDS * 256 + RING * STAGE <= 1 << 16, "what is copied to LDS lies in its first 64 KB (16 bits of m0)");
    static_assert(SROWS % 32 == 0 && SROWS <= 64, "a stage holds one or two key blocks");
    static_assert(ND * WAVES * 1024 == STAGE, "wavefronts must tile a stage");
    unsigned char* stage_buf = lds_raw + IDS * 256;
    const int tid = threadIdx.x, wv = tid / RA_WAVE, lane = tid % RA_WAVE;
    const int col = lane & 31, half = lane >> 5;
    const int graph = g0 + (int)blockIdx.y, seq = graph / n_q, h = graph % n_q, kvh = h / (n_q / n_kv);
    const size_t esz = DT == RA_BF16 ? 2 : 4;
    const char* Kh = reinterpret_cast<const char*>(K) + ((size_t)seq * n_kv + kvh) * N * RA_D * esz;
    const char* Qh = reinterpret_cast<const char*>(Q) + (size_t)graph * M * RA_D * esz;
    const int64_t q0 = (int64_t)blockIdx.x * QPB + wv * 32;   // first query of this wave
    // the key streamed p-th: the low word of the head's p-th order entry (used as loaded: arithmetic
    // on it would sit right behind the load and wait for it)
    const int* ord = reinterpret_cast<const int*>(order + (size_t)graph * order_stride);
    const int last_pos = (int)n_stream - 1;               // ids and stream positions fit 31 bits

    int64_t st0 = 0, my_st0 = 0;                   // first stage of the workgroup and of this wavefront
    if (resume) {
        int64_t least = n_stream;
        for (int w = 0; w < WAVES; ++w) {
            const int64_t qw = (int64_t)blockIdx.x * QPB + 32 * w;
            const int64_t pos = qw < M ? resume[(size_t)blockIdx.y * resume_blocks + qw / resume_queries] : n_stream;
            if (pos < least) least = pos;
            if (w == wv) my_st0 = pos < n_stream ? pos / SROWS : 0x7fffffff;
        }
        if (least >= n_stream) return;             // (the whole workgroup)
        st0 = least / SROWS;
        my_st0 = __builtin_amdgcn_readfirstlane((int)my_st0);
    }
    // the list of query q0 + col: ranks half * LN + i
    double list[LN];
#pragma unroll
    for (int i = 0; i < LN; ++i) {
        u64 k = 0ull;
        if (resume) {
            const int64_t qr = q0 + col;
            const int e = half * LN + i;
            if (qr < M && e < knn) {
                const float sc = scores[((size_t)blockIdx.y * M + qr) * knn + e];
                if (sc > -INFINITY) k = knn_key(sc, L_out[((size_t)graph * M + qr) * knn + e]);
            }
        }
        list[i] = __builtin_bit_cast(double, k);
    }
    uint32_t* run0 = reinterpret_cast<uint32_t*>(stage_buf + RING * STAGE + wv * KN_RUN_BYTES);
    uint32_t* run = run0 + lane;
    const int* ids_ring = reinterpret_cast<const int*>(lds_raw);       // [IDS][64] key ids of the stages' rows

    Operand<DT> b;                                 // (loads clamped: columns beyond M are never written)
    load_operand<DT>(Qh, q0 + col < M ? q0 + col : M - 1, half, b);
    settle_operand<DT>(b);
    __syncthreads();

    float tau = knn_threshold<LN>(list, knn, half, lane);      // (the lowest number but for a resumed stream)
    int fill = 0;                                  // keys in this lane's pending run

    const int64_t nstage = (n_stream + SROWS - 1) / SROWS;
    // The ids of a stage's rows come D stages before its rows; every wavefront copies them all (the same bytes), so that it needs
    // to wait for its own only. Positions beyond the stream copy the last key again; those are masked or not multiplied.
    const uint32_t lds_at = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds_raw;
    auto copy_ids = [&](int st) __attribute__((always_inline)) {
        const int p = st * SROWS + (lane & (SROWS - 1));
        const int* src = ord + 2 * (size_t)(unsigned)(p < last_pos ? p : last_pos);
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off"
                     ::"s"(__builtin_amdgcn_readfirstlane(lds_at + (st & (IDS - 1)) * 256)), "v"(src) : "m0", "memory");
    };
    auto copy_rows = [&](int st, int buf) __attribute__((always_inline)) {      // buf: st % RING
        int id[ND];
#pragma unroll
        for (int i = 0; i < ND; ++i) id[i] = ids_ring[(st & (IDS - 1)) * 64 + (wv * ND + i) * RPD + lane / CPR];
#pragma unroll
        for (int i = 0; i < ND; ++i) {
            const int row = (wv * ND + i) * RPD + lane / CPR;
            const char* src = Kh + (size_t)(unsigned)id[i] * ROWB + (((lane & (CPR - 1)) ^ (row & 15)) << 4);
            if constexpr (DIRECT)
                asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                             ::"s"(__builtin_amdgcn_readfirstlane(lds_at + IDS * 256 + buf * STAGE + (wv * ND + i) * 1024)), "v"(src)
                             : "m0", "memory");
            else
                *reinterpret_cast<u32x4*>(stage_buf + buf * STAGE + (wv * ND + i) * 1024 + lane * 16) =
                    *reinterpret_cast<const kn_any16*>(src);
        }
    };
    // scores of one 32-key block against the wave's queries, then the selection
    // (kb: the block's place in the stream; block_ids: the ids of its rows)
    auto process = [&](f32x16 cs, int64_t kb, const int* block_ids) __attribute__((always_inline)) {
        const int64_t kbase = kb * 32;
        if (kbase + 32 > n_stream) {               // ragged tail: rows beyond the stream never qualify
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (kbase + (r / 4) * 8 + half * 4 + (r % 4) >= n_stream) cs[r] = -INFINITY;
        }
        float gm[4];
#pragma unroll
        for (int g = 0; g < 4; ++g)
            gm[g] = fmaxf(fmaxf(cs[4 * g], cs[4 * g + 1]), fmaxf(cs[4 * g + 2], cs[4 * g + 3]));
        const float mx = fmaxf(fmaxf(gm[0], gm[1]), fmaxf(gm[2], gm[3]));
        if (__ballot(mx >= tau) == 0ull) return;
        // a lane needs room for the keys of this block that reach its threshold (their number can
        // only fall when a merge raises the threshold)
        int n = 0;
#pragma unroll
        for (int r = 0; r < 16; ++r) n += cs[r] >= tau ? 1 : 0;
        if (__ballot(fill + n > KN_PEND)) {
            knn_fold<LN>(list, run, half, fill);
            tau = knn_threshold<LN>(list, knn, half, lane);
            fill = 0;
        }
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            if (__ballot(gm[g] >= tau) == 0ull) continue;
            const int4 id4 = *reinterpret_cast<const int4*>(block_ids + 8 * g + 4 * half);
            const int id[4] = {id4.x, id4.y, id4.z, id4.w};
            // a lane writes every score to the next free place, and only one that belongs there makes the place taken
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int place = min(fill, KN_PEND);         // (fill itself, for scores that are numbers)
                run[place * 128] = __float_as_uint(cs[4 * g + r]);
                run[place * 128 + 64] = (uint32_t)id[r];
                fill = place + (cs[4 * g + r] >= tau ? 1 : 0);
            }
        }
    };
    OperandAt<DT> a_at;                            // where this lane's key operand sits in a stage buffer
    operand_offsets<DT>((int)(stage_buf - lds_raw), col, half, a_at);
    const int first = (int)st0;
#pragma unroll
    for (int i = 0; i < D; ++i) copy_ids(first + i);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
    for (int i = 0; i < D; ++i) {
        copy_ids(first + D + i);
        copy_rows(first + i, i);
    }
    // Every turn starts the same number of copies, so that "all but those of the last D - 1 turns" are the rows of the next stage and
    // the ids the next turn needs. The loop has one copy of its code (the merge is most of it, and the instruction
    // cache of two compute units is 64 KB).
    constexpr int LEFT = DIRECT ? (D - 1) * (ND + 1) : 0;
    // (lgkmcnt: rows that went through registers are LDS writes, which the barrier does not wait for)
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"i"(LEFT) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    int buf = 0;                                   // of stage st
#pragma unroll 1
    for (int st = first; st < (int)nstage; ++st) {
        copy_ids(st + 2 * D);
        copy_rows(st + D, buf == 0 ? RING - 1 : buf - 1);      // (over stage st - 1, which every wavefront is done with)
        if (st >= (int)my_st0) {                   // (else: keys that this wavefront's queries have seen)
#pragma unroll 1
            for (int k = 0; k < SBLK; ++k) {
                Operand<DT> a;
                read_operand<DT>(lds_raw, a_at, buf * STAGE + k * 32 * ROWB, a);
                // all its reads are on their way before the first product (float32: no registers for that)
                if constexpr (DT == RA_BF16) __builtin_amdgcn_sched_barrier(0);
                // (a block beyond the stream is all masked)
                process(block_scores<DT>(a, b), (int64_t)st * SBLK + k, ids_ring + (st & (IDS - 1)) * 64 + 32 * k);
            }
        }
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"i"(LEFT) : "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        buf = buf == RING - 1 ? 0 : buf + 1;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // nothing is left on its way to LDS
    // write ids and scores, best first, a query's list at a time, through the runs' place (word of rank e of query col at
    // 32 e + (col ^ e % 32): a rank of the 32 queries, like 32 ranks of a query, is in different banks)
    knn_fold<LN>(list, run, half, fill);
    static_assert(2 * LN * 32 * 4 <= KN_RUN_BYTES, "the lists' words fit the runs' place");
    for (int what = 0; what < (scores ? 2 : 1); ++what) {
        kn_wave_sync();
#pragma unroll
        for (int i = 0; i < LN; ++i) {
            const u64 k = __builtin_bit_cast(u64, list[i]);
            const uint32_t word = what == 0 ? (uint32_t)knn_key_id(k)
                                            : __float_as_uint(k == 0ull ? -INFINITY : knn_key_score(k));
            run0[32 * (half * LN + i) + (col ^ (i & 31) ^ (LN == 16 ? 16 * half : 0))] = word;
        }
        kn_wave_sync();
        for (int jq = 0; jq < 32; ++jq) {
            const int64_t qr = q0 + jq;
            if (qr >= M) break;
            if (lane < knn) {
                const uint32_t word = run0[32 * lane + (jq ^ (lane & 31))];
                if (what == 0) L_out[((size_t)graph * M + qr) * knn + lane] = (int)word;
                else scores[((size_t)blockIdx.y * M + qr) * knn + lane] = __uint_as_float(word);      // (the filter goes on with these)
            }
        }
    }
}

// graphs [g0, g0 + n_graphs) of the call
struct KnnCall {
    const void *K, *Q, *order;
    int g0, n_graphs, n_q, n_kv;
    int64_t N, n_stream, M;
    int knn;
    int32_t* L;
    float* scores;
    hipStream_t st;
    const int* resume;
    int resume_queries, resume_blocks;
};
template <int DT, int WAVES, int LN, int STAGE, bool DIRECT>
static ra_status knn_launch_as(const KnnCall& c) {
    constexpr int QPB = 32 * WAVES;
    const size_t lds = WAVES * KN_RUN_BYTES + kn_ring<DT>() * STAGE + KN_IDS * 256;
    RA_LDS_OPT_IN((knn_kernel<DT, WAVES, LN, STAGE, DIRECT>), lds);
    const dim3 grid((unsigned)((c.M + QPB - 1) / QPB), (unsigned)c.n_graphs);
    hipLaunchKernelGGL((knn_kernel<DT, WAVES, LN, STAGE, DIRECT>), grid, dim3(WAVES * RA_WAVE), lds, c.st, c.K, c.Q,
                       reinterpret_cast<const u64*>(c.order), ra_knn_order_stride(c.N), c.g0, c.n_q, c.n_kv, c.N,
                       c.n_stream, c.M, c.knn, c.L, c.scores, c.resume, c.resume_queries, c.resume_blocks);
    RA_HIP(hipGetLastError());
    return RA_OK;
}

// RA_TEST_KNN_SELECTION (ra_test_configure): whether the 8-bit products take the rest of the stream
static int g_knn_selection_override = RA_TEST_KNN_AUTO;
void ra_knn_set_selection_override(int v) { g_knn_selection_override = v; }
// RA_TEST_KNN_RESUME: where to, and how much is there
static int* g_knn_resume_copy = nullptr;
static size_t g_knn_resume_copied = 0;
void ra_knn_set_resume_copy(int* to) {
    g_knn_resume_copy = to;
    g_knn_resume_copied = 0;
}
static ra_status knn_copy_resume(const KnnCall& c) {
    const size_t n = (size_t)c.n_graphs * c.resume_blocks;
    if (!g_knn_resume_copy || g_knn_resume_copied + n > RA_TEST_KNN_RESUME_INTS) return RA_OK;
    RA_HIP(hipMemcpyAsync(g_knn_resume_copy + g_knn_resume_copied, c.resume, n * sizeof(int), hipMemcpyDeviceToDevice, c.st));
    g_knn_resume_copied += n;
    return RA_OK;
}

// bf16: 8 wavefronts per workgroup (two per SIMD: registers). fp32 operands take twice the registers: 4 wavefronts.
template <bool DIRECT>
static ra_status knn_launch_to(const KnnCall& c, ra_dtype dt) {
    if (dt == RA_BF16)
        return c.knn <= 32 ? knn_launch_as<RA_BF16, 8, 16, 16384, DIRECT>(c) : knn_launch_as<RA_BF16, 8, 32, 16384, DIRECT>(c);
    return c.knn <= 32 ? knn_launch_as<RA_F32, 4, 16, 16384, DIRECT>(c) : knn_launch_as<RA_F32, 4, 32, 16384, DIRECT>(c);
}
static ra_status knn_launch(const KnnCall& c, ra_dtype dt) {
    return reinterpret_cast<uintptr_t>(c.K) % 16 == 0 ? knn_launch_to<true>(c, dt) : knn_launch_to<false>(c, dt);
}

// Keys of the stream that are multiplied as they are before knn_filter.hip takes over (N: all of them): enough that
// thresholds are near final for queries with much in common (in the filter a kept key costs about ten ruled-out
// ones; where it keeps too many it gives up, and is tried again after an eighth of the stream). bf16: a
// thirty-second of the stream and at least 4096. float32, whose products cost sixteen times as much: a sixty-fourth
// and at least sixteen times a list's length. The filter pays where what it saves on N x M products exceeds what packing
// N keys and M queries and the larger scratch allocation cost. Whole calls of ra_knn, lists of 32, ms without -> with:
//   bf16, 32 heads: 8K keys x 8K queries 0.78 -> 1.12; 16K x 4K 0.78 -> 1.04, x 16K 2.43 -> 2.10; 32K x 4K 1.38 -> 1.41, x
//     32K 8.3 -> 4.6; 128K x 2K 2.92 -> 2.94, x 32K 31.9 -> 12.1.
//   bf16, fewer heads: 4 heads, 16K x 16K 0.40 -> 0.48; 8 heads, 64K x 64K 8.1 -> 3.8.
//   bf16, first keys 1024 / 2048 / 4096 / 8192: 32K x 32K x 32 4.83 / 4.86 / 4.91 / 5.34; 128K x 64K x 4 of the mixture law, lists
//     of 48: 11.8 / 11.5 / 10.5 / 10.3.
//   float32: 32 heads, 2K x 2K 0.37 -> 0.35, 4K x 4K 1.24 -> 0.56, 16K x 4K 4.3 -> 1.23; 8 heads, 8K x 8K 1.18 -> 0.47; one head with 512
//     queries gains from 8K keys on (0.65 -> 0.30). First keys 512 / as below / 2048: 16K x 4K x 32 1.23 / 1.25 / 1.52; 64K x 8K x 8
//     1.46 / 1.47 / 1.55; lists of 64, 16K x 8K x 8 1.00 / 0.69 / 0.79.
// What decides in bf16 is the number of queries in all heads together, about 100K from 48K keys on and 260K below; the
// line takes the queries of one head below 48K keys (32 heads: the same) and none from there on, which
// costs calls with few queries up to 0.1 ms. In float32 the number of products decides below 8K keys.
static int64_t knn_first_keys(ra_dtype dt, int graphs, int64_t N, int64_t M, int knn) {
    if (g_knn_selection_override == RA_TEST_KNN_LDS) return N;
    if (g_knn_selection_override == RA_TEST_KNN_FILTER) return N > 128 ? 128 : N;
    if (dt == RA_BF16) {
        if (N < 16384 || (N < 49152 && M < 8192)) return N;
        const int64_t first = N / 32 > 4096 ? N / 32 : 4096;
        return (first + 127) & ~(int64_t)127;
    }
    if (N < 2048 || (N < 8192 && (double)graphs * N * M < 1e8)) return N;
    const int64_t first = N / 64 > 16 * knn ? N / 64 : 16 * knn;
    return (first + 127) & ~(int64_t)127;
}
// graphs whose 8-bit copies and scores are in memory at one time
static int knn_graphs_at_once(int graphs, int64_t N, int64_t M, int knn) {
    const size_t one = ra_knn_filter_bytes(1, N, M, knn), most = (size_t)3 << 29;
    const size_t fit = most / one < 1 ? 1 : most / one;
    const int calls = (int)((graphs + fit - 1) / fit);
    return (graphs + calls - 1) / calls;
}
static size_t align_256(size_t x) { return (x + 255) & ~(size_t)255; }

// the stream order, then (where the filter is used, and not `plain`) the column maxima of the KV heads and
// the filter's own workspace
size_t ra_knn_workspace_bytes(ra_dtype dt, int n_seq, int n_q, int n_kv, int64_t N, int64_t M, int knn, bool plain) {
    const int graphs = n_seq * n_q;
    size_t b = align_256(ra_knn_order_bytes(graphs, N));
    if (!plain && knn_first_keys(dt, graphs, N, M, knn) < N)
        b += align_256((size_t)n_seq * n_kv * RA_D * 4) +
             ra_knn_filter_bytes(knn_graphs_at_once(graphs, N, M, knn), N, M, knn);
    return b;
}

ra_status ra_launch_knn(const void* K, const void* Q, ra_dtype dt, int n_seq, int n_q, int n_kv,
                        int64_t N, int64_t M, int knn, void* workspace, size_t workspace_bytes, hipStream_t st,
                        int32_t* L) {
    // the order the keys are streamed in (knn_order.hip), at the start of the workspace
    ra_status rc = ra_launch_knn_order(K, Q, dt, n_seq, n_q, n_kv, N, M, workspace, st);
    if (rc != RA_OK) return rc;
    const int graphs = n_seq * n_q;
    // (without room for the 8-bit copies the whole stream is multiplied as it is: the same lists)
    const bool room = workspace_bytes >= ra_knn_workspace_bytes(dt, n_seq, n_q, n_kv, N, M, knn, false);
    const int64_t first = room ? knn_first_keys(dt, graphs, N, M, knn) : N;
    KnnCall c{K, Q, workspace, 0, graphs, n_q, n_kv, N, first, M, knn, L, nullptr, st, nullptr, 0, 0};
    if (first == N) return knn_launch(c, dt);
    char* ws = reinterpret_cast<char*>(workspace) + align_256(ra_knn_order_bytes(graphs, N));
    uint32_t* maxabs = reinterpret_cast<uint32_t*>(ws);
    ws += align_256((size_t)n_seq * n_kv * RA_D * 4);
    rc = ra_launch_knn_filter_scales(K, dt, n_seq * n_kv, N, maxabs, st);
    const int most = knn_graphs_at_once(graphs, N, M, knn);
    for (int g0 = 0; g0 < graphs && rc == RA_OK; g0 += most) {
        c.g0 = g0;
        c.n_graphs = graphs - g0 < most ? graphs - g0 : most;
        c.scores = ra_knn_filter_scores(ws, c.n_graphs, N, M, knn);
        c.n_stream = first;
        c.resume = nullptr;
        rc = knn_launch(c, dt);
        if (rc != RA_OK) return rc;
        // The filter goes to an eighth of the stream, then to the end; what gives up goes on here to the same place. (When only what had
        // given up came back for the second part, the others having gone to the end at once, a launch of a few workgroups
        // took as long again: 4 heads of the mixture law, 287754 keys, 64K queries, lists of 32 22.8 ms, now 17.0, and 1M keys 39.7 and 40.0. With a third
        // part up to a thirty-second, which only float32 streams of a multiple of 8192 keys had, 8192 queries, 64K
        // keys 3.50 ms, without 3.25, 128K 5.01 and 4.83.)
        int64_t from = first;
        for (int more : {8, 1}) {
            const int64_t next = more == 1 ? N : first + (N / more - first + KN_FILTER_SEGMENT - 1) / KN_FILTER_SEGMENT * KN_FILTER_SEGMENT;
            if (more > 1 && (N / more < 2 * from || next >= N)) continue;
            rc = ra_launch_knn_filter(K, Q, dt, workspace, graphs, g0, c.n_graphs, n_q, n_kv, N, M, knn, first, from, next, maxabs, ws,
                                      st, L, &c.resume, &c.resume_queries, &c.resume_blocks);
            if (rc == RA_OK) rc = knn_copy_resume(c);
            if (rc != RA_OK) return rc;
            c.n_stream = from = next;
            rc = knn_launch(c, dt);
            if (rc != RA_OK) return rc;
        }
    }
    return rc;
}
