// VectorSearch(q) of Algorithm 1: bounded best-first walk over one head's key graph
// (Sec. 2.4 describes proximity-graph search as a greedy walk towards the most similar
// vectors). One workgroup per (sequence, query head), of 1024, 512 or 256 threads (search_threads
// below, for the stand-alone and the fused launch); the whole search state lives in LDS:
//   * visited: an exact bitset over the N keys (N/8 bytes; a global-memory bitset is used
//     instead when the context is too long for LDS),
//   * beam: at most ef entries, always sorted, as 64-bit keys
//         [ordered(score) : 32][0x7fffffff - id : 31][not-yet-expanded : 1]
//     so that "larger key" is exactly "(score descending, id ascending)" and one integer
//     compare decides; ids are unique in the beam, so the flag bit never decides.
// A walk of narrow steps is bound by the length of a step's dependent chain: LDS round trips, a trip to
// L2 for the adjacency rows and one to memory for the key rows, barriers, and on the way every
// instruction, taken branches above all: there are one or two wavefronts per SIMD to hide them. So the
// common step is laid out as straight code (__builtin_expect), what the next phase needs first is read
// along with the counter that says how much of it there is, and key rows take as few trips as they can.
// 16 picks per step over 64K keys: 68.6 -> 51.1 us; one pick per step: 248 -> 185 us.
// Each step expands the `expand` best unexpanded entries at once: their adjacency rows
// are read with one coalesced load per row, unvisited neighbours are claimed with an LDS
// atomic-or (which also removes duplicates), their key rows are gathered by 16-lane
// groups (16 B per lane; four rows per wavefront load), scored, filtered against the
// beam's worst entry, and merged into the beam by rank: a kept candidate's place is the
// number of beam entries above it (a search) plus the number of candidates above it
// (counted); a beam entry's place is its index plus a prefix sum over the candidates' slots.
// No sort, no serial insertion, and the next step's picks fall out of the same numbers. The
// beam after a step is the top-ef of a set union, so it does not depend on the order in which
// candidates were claimed.
//
// Scores decide integer results, so every kernel that ranks keys (this walk, the flat scan, the
// re-rank) computes them in one and the same way: each of 16 lanes sums its 8 contiguous products,
// then the 16 partial sums are added pairwise over adjacent lanes (xor 1, 2, 4, 8). Identical key
// rows therefore score identically everywhere. fp32 keys and 8-bit keys: product rounded, then
// added, left to right (a CPU reference can reproduce every bit). bf16 keys: four two-element dot
// instructions per lane (exact products, the hardware's own accumulation).
#pragma once
#include "common.h"

#define SR_THREADS 1024          // largest workgroup; the kernels are also built for 512 and 256 threads
// Wavefronts per SIMD that the kernels leave registers for: two workgroups of 512 threads, or four of 256, share a compute unit, in
// float32 three of 256. (Where searches outnumber the compute units, that is what counts: with 136 registers per lane in place
// of 128, 448 searches of 33K keys, ef 512, took 206 us instead of 134.)
#define SR_WAVES(KT, T) ((KT) != RA_F32 || (T) == 1024 ? 4 : 3)
#define SR_LDS_LIMIT RA_LDS_LIMIT
#define SR_BITSET_LDS_MAX (128 * 1024) // a longer visited bitset (over 2^20 keys) lives in global memory
#ifndef SR_UNROLL
#define SR_UNROLL 8               // key rows in flight per 16-lane group
#endif
#ifndef SR_ADJ_LOADS
#define SR_ADJ_LOADS 8            // adjacency cells a thread has in flight while it claims neighbours
#endif


enum { C_MISSED = 0, C_LO = 1, C_HI = 2, C_NSURV = 3, C_BIN = 4, C_STEP = 5, C_STEP2 = 8, C_WTOT = 11,
       C_COUNT = C_WTOT + SR_THREADS / RA_WAVE };
enum { S_NCAND = 0, S_NKEEP = 1, S_NUNEXP = 2 };      // of the three words at C_STEP and at C_STEP2
#define SR_TOUCH_BYTES (4 * RA_WAVE) // where touched words land (touch_line)
#define SR_PREFILTER_SLACK 64     // a step that keeps more than ef + this many candidates drops the hopeless ones first
#define SR_PREFILTER_REGS 8       // ... when a thread can hold its share of them (nk <= 8 T)
#define SR_START_REGS 8           // keys of a start set that a thread can hold
// A merge of up to SR_NARROW candidates takes one phase, with 1024 threads of up to twice as many; one of more than SR_DIRECT goes
// through buckets. (Geometric means over settings of 32 heads of 32K keys. Up to 512 threads, 170 settings: limits 8 and 32 instead
// of 16 +1.4 and -0.3 %. 1024 threads, 66 settings, beams of 384 to 2048: 24 and 64 instead of 32 +0.5 and +1.7 %; 8, with every
// candidate compared with every entry, +7 %. Buckets from 33 and 129 candidates on: +1.8 and -0.7 %, up to 512 threads 0 and 0 %.)
#define SR_NARROW 16
#define SR_DIRECT 64
#define SR_MERGE_REGS 2           // ... when a thread can hold its share of them
#define SR_LIST_AT (T <= 512 ? 512 : T)       // words of cid in front of the new cells of a seed set's first picks
#define SR_FRESH_CELLS 16         // a pick with more new cells than this has its whole row read, and so have all others (4, 64: the same times)

typedef unsigned long long u64;

// Phase clocks for tuning builds (-DSR_PHASE_CLOCKS): thread 0 of the workgroups of the first 64 searches adds the
// ticks spent in each phase to a device array that ra_dbg_phase_ticks copies out. Off otherwise.
#ifdef SR_PHASE_CLOCKS
#define SR_NPHASE 16
#define SR_NITER 16
static __device__ long long sr_phase_ticks[64 * SR_NITER * SR_NPHASE];
#ifdef SR_WAVE_CLOCKS
// (with -DSR_WAVE_CLOCKS: wall-clock stamps of the first head's workgroup, [0..3] search entered,
// state cleared, claims made, start set's keys in LDS, and of the first and last of its seed
// workgroups, [8..11] and [16..19]: entered, header read, first rows scored, first keys stored; [24..31]
// every 128th key taken; [32..] keys stored by each wavefront of each seed workgroup; ra_dbg_wave_ticks
// copies SR_NWAVE of them out)
#define SR_NWAVE (32 + 8 * RA_SEED_PARTS_MAX)
static __device__ long long sr_wave_ticks[SR_NWAVE];
#endif
// ticks are added up in LDS (a fire-and-forget add) and copied out when the search has ended
#define SR_TICK_INIT                                                                           \
    __shared__ long long tick_lds_[SR_NITER * SR_NPHASE];                                      \
    for (int i_ = threadIdx.x; i_ < SR_NITER * SR_NPHASE; i_ += blockDim.x) tick_lds_[i_] = 0; \
    __syncthreads();                                                                           \
    long long tick_ = clock64(); int tick_it_ = 0
#define SR_TICK_ITER(i) tick_it_ = (i) < SR_NITER ? (i) : SR_NITER - 1
#define SR_TICK(p)                                                                             \
    do {                                                                                       \
        if (threadIdx.x == 0) {                                                                \
            const long long now_ = clock64();                                                  \
            tick_lds_[tick_it_ * SR_NPHASE + (p)] += now_ - tick_;                             \
            tick_ = now_;                                                                      \
        }                                                                                      \
    } while (0)
#define SR_TICK_FLUSH                                                                          \
    do {                                                                                       \
        if (head < 64)                                                                         \
            for (int i_ = threadIdx.x; i_ < SR_NITER * SR_NPHASE; i_ += blockDim.x)            \
                sr_phase_ticks[head * SR_NITER * SR_NPHASE + i_] += tick_lds_[i_];             \
    } while (0)
#else
#define SR_TICK_INIT
#define SR_TICK_ITER(i)
#define SR_TICK(p)
#define SR_TICK_FLUSH
#endif

template <int V> struct sr_int { static constexpr int value = V; };      // a compile-time row count as an argument

__device__ __forceinline__ u64 make_key(float score, int id) {
    return ((u64)f32_ordered(score) << 32) | ((u64)(uint32_t)(0x7fffffff - id) << 1) | 1ull;
}
// what lane l holds
__device__ __forceinline__ u64 lane_key(u64 k, int l) {
    return (u64)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(k >> 32), l) << 32 |
           (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)k, l);
}
__device__ __forceinline__ int key_id(u64 k) { return 0x7fffffff - (int)((uint32_t)k >> 1); }

template <int DT>
__device__ __forceinline__ void load_q8(const void* q, int lane16, float* qv) {
    if (DT == RA_BF16) {
        const uint4 u = reinterpret_cast<const uint4*>(q)[lane16];
        qv[0] = bf16_lo(u.x); qv[1] = bf16_hi(u.x); qv[2] = bf16_lo(u.y); qv[3] = bf16_hi(u.y);
        qv[4] = bf16_lo(u.z); qv[5] = bf16_hi(u.z); qv[6] = bf16_lo(u.w); qv[7] = bf16_hi(u.w);
    } else {
        const float4 a = reinterpret_cast<const float4*>(q)[lane16 * 2];
        const float4 b = reinterpret_cast<const float4*>(q)[lane16 * 2 + 1];
        qv[0] = a.x; qv[1] = a.y; qv[2] = a.z; qv[3] = a.w;
        qv[4] = b.x; qv[5] = b.y; qv[6] = b.z; qv[7] = b.w;
    }
}

// A lane's share of the query in the form the score wants it: bf16 pairs stay packed (they go
// through the two-element dot instruction), fp32 queries and queries over 8-bit keys are floats.
template <int KT> struct ScoreQuery { float v[8]; };
template <> struct ScoreQuery<RA_BF16> { uint4 p; };
template <int DT, int KT>
__device__ __forceinline__ void load_score_query(const void* qrow, int lane16, ScoreQuery<KT>& sq) {
    if constexpr (KT == RA_BF16) sq.p = reinterpret_cast<const uint4*>(qrow)[lane16];
    else load_q8<DT>(qrow, lane16, sq.v);
}

// Raw 32 B (fp32) / 16 B (bf16) of a key row owned by this lane.
template <int DT> struct RowBits { uint4 a; uint4 b; };

template <int DT>
__device__ __forceinline__ RowBits<DT> load_key(const void* Kh, int64_t row, int lane16) {
    RowBits<DT> r;
    if (DT == RA_KEYS_I8) {
        // 8 of the row's 128 signed bytes
        const uint2 u = reinterpret_cast<const uint2*>(reinterpret_cast<const int8_t*>(Kh) + row * RA_D)[lane16];
        r.a = make_uint4(u.x, u.y, 0u, 0u);
        r.b = r.a;
    } else if (DT == RA_BF16) {
        r.a = reinterpret_cast<const uint4*>(reinterpret_cast<const uint16_t*>(Kh) + row * RA_D)[lane16];
        r.b = r.a;
    } else {
        const uint4* p = reinterpret_cast<const uint4*>(reinterpret_cast<const float*>(Kh) + row * RA_D);
        r.a = p[lane16 * 2];
        r.b = p[lane16 * 2 + 1];
    }
    return r;
}

// The same for a kernel that streams every row once (a scan): non-temporal loads, which leave the
// caches to data that is read again (measured on a plain read of 1 GiB: 7.1 against 6.2 TB/s). Not in float32, where two
// instructions touch the same cache lines and the second would fetch them again (layers in turn, us per layer: 8 KV heads, 60001
// tokens 70 -> 64, 20001 tokens 43 -> 37; one head, 400000 66 -> 61, 5000 21 -> 16).
typedef unsigned int ra_u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int ra_u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint4 load16_stream(const void* p) {
    const ra_u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const ra_u32x4*>(p));
    return make_uint4(v.x, v.y, v.z, v.w);
}
template <int DT>
__device__ __forceinline__ RowBits<DT> load_key_stream(const void* Kh, int64_t row, int lane16) {
    RowBits<DT> r;
    if (DT == RA_KEYS_I8) {
        const ra_u32x2 u = __builtin_nontemporal_load(
            reinterpret_cast<const ra_u32x2*>(reinterpret_cast<const int8_t*>(Kh) + row * RA_D) + lane16);
        r.a = make_uint4(u.x, u.y, 0u, 0u);
        r.b = r.a;
    } else if (DT == RA_BF16) {
        r.a = load16_stream(reinterpret_cast<const uint4*>(reinterpret_cast<const uint16_t*>(Kh) + row * RA_D) + lane16);
        r.b = r.a;
    } else {
        r = load_key<DT>(Kh, row, lane16);
    }
    return r;
}

template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}

// The fixed-order inner product described in the file header, in two parts: a lane's share (its 8
// dimensions, summed left to right), then the pairwise tree over the 16 lanes of the group.
typedef __bf16 sr_bf16x2 __attribute__((ext_vector_type(2)));
template <int DT>
__device__ __forceinline__ float score_share(const RowBits<DT>& r, const ScoreQuery<DT>& sq) {
    float acc;
    if constexpr (DT == RA_KEYS_I8) {
        const float* qv = sq.v;
        // qv holds query * scale; the key bytes convert to float32 exactly; product rounded, then added
        acc = __fmul_rn(qv[0], (float)(int8_t)(r.a.x));
        acc = __fadd_rn(acc, __fmul_rn(qv[1], (float)(int8_t)(r.a.x >> 8)));
        acc = __fadd_rn(acc, __fmul_rn(qv[2], (float)(int8_t)(r.a.x >> 16)));
        acc = __fadd_rn(acc, __fmul_rn(qv[3], (float)(int8_t)(r.a.x >> 24)));
        acc = __fadd_rn(acc, __fmul_rn(qv[4], (float)(int8_t)(r.a.y)));
        acc = __fadd_rn(acc, __fmul_rn(qv[5], (float)(int8_t)(r.a.y >> 8)));
        acc = __fadd_rn(acc, __fmul_rn(qv[6], (float)(int8_t)(r.a.y >> 16)));
        acc = __fadd_rn(acc, __fmul_rn(qv[7], (float)(int8_t)(r.a.y >> 24)));
    } else if constexpr (DT == RA_BF16) {
        // four two-element dot instructions (exact products, float32 accumulation in the hardware's
        // own rounding: within an ulp of the running sum per instruction, the same bits for the same
        // operands): 4 vector instructions per row share instead of 8 conversions and 8 fma
        acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(sr_bf16x2, sq.p.x), __builtin_bit_cast(sr_bf16x2, r.a.x), 0.f, false);
        acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(sr_bf16x2, sq.p.y), __builtin_bit_cast(sr_bf16x2, r.a.y), acc, false);
        acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(sr_bf16x2, sq.p.z), __builtin_bit_cast(sr_bf16x2, r.a.z), acc, false);
        acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(sr_bf16x2, sq.p.w), __builtin_bit_cast(sr_bf16x2, r.a.w), acc, false);
    } else {
        const float* qv = sq.v;
        // product rounded, then added (this file is compiled with contraction off)
        acc = __fmul_rn(qv[0], __uint_as_float(r.a.x));
        acc = __fadd_rn(acc, __fmul_rn(qv[1], __uint_as_float(r.a.y)));
        acc = __fadd_rn(acc, __fmul_rn(qv[2], __uint_as_float(r.a.z)));
        acc = __fadd_rn(acc, __fmul_rn(qv[3], __uint_as_float(r.a.w)));
        acc = __fadd_rn(acc, __fmul_rn(qv[4], __uint_as_float(r.b.x)));
        acc = __fadd_rn(acc, __fmul_rn(qv[5], __uint_as_float(r.b.y)));
        acc = __fadd_rn(acc, __fmul_rn(qv[6], __uint_as_float(r.b.z)));
        acc = __fadd_rn(acc, __fmul_rn(qv[7], __uint_as_float(r.b.w)));
    }
    return acc;
}
// All 16 lanes of the group return the same value.
template <int DT>
__device__ __forceinline__ float score_fixed(const RowBits<DT>& r, const ScoreQuery<DT>& sq) {
    float acc = score_share<DT>(r, sq);
    // pairwise tree over adjacent lanes with DPP lane permutations inside a row of 16:
    // quad_perm [1,0,3,2] and [2,3,0,1] are xor 1 and xor 2; after them the four lanes of a
    // quad hold the same sum, so half-mirror (i -> 7-i) and mirror (i -> 15-i) deliver exactly
    // what xor 4 and xor 8 would, and float addition commutes.
    acc = __fadd_rn(acc, dpp_f32<0xB1>(acc));
    acc = __fadd_rn(acc, dpp_f32<0x4E>(acc));
    acc = __fadd_rn(acc, dpp_f32<0x141>(acc));
    acc = __fadd_rn(acc, dpp_f32<0x140>(acc));
    return acc;
}

// The same tree for R rows at once (R = 1, 2, 4, 8 or 16 shares per lane): at level k a lane and its
// partner (lane ^ 2^k) split the rows they both still hold, each adding the partner's share of the
// rows it keeps, so the work halves per level instead of every lane adding up every row; once one
// row is left the remaining levels add as in score_fixed. Lane l of the group ends with the sum of
// row l & (R - 1): the same operands added in the same pairs as in score_fixed, hence the same bits.
// Partner values: quad_perm for xor 1 and 2, a row rotation by 8 for xor 8, and for xor 4 two
// row shifts by 4, each written to the banks of four lanes it is right for.
template <int K>
__device__ __forceinline__ float lane16_xor(float x) {
    if constexpr (K == 0) return dpp_f32<0xB1>(x);
    else if constexpr (K == 1) return dpp_f32<0x4E>(x);
    else if constexpr (K == 3) return dpp_f32<0x128>(x);
    else {
        const int v = __float_as_int(x);
        int t = __builtin_amdgcn_update_dpp(v, v, 0x104, 0xF, 0x5, false);      // lanes 0-3, 8-11 <- lane + 4
        t = __builtin_amdgcn_update_dpp(t, v, 0x114, 0xF, 0xA, false);          // lanes 4-7, 12-15 <- lane - 4
        return __int_as_float(t);
    }
}
template <int K, int N>
__device__ __forceinline__ void rows_tree_level(float* a, int lane16) {
    if constexpr (N > 1) {
        const bool hi = (lane16 >> K) & 1;
#pragma unroll
        for (int j = 0; j < N / 2; ++j) {
            const float keep = hi ? a[2 * j + 1] : a[2 * j];
            const float send = hi ? a[2 * j] : a[2 * j + 1];
            a[j] = __fadd_rn(keep, lane16_xor<K>(send));
        }
    } else {
        a[0] = __fadd_rn(a[0], lane16_xor<K>(a[0]));
    }
}
template <int R>
__device__ __forceinline__ float rows_tree(float (&a)[R], int lane16) {
    static_assert(R == 1 || R == 2 || R == 4 || R == 8 || R == 16, "a power of two up to the lanes of a group");
    rows_tree_level<0, R>(a, lane16);
    rows_tree_level<1, (R > 1 ? R / 2 : 1)>(a, lane16);
    rows_tree_level<2, (R > 2 ? R / 4 : 1)>(a, lane16);
    rows_tree_level<3, (R > 4 ? R / 8 : 1)>(a, lane16);
    return a[0];
}

// Inclusive prefix sum over the 64 lanes of a wavefront (all lanes active): shifts inside each
// row of 16 lanes, then lane 15 of a row added to the next row, then lane 31 to the upper half.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int dpp_or_zero(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, ROW_MASK, 0xF, false);
}
__device__ __forceinline__ int wave_incl_scan(int v) {
    v += dpp_or_zero<0x111, 0xF>(v);      // row_shr:1
    v += dpp_or_zero<0x112, 0xF>(v);      // row_shr:2
    v += dpp_or_zero<0x114, 0xF>(v);      // row_shr:4
    v += dpp_or_zero<0x118, 0xF>(v);      // row_shr:8
    v += dpp_or_zero<0x142, 0xA>(v);      // row_bcast:15 into rows 1 and 3
    v += dpp_or_zero<0x143, 0xC>(v);      // row_bcast:31 into rows 2 and 3
    return v;
}

// Smallest lo and largest hi of the wavefront, in lane 63 (lane permutations inside the rows of 16, then the
// rows: no trips through LDS).
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ void min_max_step(uint32_t& lo, uint32_t& hi) {
    lo = min(lo, (uint32_t)__builtin_amdgcn_update_dpp((int)lo, (int)lo, CTRL, ROW_MASK, 0xF, false));
    hi = max(hi, (uint32_t)__builtin_amdgcn_update_dpp((int)hi, (int)hi, CTRL, ROW_MASK, 0xF, false));
}
__device__ __forceinline__ void wave_min_max(uint32_t& lo, uint32_t& hi) {
    min_max_step<0xB1, 0xF>(lo, hi);
    min_max_step<0x4E, 0xF>(lo, hi);
    min_max_step<0x141, 0xF>(lo, hi);
    min_max_step<0x140, 0xF>(lo, hi);
    min_max_step<0x142, 0xA>(lo, hi);        // lane 15 of a row into the next one, then lane 31 to the upper half
    min_max_step<0x143, 0xC>(lo, hi);
}

// 256 equal-width bins of scores between the smallest and the largest: bin = (score - lowest) * 255 / (highest - lowest), truncated.
// Every operation is monotone in the score, so a larger score never lands in a lower bin. Non-finite scores (from non-finite inputs)
// leave the factor at zero: one bin.
struct ScoreBins {
    float lowest, to_bin;
    __device__ __forceinline__ ScoreBins(uint32_t lo, uint32_t hi) : lowest(f32_from_ordered(lo)) {
        const float width = f32_from_ordered(hi) - lowest;
        to_bin = width > 0.f && width < INFINITY ? 255.0f / width : 0.f;
    }
    __device__ __forceinline__ int bin(u64 key) const {
        const float b = (f32_from_ordered((uint32_t)(key >> 32)) - lowest) * to_bin;
        return b >= 255.f ? 255 : b > 0.f ? (int)b : 0;
    }
};

// A head's row of the seed sets: [0] the number of ids, [1] 0, then places for n ids, then for n masks of 32 or, where the degree is
// above 32, 64 bits (lower half first): of the cells of the id's adjacency row, those whose neighbour is no member of the set.
__host__ __device__ static inline int seed_mask_words(int deg) { return deg > 32 ? 2 : 1; }
__host__ __device__ static inline int seed_row_words(int n, int deg) { return 2 + n * (1 + seed_mask_words(deg)); }
__host__ __device__ static inline int seed_places(int row_words, int deg) { return (row_words - 2) / (1 + seed_mask_words(deg)); }

static_assert(RA_MAX_EF + RA_MAX_EXPAND * RA_MAX_DEG < 65536, "ranks and merge counts are kept in 16 bits");

// Workgroup -> (sequence, query head). Consecutive workgroup ids are dealt round-robin to the 8
// XCDs, each with its own L2. The query heads of a GQA group read the same key and value rows, so
// they are given workgroup ids that are congruent modulo 8 (group + n_groups * member) and share
// one L2, whenever the number of groups is a multiple of 8; otherwise the identity map is used.
__device__ __forceinline__ int xcd_aware_head(int block, int heads, int G) {
    const int n_groups = heads / G;
    if (G == 1 || (n_groups & 7)) return block;
    return (block % n_groups) * G + block / n_groups;
}

// Sets key id's bit of the visited set and returns the word as it was. One workgroup owns the bitset, in
// LDS or in device memory, so workgroup scope is enough (and the workgroup clears it itself: no launch
// ahead of the walk).
__device__ __forceinline__ uint32_t claim_key(uint32_t* bits, int id) {
    return __hip_atomic_fetch_or(&bits[id >> 5], 1u << (id & 31), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Brings p's line into this XCD's L2 (p 4-byte aligned, in bounds): a load of one word that goes straight to
// LDS, to 4 bytes per lane at lds_off that nothing reads, so that no register waits for it. (Ordinary loads
// whose words fed a test that never held were waited for when the walk's loop turned: 700 of 7500 ticks
// of a step that expands 16 nodes.) A wavefront waits for its own before it ends.
__device__ __forceinline__ void touch_line(const void* p, uint32_t lds_off) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" ::"s"(lds_off), "v"(p) : "m0");
}

// The same for p that is only 2-byte aligned.
__device__ __forceinline__ void touch_line_of_halves(const void* p, uint32_t lds_off) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_ushort %1, off" ::"s"(lds_off), "v"(p) : "m0");
}

__device__ __forceinline__ void end_touches() { __builtin_amdgcn_s_waitcnt(0x0F70); }      // vmcnt(0)

// Claims L neighbours per lane and appends those not visited before to cid, `n_claimed` of them so far; bit_word(id) is the word of the
// visited set that has id's bit, wanted(id) whether id is to be claimed here. All claims are on their way before the first
// result is looked at, and a wavefront appends with one atomic. (In the head's own steps this code next to the other cost the common
// kernels 1 to 2 %, in registers, and gave the widest steps nothing.)
template <int L, typename Word, typename Wanted>
__device__ __forceinline__ void claim_cells(const int (&nb)[L], uint32_t n_keys, int flag, int lane, int* cid, int* n_claimed,
                                            const Word& bit_word, const Wanted& wanted) {
    uint32_t old[L];
    u64 fresh[L];
#pragma unroll
    for (int u = 0; u < L; ++u) {
        old[u] = ~0u;
        if ((uint32_t)nb[u] < n_keys && wanted(nb[u]))
            old[u] = __hip_atomic_fetch_or(bit_word(nb[u]), 1u << (nb[u] & 31), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    int total = 0;
#pragma unroll
    for (int u = 0; u < L; ++u) {
        fresh[u] = __builtin_amdgcn_ballot_w64(!((old[u] >> (nb[u] & 31)) & 1u));
        total += __popcll(fresh[u]);
    }
    if (total == 0) return;
    int at = 0;
    if (lane == 0) at = atomicAdd(n_claimed, total);
    at = __builtin_amdgcn_readfirstlane(at);
#pragma unroll
    for (int u = 0; u < L; ++u) {
        if ((fresh[u] >> lane) & 1ull) cid[at + __popcll(fresh[u] & ((1ull << lane) - 1ull))] = nb[u] | flag;
        at += __popcll(fresh[u]);
    }
}

// The whole search of one (sequence, query head) by one workgroup of T threads.
// N is the number of keys the graph covers; the key rows of a (sequence, KV head) start every
// kv_stride rows (kv_stride >= N: the cache may hold tokens appended after the index was built).
// `lds_raw` is the workgroup's dynamic LDS (ra_search_lds_bytes of it). Writes ids/stats of
// `head`; when `lds_ids` is not null the ids are also left there (LDS) for a fused consumer.
// Returns the number of valid ids. Ends with the whole workgroup past a barrier. Touched words may still be on their way to the first
// SR_TOUCH_BYTES of lds_raw: the caller leaves these alone, and every wavefront waits for its loads before it ends (end_touches).
// A caller's hook into run_search: note_off_words() is called by one thread ahead of the first barrier, for words that
// another workgroup may set at any moment: the wavefronts of a workgroup must not decide by what each of them has read (they
// would part at the barriers behind the decision), but by what one thread has read and left in LDS. kSeedShare says whether the start set of a seeded walk may be scored by other workgroups of
// the launch (score_seed_share below): then seeds_shared() says whether it is in this launch,
// take_seed_keys(c0, c1, k0, k1) waits (bounded) for keys c0 and c1 of the set (c1 < 0: only c0; k1 is
// then k0 again) and leaves 0 for one that did not come, and seeds_missed() is called by one thread
// when some key did not.
// kShareSteps says whether workers take the claims and the scores of its steps (serve_walk below) if steps_shared(), with
// `parts_log2`, `spin` and the head's `area`. If not, and when an answer does not come, upon which steps_missed() is called by
// one thread, the search returns -1, with no ids and no counters written.
// kValues says whether the caller reads rows of its own of the ids found: then touch_value(id, line, off) brings a line of
// such a row into this XCD's L2 (see touch_line).
struct NoHook {
    static constexpr bool kSeedShare = false;
    static constexpr bool kShareSteps = false;
    static constexpr bool kValues = false;
    __device__ __forceinline__ void note_off_words() const {}
};

// Words that cross workgroups inside one launch: relaxed agent-scope atomics, which go around the
// cache levels that are not coherent across the part's XCDs.
__device__ __forceinline__ void xwg_store(uint32_t* p, uint32_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void xwg_store(u64* p, u64 v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t xwg_load(const uint32_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ u64 xwg_load(const u64* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One of `parts` shares of a head's seed set, scored by a workgroup of its own (T threads) while the
// head's workgroup clears its state and claims the set's ids: what bounds the scoring of a start set
// is the rate at which one compute unit takes in scattered rows, and a launch with few searches
// leaves most compute units idle. The keys (the same bits the head would have made: same share
// sums, same tree) go to keys[c] for the share's positions c of the set. A key is never zero and
// is written by one 64-bit store, so the slot itself tells the head that its key has come; the head
// zeroes it again when it has taken the key. n_cfg is the size the sets were listed for (a head's
// set may have fewer ids): shares are cut by it, so the ids can be requested together with the set's
// header. A set that is no seed set, or does not fit the candidate array of the walk (maxc), is
// left to the head, which applies the same test and does not wait then.
template <int DT, int KT, int T>
__device__ __forceinline__ void score_seed_share(int head, int part, int parts, const void* __restrict__ q,
                                                 const void* __restrict__ K, int n_q, int n_kv, int64_t kv_stride,
                                                 const int32_t* __restrict__ roots, int root_cap, int n_cfg,
                                                 int maxc, const float* __restrict__ kscale, u64* keys) {
    const int tid = threadIdx.x, grp = tid >> 4, lane16 = tid & 15;
    const int seq = head / n_q, h = head % n_q, kvh = h / (n_q / n_kv);
    const size_t esz = DT == RA_BF16 ? 2 : 4;
    const size_t ksz = KT == RA_KEYS_I8 ? 1 : KT == RA_BF16 ? 2 : 4;
    const int32_t* root = roots + (size_t)head * root_cap;
    const int per = (n_cfg + parts - 1) / parts;
    const int c_beg = part * per;
    // (twice the rows in flight per lane group where the workgroup is small: the walk's own registers
    // are not live here, and a share is then one trip to memory again)
    constexpr int R = (T <= 512 && KT != RA_F32) ? 16 : SR_UNROLL, PER = T / 16;
    const char* Kh = reinterpret_cast<const char*>(K) + ((size_t)seq * n_kv + kvh) * kv_stride * RA_D * ksz;
    ScoreQuery<KT> qv;
    load_score_query<DT, KT>(reinterpret_cast<const char*>(q) + (size_t)head * RA_D * esz, lane16, qv);
    if constexpr (KT == RA_KEYS_I8) {
        const float* sc = kscale + ((size_t)seq * n_kv + kvh) * RA_D + lane16 * 8;
#pragma unroll
        for (int e = 0; e < 8; ++e) qv.v[e] = __fmul_rn(qv.v[e], sc[e]);
    }
    const int n_root = root[0], n_first = root[1];
#ifdef SR_WAVE_CLOCKS
    const int wslot_ = head == 0 && tid == 0 ? (part == 0 ? 8 : part == parts - 1 ? 16 : -1) : -1;
    if (wslot_ >= 0) sr_wave_ticks[wslot_] = wall_clock64();
    if (wslot_ >= 0 && n_root >= 0) sr_wave_ticks[wslot_ + 1] = wall_clock64();
#endif
    for (int c0 = c_beg; c0 < c_beg + per; c0 += R * PER) {
        // ids first, wherever the set ends (slots up to root_cap - 3 exist), then the header decides
        const int cw = c0 + (lane16 & (R - 1)) * PER + grp;      // the key this lane will write
        int idw = root[2 + min(cw, root_cap - 3)];
        int idv[R];
#pragma unroll
        for (int u = 0; u < R; ++u) idv[u] = root[2 + min(c0 + u * PER + grp, root_cap - 3)];
        if (n_first != 0 || n_root < 1 || n_root > maxc) return;
        const int c_end = min(n_root, c_beg + per);
        if (c0 >= c_end) return;
        const int id0 = root[2];
        RowBits<KT> rows[R];
#pragma unroll
        for (int u = 0; u < R; ++u)                           // past the end: the set's first row again
            rows[u] = load_key<KT>(Kh, c0 + u * PER + grp < c_end ? idv[u] : id0, lane16);
        float sh[R];
#pragma unroll
        for (int u = 0; u < R; ++u) sh[u] = score_share<KT>(rows[u], qv);
        const float sc = rows_tree<R>(sh, lane16);
#ifdef SR_WAVE_CLOCKS
        if (wslot_ >= 0 && sc == sc) sr_wave_ticks[wslot_ + 2] = wall_clock64();
#endif
        if (lane16 < R && cw < c_end) xwg_store(keys + cw, make_key(sc, idw));
#ifdef SR_WAVE_CLOCKS
        __builtin_amdgcn_s_waitcnt(0x0F70);
        if (wslot_ >= 0) sr_wave_ticks[wslot_ + 3] = wall_clock64();
        if (head == 0 && (tid & 63) == 0 && tid < 512) sr_wave_ticks[32 + part * 8 + tid / 64] = wall_clock64();
#endif
    }
}

// ---- Steps of a walk shared out over workgroups ----------------------------------------------------------
// A walk whose visited set is in device memory is bound by what one compute unit can take in: it has some 330 cache lines on
// their way at a time, whatever the load instructions are (a thousand scattered rows of 256 bytes: 5 ticks each from L2, 12 from
// memory), and an atomic to the visited set takes four ticks. A launch of few searches has compute units to spare, so there a
// head has 2^parts_log2 worker workgroups. Each owns a share of the keys (the 32-key words of the visited set in turn), claims
// those of the start set and of all steps' neighbours that are its own, in an LDS bitset of its share, and scores them. What can enter the beam goes back to the head, which picks and merges. Beams are top-ef sets of unions, so no result
// depends on who scored what. A hand-over (relaxed agent-scope stores, polled) takes 1000 to 1500 ticks one way.
// A head has one message, which all its workers poll: words with a number of the message in the upper half, one more each time,
// over all launches (SR_MSG_LAST keeps the last): [0] the number of picks (0: the walk has ended), [1], [2] the
// worst beam entry that counts, then their ids. An answer, a worker's own: [0] bit 63, keys claimed << 32, keys that can enter the
// beam, then those; answer 0, to no message, is the start set (the head sends nothing before it: all workers have read by then
// where the numbers stand). Every word says itself whether it has come. Answers are zeroed by the head
// when it has taken them, and have two places, used in turn: a word is written again two messages later, when the head has seen its zeroes
// written (it waits for those of answer k when it has received k + 1: they are by then). Both are stored 64 words at a
// time: keys stored as they were scored, a few words per instruction, took 2 to 3 us to arrive. All waits are bounded: a head whose
// answers do not come walks alone from the start, and the handle shares no walk any more, so words that come late are
// never taken for the next launch's. (That walk is a search of its own in the kernel: with both in one, behind a flag, the kernel of
// bf16 keys and 1024 threads had 128 VGPRs and 112 bytes of scratch memory per lane instead of 114 and none, and
// 1M keys took 1.5 % longer.)
#define SR_VALID (1ull << 63)
#define SR_MSG_LAST 0             // words of a head's part of the hand-over area
#define SR_MSG_WORDS 8
#define SR_ANSWERS_AT (SR_MSG_WORDS + 3 + RA_MAX_EXPAND + 5)
#define SR_ANSWER_WORDS (RA_WALK_CELLS + 8)
static_assert(SR_ANSWERS_AT == RA_WALK_HEAD_WORDS && 2 * SR_ANSWER_WORDS == RA_WALK_PART_WORDS, "the allocation's sizes");
__device__ __forceinline__ u64* sr_answer(u64* area, int part, int k) { return area + SR_ANSWERS_AT + (2 * part + (k & 1)) * SR_ANSWER_WORDS; }

// The rows of the n keys listed in cid (bit 31: enters the beam as expanded) scored, those that beat `worst` added to `kept`.
template <int KT, int T>
__device__ __forceinline__ void serve_rows(const char* Kh, const ScoreQuery<KT>& qv, const int* cid, int n, u64 worst, u64* kept,
                                           int* n_kept) {
    const int grp = threadIdx.x >> 4, lane16 = threadIdx.x & 15;
    constexpr int PER = T / 16;
    auto rows_at = [&](auto rows_c, int c0) __attribute__((always_inline)) {
        constexpr int R = decltype(rows_c)::value;
        RowBits<KT> rows[R];
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const int c = c0 + u * PER + grp;
            rows[u] = load_key<KT>(Kh, cid[c < n ? c : 0] & 0x7fffffff, lane16);
        }
        const int cw = c0 + (lane16 & (R - 1)) * PER + grp;
        const int idw = cid[cw < n ? cw : 0];
        float part[R];
#pragma unroll
        for (int u = 0; u < R; ++u) part[u] = score_share<KT>(rows[u], qv);
        const float sc = rows_tree<R>(part, lane16);
        if (lane16 < R && cw < n) {
            u64 key = make_key(sc, idw & 0x7fffffff);
            if (idw < 0) key &= ~1ull;
            if ((key >> 1) > worst) kept[atomicAdd(n_kept, 1)] = key;
        }
    };
    int c0 = 0;
    for (; n - c0 > 4 * PER; c0 += SR_UNROLL * PER) rows_at(sr_int<SR_UNROLL>{}, c0);
    if (n - c0 > 2 * PER) rows_at(sr_int<4>{}, c0);
    else if (n - c0 > PER) rows_at(sr_int<2>{}, c0);
    else if (n - c0 > 0) rows_at(sr_int<1>{}, c0);
}

// LDS bytes of a worker.
static inline size_t serve_lds_bytes(int64_t N, int deg, int expand, int parts_log2) {
    return 64 + (size_t)expand * deg * 12 + (size_t)expand * 4 + ((((size_t)(N + 31) >> 5) >> parts_log2) + 1) * 4;
}

// Worker `part` of `head`. (deg >= 2: see the reciprocals of run_search.)
template <int DT, int KT, int T>
__device__ __forceinline__ void serve_walk(unsigned char* lds_raw, int head, int part, int parts_log2, const void* __restrict__ q,
                                           const int32_t* __restrict__ adj, const int32_t* __restrict__ entry,
                                           const void* __restrict__ K, int n_q, int n_kv, int64_t N, int64_t kv_stride, int deg,
                                           int ef, int expand, const int32_t* __restrict__ roots, int root_cap,
                                           const float* __restrict__ kscale, u64* area, uint32_t is_off, int spin) {
    const int tid = threadIdx.x, lane = tid & (RA_WAVE - 1), lane16 = tid & 15;
    const int seq = head / n_q, h = head % n_q, kvh = h / (n_q / n_kv);
    const size_t esz = DT == RA_BF16 ? 2 : 4;
    const size_t ksz = KT == RA_KEYS_I8 ? 1 : KT == RA_BF16 ? 2 : 4;
    const char* Kh = reinterpret_cast<const char*>(K) + ((size_t)seq * n_kv + kvh) * kv_stride * RA_D * ksz;
    const int32_t* adj_h = adj + (size_t)head * N * deg;
    const int maxc = expand * deg;
    int* ctr = reinterpret_cast<int*>(lds_raw);      // [0] claimed, [1] kept, [2] picks, [3] steps are not shared, or a wait ran out, [4..5] worst
    u64* worst_at = reinterpret_cast<u64*>(ctr + 4);
    u64* kept = reinterpret_cast<u64*>(ctr + 16);
    int* cid = reinterpret_cast<int*>(kept + maxc);
    int* picks = cid + maxc;
    uint32_t* bits = reinterpret_cast<uint32_t*>(picks + expand);
    const uint32_t n_keys = (uint32_t)N, mask = (1u << parts_log2) - 1u;
    ScoreQuery<KT> qv;
    load_score_query<DT, KT>(reinterpret_cast<const char*>(q) + (size_t)head * RA_D * esz, lane16, qv);
    if constexpr (KT == RA_KEYS_I8) {
        const float* sc = kscale + ((size_t)seq * n_kv + kvh) * RA_D + lane16 * 8;
#pragma unroll
        for (int e = 0; e < 8; ++e) qv.v[e] = __fmul_rn(qv.v[e], sc[e]);
    }
    const int e0 = entry[head];
    const uint32_t last = (uint32_t)xwg_load(area + SR_MSG_LAST);
    const u64* message = area + SR_MSG_WORDS;
    const int32_t* root = roots + (size_t)head * root_cap;
    const int n_root = root[0], n_first = root[1];
    for (int i = tid; i < (int)((((N + 31) >> 5) >> parts_log2) + 1); i += T) bits[i] = 0u;
    if (tid < 16) ctr[tid] = tid == 3 ? (int)is_off : 0;
    __syncthreads();
    if (ctr[3]) return;
    auto mine = [&](int id) __attribute__((always_inline)) { return (((uint32_t)id >> 5) & mask) == (uint32_t)part; };
    auto word_of = [&](int id) __attribute__((always_inline)) { return bits + (((uint32_t)id >> 5) >> parts_log2); };
    // the start set (run_search applies the same test)
    if (n_root <= maxc && (n_first == 0 ? n_root >= 1 : n_first > 1 && expand >= n_first - 1 && ef >= n_first)) {
        for (int c0 = 0; c0 < n_root; c0 += T) {
            const int id[1] = {c0 + tid < n_root ? root[2 + c0 + tid] : -1};
            claim_cells(id, n_keys, c0 + tid < n_first ? (int)0x80000000u : 0, lane, cid, ctr, word_of, mine);
        }
    } else if (tid == 0 && mine(e0)) {
        *word_of(e0) |= 1u << (e0 & 31);             // (scored by the head)
    }
    const uint32_t deg_m = 0xffffffffu / (uint32_t)deg + 1u;
    u64 worst = 0ull;
    for (int k = 0;; ++k) {
        __syncthreads();
        const int n = __builtin_amdgcn_readfirstlane(ctr[0]);
        serve_rows<KT, T>(Kh, qv, cid, n, worst, kept, &ctr[1]);
        __syncthreads();
        const int n_kept = __builtin_amdgcn_readfirstlane(ctr[1]);
        u64* answer = sr_answer(area, part, k);
        for (int i = tid; i <= n_kept; i += T) xwg_store(answer + i, i == 0 ? SR_VALID | (u64)n << 32 | (u64)n_kept : kept[i - 1]);
        // ---- the next message
        const uint32_t number = last + 1u + (uint32_t)k;
        if (tid < expand) {
            u64 w[3] = {0ull, 0ull, 0ull}, own = 0ull;
            bool came = false;
            for (int i = 0; i < spin; ++i) {
#pragma unroll
                for (int j = 0; j < 3; ++j)
                    if ((uint32_t)(w[j] >> 32) != number) w[j] = xwg_load(message + j);
                if ((uint32_t)(own >> 32) != number) own = xwg_load(message + 3 + tid);
                came = (uint32_t)(w[0] >> 32) == number && (uint32_t)(w[1] >> 32) == number && (uint32_t)(w[2] >> 32) == number &&
                       (tid >= (int)(uint32_t)w[0] || (uint32_t)(own >> 32) == number);
                if (came) break;
                __builtin_amdgcn_s_sleep(1);
            }
            if (!came) ctr[3] = 1;
            picks[tid] = (int)(uint32_t)own;
            if (tid == 0) {
                ctr[2] = (int)(uint32_t)w[0];
                *worst_at = w[1] << 32 | (uint32_t)w[2];
            }
        }
        __syncthreads();
        const int np = __builtin_amdgcn_readfirstlane(ctr[3] ? 0 : ctr[2]);
        if (np == 0) return;
        if (tid == 0) {
            ctr[0] = 0;
            ctr[1] = 0;
        }
        worst = *worst_at;
        const int cells = np * deg;
        __syncthreads();
        if ((deg & 3) == 0) {
            // rows are 16-byte aligned: four cells per load
            const int quads = cells >> 2;
            for (int x0 = 0; x0 < quads; x0 += 2 * T) {
                int nb[8];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int x = 4 * min(x0 + u * T + tid, quads - 1), xr = (int)__umulhi((uint32_t)x, deg_m);
                    const int4 v = *reinterpret_cast<const int4*>(adj_h + (size_t)picks[xr] * deg + (x - xr * deg));
                    nb[4 * u] = v.x; nb[4 * u + 1] = v.y; nb[4 * u + 2] = v.z; nb[4 * u + 3] = v.w;
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) nb[u] = x0 + (u / 4) * T + tid < quads ? nb[u] : -1;
                claim_cells(nb, n_keys, 0, lane, cid, ctr, word_of, mine);
            }
        } else {
            for (int x0 = 0; x0 < cells; x0 += 4 * T) {
                int nb[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int x = min(x0 + u * T + tid, cells - 1), xr = (int)__umulhi((uint32_t)x, deg_m);
                    nb[u] = adj_h[(size_t)picks[xr] * deg + (x - xr * deg)];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) nb[u] = x0 + u * T + tid < cells ? nb[u] : -1;
                claim_cells(nb, n_keys, 0, lane, cid, ctr, word_of, mine);
            }
        }
    }
}

template <int DT, int KT, bool GBITS, int T, typename Hook>
__device__ __forceinline__ int run_search(
    unsigned char* lds_raw, int head, const void* __restrict__ q, const int32_t* __restrict__ adj,
    const int32_t* __restrict__ entry, const void* __restrict__ K, int n_q, int n_kv, int64_t N,
    int64_t kv_stride, int deg, int s, int w, int topk, int take, int ef, int expand,
    uint32_t* __restrict__ gbits, int32_t* __restrict__ ids, ra_stats* __restrict__ stats, int32_t* lds_ids,
    const int32_t* __restrict__ roots, int root_cap, const float* __restrict__ kscale, const Hook& hook) {
    const int tid = threadIdx.x, grp = tid >> 4, lane16 = tid & 15;
    const int lane = tid & (RA_WAVE - 1), wv = tid / RA_WAVE;
    const int seq = head / n_q, h = head % n_q, kvh = h / (n_q / n_kv);
    const size_t esz = DT == RA_BF16 ? 2 : 4;                                   // of the query
    const size_t ksz = KT == RA_KEYS_I8 ? 1 : KT == RA_BF16 ? 2 : 4;            // of the keys the walk scores
    const char* Kh = reinterpret_cast<const char*>(K) + ((size_t)seq * n_kv + kvh) * kv_stride * RA_D * ksz;
    const int32_t* adj_h = adj + (size_t)head * N * deg;
    const int maxc = expand * deg;
    const int nwords = (int)((N + 31) >> 5);

    // A beam entry's place needs the number of candidates in the beam slots before its wavefront's 64. A
    // large workgroup (wide beams are its only ones) keeps sums per 64 slots; with 512 threads or fewer
    // the beam is a few blocks and adding them up is cheaper than one more LDS add per candidate.
    constexpr bool HSUM = T == 1024;
    SR_TICK_INIT;
#ifdef SR_WAVE_CLOCKS
    if (head == 0 && tid == 0) sr_wave_ticks[0] = wall_clock64();      // search entered
#endif
    // (the piece touched words land in comes first: its LDS address has to fit 16 bits)
    const uint32_t touch_off = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds_raw;
    u64* cur = reinterpret_cast<u64*>(lds_raw + SR_TOUCH_BYTES);
    u64* nxt = cur + ef;
    u64* ckey = nxt + ef;            // [maxc + 16] candidates that passed the beam threshold
    int* cid = reinterpret_cast<int*>(ckey + maxc + 16);  // [maxc] claimed neighbour ids
    int* cnt = cid + maxc;           // [maxc] merge counters of the candidates, zero between steps
    int* hist = cnt + maxc;          // [ef + 1] candidates per beam slot, zero when a merge begins
    int* hsum = hist + ef + 1;       // [(ef + 64) / 64] candidates per 64 beam slots, likewise
    const int nsum = (ef + 64) / 64, nhist = ef + 1 + nsum;
    int* picks = hist + nhist;       // [expand]
    int* ctr = picks + expand;
    // A step's counters: candidates claimed and kept, and the unexpanded entries of the beam it starts
    // from. The next step uses the other three words, which are cleared at the start of this one (no
    // barrier has to part a counter's last reader from its clearing).
    int* cc = ctr + C_STEP;
    int* cc_nxt = ctr + C_STEP2;
    bool hist_used = false;
    bool masked = false;             // cnt holds the masks of the seed set the walk starts from, until its first step behind that
    int* wtot = ctr + C_WTOT;
    // urank[i], i in [0, bn]: unexpanded entries among the first i of the beam, as of the last pick
    // but before its picks were marked expanded (two buffers, swapped with the beam's)
    uint16_t* urank = reinterpret_cast<uint16_t*>(ctr + C_COUNT);    // [ef + 1]
    uint16_t* urank_nxt = urank + ef + 1;                            // [ef + 1]
    uint32_t* bits = GBITS ? gbits + (size_t)head * nwords
                           : reinterpret_cast<uint32_t*>(urank_nxt + ef + 1);

    ScoreQuery<KT> qv;
    load_score_query<DT, KT>(reinterpret_cast<const char*>(q) + (size_t)head * RA_D * esz, lane16, qv);
    if constexpr (KT == RA_KEYS_I8) {
        // 8-bit keys: k ~ k8 * scale per dimension, so the walk scores <q * scale, k8>
        const float* sc = kscale + ((size_t)seq * n_kv + kvh) * RA_D + lane16 * 8;
#pragma unroll
        for (int e = 0; e < 8; ++e) qv.v[e] = __fmul_rn(qv.v[e], sc[e]);
    }
    const int e0 = entry[head];
    // The first two steps of a walk do not depend on the query: the entry point is expanded, then
    // all its neighbours are (when `expand` and ef are at least their number). What they visit,
    // the entry point's root set, is listed with the index (ra_launch_roots): [0] its size,
    // [1] 1 + the number of the entry point's neighbours, then the ids, those first. With it the
    // two steps become one: every key of the set is scored in one gather and the beam is the
    // top ef of them, the entry point and its neighbours marked expanded. Same beam, same visited
    // set, same counters as the two steps taken one after the other.
    const int32_t* root = roots ? roots + (size_t)head * root_cap : nullptr;
    int n_root = 0, n_first = 0;
    // (of a thread's first ids, and of a seed set their masks, unconditional: same trip as the header)
    constexpr int AHEAD = 4;
    int my_root[AHEAD] = {}, my_mask[AHEAD] = {};
    const int mask_words = seed_mask_words(deg), masks_at = 2 + seed_places(root_cap, deg);
    if (root) {
        n_root = root[0];
        n_first = root[1];
        if constexpr (!Hook::kShareSteps)
#pragma unroll
            for (int r = 0; r < AHEAD; ++r) {
                my_root[r] = root[2 + min(tid + r * T, root_cap - 3)];
                my_mask[r] = root[min(masks_at + (tid + r * T) * mask_words, root_cap - 1)];
            }
    }
    int n_posted = 0;                // (kShareSteps: claims and scores are the workers', serve_walk)
    uint32_t last_message = 0u;
    if constexpr (Hook::kShareSteps) last_message = (uint32_t)xwg_load(hook.area + SR_MSG_LAST);
    // (the loads above are in flight while the LDS state is cleared)
    if constexpr (!Hook::kShareSteps)
        for (int i = tid; i < nwords; i += T) bits[i] = 0u;
    for (int i = tid; i < maxc + nhist; i += T) cnt[i] = 0;      // cnt, hist and hsum
    for (int i = tid; i < 2 * ef; i += T) cur[i] = 0ull;         // both beams (what follows a beam's last entry is zero)
    // A seed set (ra_launch_seeds) has the same layout with [1] = 0: the walk starts from all of its
    // keys at once, scored in one gather, the best ef of them in the beam and none of them expanded.
    // That is a start of its own, not a shortcut for steps of the single-entry walk: no step is
    // counted for it. (The host checks that a seed set fits the candidate arrays.)
    const bool seeded = root && n_first == 0;
    const bool fill = root && n_root <= maxc &&
                      (seeded ? n_root >= 1 : n_first > 1 && expand >= n_first - 1 && ef >= n_first);
    if (tid == 0) hook.note_off_words();
    __syncthreads();                                             // the LDS state is cleared
    SR_TICK(12);
    bool seeds_shared = false;               // (asked for here: the claims cover the trip to LDS)
    if constexpr (Hook::kSeedShare) seeds_shared = hook.seeds_shared();
#ifdef SR_WAVE_CLOCKS
    if (head == 0 && tid == 0) sr_wave_ticks[1] = wall_clock64();
#endif
    // with masks: new cells (pick, cell) of the first picks, up to T of them, and the places in the seed set of the keys
    // that the first beam is made of, behind what that and a step's claims of that few cells use of cid
    static_assert(SR_LIST_AT >= 512 && SR_LIST_AT >= T && RA_MAX_EXPAND * 64 <= 65536, "a pick and a cell of its row in 16 bits");
    uint16_t* fresh_cells = reinterpret_cast<uint16_t*>(cid + SR_LIST_AT);
    uint16_t* seed_at = fresh_cells + T;
    // whether a start set is ordered through bins (below)
    auto start_bins = [&]() __attribute__((always_inline)) { return n_root > SR_DIRECT && n_root <= SR_START_REGS * T && maxc >= 512; };
    int bn, n_visited, n_expanded, n_iters;
    if (Hook::kShareSteps && tid == 0) ctr[C_MISSED] = 0;
    if (fill) {
        if constexpr (!Hook::kShareSteps) {
            masked = seeded && start_bins() && n_root * mask_words <= maxc && maxc >= SR_LIST_AT + (n_root + T + 1) / 2;
            auto enter = [&](int c, int id, int m) __attribute__((always_inline)) {
                cid[c] = id;
                (void)claim_key(bits, id);
                if (masked) {
                    cnt[c] = m;
                    if (mask_words == 2) cnt[n_root + c] = root[masks_at + 2 * c + 1];
                }
            };
#pragma unroll
            for (int r = 0; r < AHEAD; ++r)
                if (tid + r * T < n_root) enter(tid + r * T, my_root[r], my_mask[r]);
            for (int c = tid + AHEAD * T; c < n_root; c += T) enter(c, root[2 + c], masked ? root[masks_at + c * mask_words] : 0);
        }
        if (tid == 0) {
            urank[0] = 0;
            for (int i = 0; i < 3; ++i) cc[i] = cc_nxt[i] = 0;
            ctr[C_LO] = -1;                  // as unsigned: the largest value; see the first beam below
            ctr[C_HI] = 0;
            ctr[C_MISSED] = 0;
            wtot[0] = 0;                     // (new cells of the first picks; the results use it otherwise)
        }
        // (of a root set the entry point's step and its neighbours' step; of a seed set none)
        bn = 0; n_visited = n_root; n_expanded = n_first; n_iters = seeded ? 0 : 2;
    } else {
        if (grp == 0) {
            const RowBits<KT> r = load_key<KT>(Kh, e0, lane16);
            const float sc = score_fixed<KT>(r, qv);
            if (tid == 0) {
                // the beam is the entry point alone, and the first step can only pick it: leave the
                // state a merge would leave (pick in place, flag cleared, counts of unexpanded entries)
                cur[0] = make_key(sc, e0) & ~1ull;
                picks[0] = e0;
                urank[0] = 0;
                cc[S_NCAND] = 0;
                cc[S_NKEEP] = 0;
                cc[S_NUNEXP] = 1;
                if constexpr (!Hook::kShareSteps) (void)claim_key(bits, e0);
            }
        }
        bn = 1; n_visited = 1; n_expanded = 0; n_iters = 0;
    }
    // The adjacency cells of a step are dealt to the threads in order (cell x is slot x % deg of pick x / deg):
    // the pick and the slot of a thread's first two cells are the same in every step. (The quotients by
    // multiplications, exact while (x + 1) * deg < 2^32: there are at most RA_MAX_EXPAND * deg cells. x / deg is
    // the upper half of (x + 1) * floor((2^32 - 1) / deg) for every degree; of x * deg_m for all but degree 1,
    // whose steps, of two cells per thread at most, never come to the loop that uses deg_m.)
    static_assert(RA_MAX_EXPAND <= 2 * T, "a step of a graph of degree 1 has at most two cells per thread");
    const uint32_t deg_f = 0xffffffffu / (uint32_t)deg, deg_m = deg_f + 1u;
    const int xr0 = min((int)__umulhi((uint32_t)tid + 1u, deg_f), expand - 1);
    const int xr1 = min((int)__umulhi((uint32_t)(tid + T) + 1u, deg_f), expand - 1);
    const int xs0 = min(tid - xr0 * deg, deg - 1), xs1 = min(tid + T - xr1 * deg, deg - 1);
    const int gi0 = min(grp, maxc - 1), gi1 = min(grp + T / 16, maxc - 1);
    // Adjacency rows likely to be expanded soon are touched ahead of time (one word of the row's
    // first line), so that the row is in this XCD's L2 when its step reads it: the rows of the
    // candidates a step keeps, touched while they are merged, and the rows of the beam entries that
    // are next in line after the coming step's picks. The words land in a spare piece of LDS and are
    // read by nothing (touch_line).
    __syncthreads();
    SR_TICK(13);
    if constexpr (Hook::kShareSteps)
        if (!hook.steps_shared()) return -1;
#ifdef SR_WAVE_CLOCKS
    if (head == 0 && tid == 0) sr_wave_ticks[2] = wall_clock64();      // claims made
#endif
    // The workers' answers to the last message: the keys go to ckey. A worker's are taken by up to 64 threads, of one wavefront (the word
    // that says how many there are is read by all of them before one zeroes it), each asking for a key together with that word. got(score): the ordered score bits of a key that has come.
    auto collect = [&](auto got) __attribute__((always_inline)) {
        if constexpr (Hook::kShareSteps) {
            const int spin = hook.spin, per_log2 = min((T == 1024 ? 10 : 9) - hook.parts_log2, 6);
            const int per = 1 << per_log2, sub = tid & (per - 1);
            if (tid >> (per_log2 + hook.parts_log2)) return;
            u64* a = sr_answer(hook.area, tid >> per_log2, n_posted);
            u64 n_word = 0ull, k0 = 0ull;
            int n = 0;
            bool came = false;
            for (int i = 0; i < spin; ++i) {
                if (n_word == 0ull) n_word = xwg_load(a);
                if (k0 == 0ull) k0 = xwg_load(a + 1 + sub);
                n = (int)(n_word & 0xffffffffull);
                came = n_word != 0ull && (sub >= n || k0 != 0ull);
                if (came) break;
                __builtin_amdgcn_s_sleep(1);
            }
            if (!came) {
                ctr[C_MISSED] = 1;
                n = 0;
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // the zeroes in the answers before these are written
            if (came && sub == 0) {
                atomicAdd(&cc[S_NCAND], (int)((n_word >> 32) & 0x7fffffffull));
                xwg_store(a, 0ull);
            }
            for (int i = sub; __builtin_amdgcn_ballot_w64(i < n) != 0ull; i += per) {
                u64 k = i == sub && i < n ? k0 : 0ull;
                for (int t = 0; t < spin && k == 0ull && i < n; ++t) k = xwg_load(a + 1 + i);
                if (i < n && k == 0ull) ctr[C_MISSED] = 1;
                const u64 m = __builtin_amdgcn_ballot_w64(k != 0ull);
                int at = 0;
                if (lane == 0 && m) at = atomicAdd(&cc[S_NKEEP], __popcll(m));
                at = __builtin_amdgcn_readfirstlane(at) + __popcll(m & ((1ull << lane) - 1ull));
                if (k != 0ull) {
                    xwg_store(a + 1 + i, 0ull);
                    ckey[at] = k;
                    got((uint32_t)(k >> 32));
                }
            }
        }
    };
    // the first np picks to the workers (0: the walk has ended)
    auto post = [&](int np, u64 worst) __attribute__((always_inline)) {
        if constexpr (Hook::kShareSteps) {
            ++n_posted;
            const u64 number = (u64)(last_message + (uint32_t)n_posted) << 32;
            if (tid < np + 3)                // (at most RA_MAX_EXPAND + 3 words: one per thread)
                xwg_store(hook.area + SR_MSG_WORDS + tid, number | (tid == 0 ? (uint32_t)np : tid == 1 ? (uint32_t)(worst >> 32) :
                                                                    tid == 2 ? (uint32_t)worst : (uint32_t)picks[tid - 3]));
        }
    };
    if constexpr (Hook::kShareSteps) {
        uint32_t lo = 0xffffffffu, hi = 0u;
        collect([&](uint32_t score) __attribute__((always_inline)) {
            lo = min(lo, score);
            hi = max(hi, score);
        });
        if (fill) {
            wave_min_max(lo, hi);
            if (lane == RA_WAVE - 1) {
                atomicMin(reinterpret_cast<unsigned int*>(&ctr[C_LO]), lo);
                atomicMax(reinterpret_cast<unsigned int*>(&ctr[C_HI]), hi);
            }
        }
    } else if (fill) {
        // ---- the start set is scored here, ahead of the loop, where few registers are live: twice
        //      the rows in flight of a step's gather (a seed set of a thousand keys is one trip to
        //      memory for 1024 threads). The beam is empty, so every key is kept; the first
        //      n_first of a root set enter as expanded.
        constexpr int SEED_ROWS = KT == RA_F32 ? SR_UNROLL : 16;
        uint32_t lo = 0xffffffffu, hi = 0u;                  // of the ordered score bits (see the first beam)
        // R rows per 16-lane group with no branch between them: the ids leave LDS in one batch, the
        // rows are all requested before the first is scored, and each is scored as it arrives
        auto score_rows = [&](auto rows_c, int c0) __attribute__((always_inline)) {
            constexpr int R = decltype(rows_c)::value;
            RowBits<KT> rows[R];
            int idv[R];
#pragma unroll
            for (int u = 0; u < R; ++u) {
                const int c = c0 + u * (T / 16) + grp;
                idv[u] = c < n_root ? cid[c] : -1;           // (only the last call of a set is ragged)
            }
#pragma unroll
            for (int u = 0; u < R; ++u) rows[u] = load_key<KT>(Kh, idv[u] >= 0 ? idv[u] : e0, lane16);
            float part[R];
#pragma unroll
            for (int u = 0; u < R; ++u) part[u] = score_share<KT>(rows[u], qv);
            const float sc = rows_tree<R>(part, lane16);     // of row lane16 (R = 16), lane16 & (R - 1) in general
            const int c = c0 + (lane16 & (R - 1)) * (T / 16) + grp;
            if (lane16 < R && c < n_root) {
                u64 key = make_key(sc, cid[c]);
                if (c < n_first) key &= ~1ull;
                ckey[c] = key;                               // all are kept: no counter needed
                const uint32_t so = (uint32_t)(key >> 32);
                lo = so < lo ? so : lo;
                hi = so > hi ? so : hi;
            }
        };
        bool shared = false;
        if constexpr (Hook::kSeedShare) {
            if (seeded && seeds_shared) {
                // the keys come from other workgroups of the launch: every thread takes those of its
                // positions as they arrive; if one does not, the set is scored here after all
                bool came = true;
                for (int c = tid; c < n_root; c += 2 * T) {
                    const bool two = c + T < n_root;
                    u64 k0, k1;
                    hook.take_seed_keys(c, two ? c + T : -1, k0, k1);
                    came = came && k0 != 0ull && k1 != 0ull;
#ifdef SR_WAVE_CLOCKS
                    if (head == 0 && (c & 127) == 0 && c < 1024) sr_wave_ticks[24 + c / 128] = wall_clock64();
#endif
                    ckey[c] = k0;
                    if (two) ckey[c + T] = k1;
                    const uint32_t s0 = (uint32_t)(k0 >> 32), s1 = (uint32_t)(k1 >> 32);
                    lo = min(lo, min(s0, s1));
                    hi = max(hi, max(s0, s1));
                }
                if (!came) ctr[C_MISSED] = 1;
                __syncthreads();
                shared = ctr[C_MISSED] == 0;
                if (!shared) {
                    if (tid == 0) hook.seeds_missed();
                    lo = 0xffffffffu;
                    hi = 0u;
                }
            }
        }
        if (!shared) {
            constexpr int PER = T / 16;                      // rows one call takes per row in flight
            int c0 = 0;
            for (; n_root - c0 >= SEED_ROWS * PER; c0 += SEED_ROWS * PER) score_rows(sr_int<SEED_ROWS>{}, c0);
            if constexpr (SEED_ROWS > 8)
                if (n_root - c0 >= 8 * PER) { score_rows(sr_int<8>{}, c0); c0 += 8 * PER; }
            if (n_root - c0 >= 4 * PER) { score_rows(sr_int<4>{}, c0); c0 += 4 * PER; }
            if (n_root - c0 >= 2 * PER) { score_rows(sr_int<2>{}, c0); c0 += 2 * PER; }
            if (n_root - c0 >= PER) { score_rows(sr_int<1>{}, c0); c0 += PER; }
            if (n_root - c0 > 0) score_rows(sr_int<1>{}, c0);
        }
        // every lane may hold extremes of its keys: fold the wavefront
        wave_min_max(lo, hi);
        if (lane == RA_WAVE - 1) {
            atomicMin(reinterpret_cast<unsigned int*>(&ctr[C_LO]), lo);
            atomicMax(reinterpret_cast<unsigned int*>(&ctr[C_HI]), hi);
        }
    }
#ifdef SR_WAVE_CLOCKS
    if (head == 0 && tid == 0) sr_wave_ticks[3] = wall_clock64();      // start set's keys in LDS
#endif
    SR_TICK(5);

    // An element of a new beam of bn_new at its place: key, position, unexpanded elements above it. What it does not have to
    // store goes to the piece that touched words land in: an address chosen by a lane costs it 4 ticks, a branch 30
    // to 60. (An element past position ef has at least as many unexpanded ones above it as there are picks.) Of a
    // wavefront's 64 beam entries there is seldom one that is picked, and one is the last: branches for all lanes.
    auto place_in = [&](int bn_new, u64 k, int pos, int ur, auto beam) __attribute__((always_inline)) {
        constexpr bool BEAM = decltype(beam)::value != 0;
        const int un = (int)(uint32_t)k & 1;
        const bool pick = (uint32_t)(ur | (un - 1)) < (uint32_t)expand, last = pos == bn_new - 1;
        if (!BEAM || __builtin_amdgcn_ballot_w64(pick)) *(pick ? picks + ur : reinterpret_cast<int*>(lds_raw)) = key_id(k);
        k ^= pick ? 1ull : 0ull;
        *(pos < ef ? nxt + pos : reinterpret_cast<u64*>(lds_raw)) = k;
        *(pos < ef ? urank_nxt + pos : reinterpret_cast<uint16_t*>(lds_raw)) = (uint16_t)ur;
        // (the last one has counted all)
        if (!BEAM || __builtin_amdgcn_ballot_w64(last)) *(last ? cc_nxt + S_NUNEXP : reinterpret_cast<int*>(lds_raw)) = ur + un;
    };
    auto touch_row = [&](int id) __attribute__((always_inline)) {
        touch_line(reinterpret_cast<const char*>(adj_h) + (u64)(uint32_t)id * (uint32_t)(deg * 4), touch_off);
    };
    // of 16 candidates those above k, and (ROOTS: of a start set) in the high half the expanded ones of them
    auto count16 = [&](int at, u64 k, auto roots_c) __attribute__((always_inline)) {
        u64 v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = ckey[at + u];
        int n = 0;
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int up = v[u] > k ? 1 : 0;
            n += up;
            if constexpr (decltype(roots_c)::value != 0) n += (up & ~(int)(uint32_t)v[u]) << 16;
        }
        return n;
    };
    auto swap_beams = [&]() __attribute__((always_inline)) {
        u64* t = cur; cur = nxt; nxt = t;
        uint16_t* tu = urank; urank = urank_nxt; urank_nxt = tu;
        int* tc = cc; cc = cc_nxt; cc_nxt = tc;
    };

    // ---- The first beam: the best ef of a start set, ahead of the loop, so that the loop has nothing of it (a test per phase and the
    //      registers of this part cost walks without seed sets up to 5 %). The scores are cut into 256 equal-width bins between the
    //      smallest and the largest; a key's place is the number of keys in higher bins plus the number of larger ones in its own,
    //      which are few and stored side by side. Of a bin the number of keys and, in the high half, of those that enter as
    //      expanded; a key's number in its bin is what its count returned, and every wavefront adds the bins up for itself, to the
    //      same words, so there are three barriers. Bins below the highest one that holds the ef-th key are left out. The claimed ids
    //      (cid) are dead by now: the bins are there, their sums behind. Counting (few keys, little LDS) is quadratic.
    //      (Inside the loop, with five barriers, and for sets to be filtered only, seed sets and float32; calls in turn, us: four layers of 128K
    //      81.8 -> 78.5, 16 sequences of 32K 41.2 -> 39.7, one float32 head 31.8 -> 29.9, 64K keys in 8 bits 20.0 -> 18.4, one
    //      node per step 329 -> 322.)
    if (fill) {
        __syncthreads();                     // keys, their extremes
        const bool bins = start_bins();
        const int bn_new = n_root < ef ? n_root : ef;
        bool missed = false;
        if constexpr (Hook::kShareSteps) missed = ctr[C_MISSED] != 0;        // (the loop ends at once then: no picks)
        if (bins && !missed) {
            if (tid < 256) cid[tid] = 0;
            __syncthreads();
            const ScoreBins score_bins((uint32_t)ctr[C_LO], (uint32_t)ctr[C_HI]);
            u64 mine[SR_START_REGS];
            int bin[SR_START_REGS];          // a key's, and from bit 8 its number in it
#pragma unroll
            for (int r = 0; r < SR_START_REGS; ++r)
                if (r * T < n_root) mine[r] = ckey[min(r * T + tid, n_root - 1)];
#pragma unroll
            for (int r = 0; r < SR_START_REGS; ++r) {
                if (r * T >= n_root) break;
                bin[r] = score_bins.bin(mine[r]);
                if (r * T + tid < n_root)
                    bin[r] |= (atomicAdd(&cid[bin[r]], 1 + ((int)(~(uint32_t)mine[r] & 1u) << 16)) & 0xffff) << 8;
            }
            __syncthreads();
            // lane l owns bins 4l .. 4l + 3; keys in the bins from b up = total - (those below b), in both halves
            const int b0 = cid[4 * lane], b1 = cid[4 * lane + 1], b2 = cid[4 * lane + 2], b3 = cid[4 * lane + 3];
            const int incl = wave_incl_scan(b0 + b1 + b2 + b3);
            const int above3 = __builtin_amdgcn_readlane(incl, RA_WAVE - 1) - incl;
            const int above2 = above3 + b3, above1 = above2 + b2, above0 = above1 + b1;
            cid[256 + 4 * lane + 3] = above3;
            cid[256 + 4 * lane + 2] = above2;
            cid[256 + 4 * lane + 1] = above1;
            cid[256 + 4 * lane] = above0;
            // the highest bin such that it and those above hold ef keys (all, where there are fewer)
            const int from3 = above2 & 0xffff, from2 = above1 & 0xffff, from1 = above0 & 0xffff, from0 = (above0 + b0) & 0xffff;
            const int best = from3 >= bn_new ? 3 : from2 >= bn_new ? 2 : from1 >= bn_new ? 1 : from0 >= bn_new ? 0 : -1;
            const int from_best = best == 3 ? from3 : best == 2 ? from2 : best == 1 ? from1 : from0;
            const int top = 63 - __clzll(__builtin_amdgcn_ballot_w64(best >= 0));
            const int bstar = 4 * top + __builtin_amdgcn_readlane(best, top), nsurv = __builtin_amdgcn_readlane(from_best, top);
#pragma unroll
            for (int r = 0; r < SR_START_REGS; ++r) {
                if (r * T >= n_root) break;
                if (r * T + tid < n_root && (bin[r] & 255) >= bstar) {
                    const int at = (cid[256 + (bin[r] & 255)] & 0xffff) + (bin[r] >> 8);
                    ckey[at] = mine[r];
                    if (masked) seed_at[at] = (uint16_t)(r * T + tid);
                }
            }
            __syncthreads();
            for (int p = tid; p < nsurv; p += T) {
                const u64 k = ckey[p];
                const int kb = score_bins.bin(k), above = cid[256 + kb], bs = above & 0xffff, n = cid[kb] & 0xffff;
                int pos = bs, ur = bs - (above >> 16), j0 = 0;
                // (past the bucket's end its last key again, taken off below)
                do {
                    u64 other[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) other[i] = ckey[bs + min(j0 + i, n - 1)];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int up = other[i] > k ? 1 : 0;
                        pos += up;
                        ur += up & (int)other[i];            // (the low bit: not expanded)
                    }
                    j0 += 4;
                } while (__builtin_amdgcn_ballot_w64(j0 < n));
                const u64 end = ckey[bs + n - 1];
                const int twice = end > k ? j0 - n : 0;
                pos -= twice;
                ur -= (int)end & 1 ? twice : 0;
                u64 m = ~0ull;
                if (masked && pos < min(ef, expand)) {       // a pick's new cells join the list, if they are few
                    const int c = seed_at[p];
                    m = (uint32_t)cnt[c] | (deg > 32 ? (u64)(uint32_t)cnt[n_root + c] << 32 : 0ull);
                    const int cells = __popcll(m);
                    int at = cells == 0 ? 0 : atomicAdd(wtot, cells > SR_FRESH_CELLS ? T + 1 : cells);
                    if (cells <= SR_FRESH_CELLS)
                        for (u64 left = m; left && at < T; left &= left - 1ull, ++at)
                            fresh_cells[at] = (uint16_t)(pos << 6 | (__ffsll((long long)left) - 1));
                }
                if ((k & 1ull) && ur < expand && m) touch_row(key_id(k));
                if constexpr (Hook::kValues)
                    // (Of a seed set's best nearly all are among those found. Four layers of 128K 80.5 -> 78.6 us; nothing where the head
                    // scores its set itself. At the step that expands all that is left, in any walk: -0.5 to -1.5 %.)
                    if (seeds_shared && seeded && pos < take)
                        for (int line = 0; line < hook.value_lines; ++line) hook.touch_value(key_id(k), line, touch_off);
                place_in(bn_new, k, pos, ur, sr_int<0>{});
            }
        } else if (!missed) {
            ckey[n_root + lane16] = 0ull;    // zeroes behind the candidates, written by each wavefront that reads them
            for (int c = T - 1 - tid; c < n_root; c += T) touch_row(key_id(ckey[c]));
            const int chunks = (n_root + 15) >> 4;
            int t = __builtin_amdgcn_readfirstlane(wv);
            for (int g0 = 0; g0 < n_root; g0 += RA_WAVE, t -= chunks)
                for (; t < chunks; t += T / RA_WAVE) {
                    const int c = min(g0 + lane, n_root - 1);
                    const int n = count16(t * 16, ckey[c], sr_int<1>{});
                    if (g0 + lane < n_root && n) atomicAdd(&cnt[c], n);
                }
            __syncthreads();
            for (int c = T - 1 - tid; c < n_root; c += T) {
                const int both = cnt[c], n = both & 0xffff;
                cnt[c] = 0;
                place_in(bn_new, ckey[c], n, n - (both >> 16), sr_int<0>{});
            }
        }
        __syncthreads();
        if (!missed) {
            bn = bn_new;
            swap_beams();
        }
    }
    SR_TICK(14);

    for (;;) {
        SR_TICK_ITER(n_iters);
        // the last merge (or the set-up) left the picks in place and counted the unexpanded entries
        const int pk0 = picks[xr0];          // the picks of a thread's first two cells (past the last pick: some earlier one or
        const int pk1 = picks[xr1];          // anything, not used)
        const int total = __builtin_amdgcn_readfirstlane(cc[S_NUNEXP]);
        const int np = total < expand ? total : expand;
        if (__builtin_expect(np == 0, 0)) break;
        if (tid == 0) urank[bn] = (uint16_t)total;
        const int unexpanded = total - np;   // entries of the beam left unexpanded by this step
        SR_TICK(0);
        ++n_iters;
        n_expanded += np;

        if (tid == 0) {                      // (read for the last time before the barrier that ended the last merge)
            cc_nxt[S_NCAND] = 0;
            cc_nxt[S_NKEEP] = 0;
            cc_nxt[S_NUNEXP] = 0;
            ctr[C_LO] = -1;
            ctr[C_HI] = 0;
            ctr[C_NSURV] = 0;
        }
        if (__builtin_expect(hist_used, 0)) {
            for (int i = tid; i < nhist; i += T) hist[i] = 0;
            hist_used = false;
        } else if (HSUM && tid < nsum) {
            hsum[tid] = 0;
        }
        if constexpr (Hook::kShareSteps) {
            // ---- the workers claim and score; their answers are waited for
            post(np, bn == ef ? (cur[bn - 1] >> 1) : 0ull);
            collect([](uint32_t) {});
            __syncthreads();
            if (ctr[C_MISSED]) break;
            n_visited += __builtin_amdgcn_readfirstlane(cc[S_NCAND]);
            SR_TICK(1);
        } else {
        // ---- read the picked adjacency rows (all loads issued before any is consumed),
        //      claim unvisited neighbours
        {
            const int cells = np * deg;
            auto claim = [&](int nb) __attribute__((always_inline)) {
                if (nb >= 0 && nb < N) {
                    const uint32_t bit = 1u << (nb & 31);
                    const uint32_t old = claim_key(bits, nb);
                    if (!(old & bit)) cid[atomicAdd(&cc[S_NCAND], 1)] = nb;
                }
            };
            // out-of-range cells read a cell of the entry row: loads without a branch around them can all be
            // issued before the first is consumed
            // The step behind a seed set: nearly all neighbours of its keys are keys of the set (128K keys, 2048 of them: 19 of
            // 8192 cells are new), and which are not is known from the graph alone (the masks), so where they are few, only
            // those are read and claimed.
            bool few = false;
            if (__builtin_expect(masked, 0)) {
                const int n = __builtin_amdgcn_readfirstlane(wtot[0]);
                few = n <= T;
                if (tid < n && few) {
                    const int e = fresh_cells[tid];
                    claim(adj_h[(size_t)picks[e >> 6] * deg + (e & 63)]);        // (no more than T are new: cid up to the list)
                }
                for (int c = tid; c < n_root * mask_words; c += T) cnt[c] = 0;
                masked = false;
            }
            if (few) {
            } else if (__builtin_expect(cells <= 2 * T, 1)) {
                const int v0 = adj_h[(size_t)(tid < cells ? pk0 : e0) * deg + xs0];
                int v1 = -1;
                if (cells > T) v1 = adj_h[(size_t)(tid + T < cells ? pk1 : e0) * deg + xs1];
                claim(tid < cells ? v0 : -1);
                if (cells > T) claim(tid + T < cells ? v1 : -1);
            } else {
                // L cells per thread and pass: as many as a step needs, up to SR_ADJ_LOADS
                auto claim_cells = [&](auto loads_c) __attribute__((always_inline)) {
                    constexpr int L = decltype(loads_c)::value;
                    for (int x0 = 0; x0 < cells; x0 += T * L) {
                        int nbv[L];
#pragma unroll
                        for (int u = 0; u < L; ++u) {
                            const int x = x0 + u * T + tid;
                            const int xc = x < cells ? x : cells - 1;
                            const int xr = (int)__umulhi((uint32_t)xc, deg_m);       // xc / deg
                            const int v = adj_h[(size_t)picks[xr] * deg + (xc - xr * deg)];
                            nbv[u] = x < cells ? v : -1;
                        }
#pragma unroll
                        for (int u = 0; u < L; ++u) claim(nbv[u]);
                    }
                };
                if (cells > 4 * T) claim_cells(sr_int<SR_ADJ_LOADS>{});
                else claim_cells(sr_int<4>{});
            }
        }
        // (the first rows' ids are read with the counter that says how many there are)
        __syncthreads();
        const int id0 = cid[gi0], id1 = cid[gi1];
        const int nc = __builtin_amdgcn_readfirstlane(cc[S_NCAND]);
        n_visited += nc;
        SR_TICK(1);

        // ---- gather and score the new candidates; keep those that can enter the beam
        const u64 worst = bn == ef ? (cur[bn - 1] >> 1) : 0ull;
        // (R rows per 16-lane group with no branch between them, as for a start set; groups without a
        // candidate re-read the entry row instead of branching)
        auto gather_ids = [&](auto rows_c, const int* ids_u, int cw, int idw) __attribute__((always_inline)) {
            constexpr int R = decltype(rows_c)::value;
            RowBits<KT> rows[R];
#pragma unroll
            for (int u = 0; u < R; ++u) rows[u] = load_key<KT>(Kh, ids_u[u] >= 0 ? ids_u[u] : e0, lane16);
            float part[R];
#pragma unroll
            for (int u = 0; u < R; ++u) part[u] = score_share<KT>(rows[u], qv);
            const float sc = rows_tree<R>(part, lane16);     // of row lane16 & (R - 1)
            if (lane16 < R && cw < nc) {
                const u64 key = make_key(sc, idw);
                if ((key >> 1) > worst) ckey[atomicAdd(&cc[S_NKEEP], 1)] = key;
            }
        };
        constexpr int PER = T / 16;
        auto gather_rows = [&](auto rows_c, int c0) __attribute__((always_inline)) {
            constexpr int R = decltype(rows_c)::value;
            int cidv[R];
#pragma unroll
            for (int u = 0; u < R; ++u) {
                const int c = c0 + u * PER + grp;
                cidv[u] = c < nc ? cid[c] : -1;
            }
            const int cw = c0 + (lane16 & (R - 1)) * PER + grp;  // the candidate this lane will keep or drop
            gather_ids(rows_c, cidv, cw, cid[cw < nc ? cw : 0]);
        };
        {
            // as few trips to memory as there can be: the last one takes the number of rows in flight that
            // covers what is left (a trip is 1300 ticks or more, a re-read of the entry row nothing)
            if (__builtin_expect(nc <= 2 * PER, 1)) {
                const int ids_u[2] = {grp < nc ? id0 : -1, grp + PER < nc ? id1 : -1};
                if (nc > PER) gather_ids(sr_int<2>{}, ids_u, (lane16 & 1) * PER + grp, lane16 & 1 ? id1 : id0);
                else if (nc > 0) gather_ids(sr_int<1>{}, ids_u, grp, id0);
            } else {
                int c0 = 0;
                for (; nc - c0 > SR_UNROLL / 2 * PER; c0 += SR_UNROLL * PER) gather_rows(sr_int<SR_UNROLL>{}, c0);
                if (nc - c0 > 2 * PER) gather_rows(sr_int<4>{}, c0);
                else if (nc - c0 > 0) gather_rows(sr_int<2>{}, c0);
            }
        }
        __syncthreads();
        }
        int nk = __builtin_amdgcn_readfirstlane(cc[S_NKEEP]);
        SR_TICK(2);
        // (uniform) Nothing enters the beam, and nothing is left to expand. (Of a step that keeps nothing, but has something
        // left, the merge of few candidates finds the next picks: a pass of its own over the beam took 1400 ticks where this
        // takes 700, and ended every walk. One node per step over 64K keys, ef 256: 380 -> 330 us.)
        if (nk == 0 && unexpanded == 0) break;
        // ---- pre-filter. At most ef of the kept candidates can enter the beam, and the merge below
        //      ranks them against each other at a cost quadratic in their number. A step that keeps
        //      many more than ef first drops those that cannot be among its best ef: a histogram of bins as for a
        //      start set finds the highest bin b such that the bins from b up hold at least ef candidates, and only those
        //      survive, compacted in place.
        //      Everything dropped is below at least ef survivors; which survive does not depend on
        //      the order of the candidates. The claimed ids (cid) are dead by now: their first 256
        //      words are the histogram.
        if (__builtin_expect(nk > ef + SR_PREFILTER_SLACK, 0) && nk <= SR_PREFILTER_REGS * T && maxc >= 256) {
            u64 mine[SR_PREFILTER_REGS];
            uint32_t lo = 0xffffffffu, hi = 0u;
#pragma unroll
            for (int r = 0; r < SR_PREFILTER_REGS; ++r) {
                const int c = r * T + tid;
                mine[r] = c < nk ? ckey[c] : 0ull;
                if (c < nk) {
                    const uint32_t sc = (uint32_t)(mine[r] >> 32);
                    lo = sc < lo ? sc : lo;
                    hi = sc > hi ? sc : hi;
                }
            }
            wave_min_max(lo, hi);
            if (lane == RA_WAVE - 1) {
                atomicMin(reinterpret_cast<unsigned int*>(&ctr[C_LO]), lo);
                atomicMax(reinterpret_cast<unsigned int*>(&ctr[C_HI]), hi);
            }
            if (tid < 256) cid[tid] = 0;
            __syncthreads();
            const ScoreBins score_bins((uint32_t)ctr[C_LO], (uint32_t)ctr[C_HI]);
            int bin[SR_PREFILTER_REGS];
#pragma unroll
            for (int r = 0; r < SR_PREFILTER_REGS; ++r) {
                bin[r] = score_bins.bin(mine[r]);
                if (r * T + tid < nk) atomicAdd(&cid[bin[r]], 1);
            }
            __syncthreads();
            if (wv == 0) {
                const int b0 = cid[4 * lane], b1 = cid[4 * lane + 1], b2 = cid[4 * lane + 2], b3 = cid[4 * lane + 3];
                const int incl = wave_incl_scan(b0 + b1 + b2 + b3);
                const int total = __builtin_amdgcn_readlane(incl, RA_WAVE - 1);
                const int from3 = total - incl + b3, from2 = from3 + b2, from1 = from2 + b1, from0 = from1 + b0;
                const int best = from3 >= ef ? 3 : from2 >= ef ? 2 : from1 >= ef ? 1 : from0 >= ef ? 0 : -1;
                const u64 has = __ballot(best >= 0);
                if (lane == 63 - __clzll(has)) ctr[C_BIN] = 4 * lane + best;
            }
            __syncthreads();
            const int bstar = ctr[C_BIN];
#pragma unroll
            for (int r = 0; r < SR_PREFILTER_REGS; ++r)
                if (r * T + tid < nk && bin[r] >= bstar) ckey[atomicAdd(&ctr[C_NSURV], 1)] = mine[r];
            __syncthreads();
            nk = ctr[C_NSURV];
        }
        SR_TICK(11);

        // ---- merge by rank into the other beam buffer, truncating at ef. The final position of
        //      an element of (beam u kept candidates) is the number of elements that beat it.
        //      A candidate: the beam entries above it (its slot) plus the candidates above it. A beam entry: its
        //      index plus the candidates whose slot is at or before it, a prefix sum over the histogram of
        //      slots. The same numbers give the count of *unexpanded* elements above each element (every
        //      candidate is unexpanded; for the beam's part urank has it), so the next step's picks, the elements with
        //      fewer than `expand` unexpanded ones above them, fall out of the merge.
        //      What bounds it is instructions: a wavefront or two per SIMD run a few hundred of them, 4 to 8 ticks each,
        //      16 for a comparison of 64 bits, 30 to 60 for a branch that lanes take apart or a test of two conditions
        //      (from vector to scalar unit and back), against 64 for a trip to LDS and 20 for a barrier. So places are
        //      searched and stored without branches, and three ways of counting the candidates above a candidate
        //      share the rest. Ticks of a merge of 65 to 116 candidates into 256 entries with 512 threads 3400 -> 2500, of 100
        //      into 2048 with 1024 threads 5200 -> 3900, of 350 into 512 15000 -> 5800, of 4 into 256 1240 -> 950;
        //      the calls: 50K keys, 2 sequences 38.4 -> 35.6 us, top-2000 185 -> 172, 1M keys 120 -> 114.6, one node per
        //      step, ef 256 397 -> 378. (Four lanes per candidate, 16-way search and all, were slower than one lane: three
        //      times the instructions.)
        const int bn_new = bn + nk < ef ? bn + nk : ef;
        auto place = [&](u64 k, int pos, int ur, auto beam) __attribute__((always_inline)) { place_in(bn_new, k, pos, ur, beam); };
        // beam entries above k, by a binary search of the same steps for every lane. (Entries from bn on are zero, and the last
        // one of a full beam is below every kept candidate, so index ef - 1 stands for all that follow.)
        typedef const __attribute__((address_space(3))) u64* lds_u64;
        const uint32_t cur_at = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)cur, cur_last = cur_at + (uint32_t)(ef - 1) * 8u;
        auto beam_above = [&](u64 k) __attribute__((always_inline)) {
            uint32_t at = cur_at - 8u;                        // of the entry before the b-th
            auto halve = [&](uint32_t half) __attribute__((always_inline)) {
                const uint32_t mid = at + half * 8u;
                at = *(lds_u64)(uintptr_t)min(mid, cur_last) > k ? mid : at;
            };
            static_assert(RA_MAX_EF <= 2048, "eleven steps");
            const int most = bn < ef ? bn : bn - 1;
            if (most >= 256) {
                if (most >= 512) {
                    if (most >= 1024) halve(1024);
                    halve(512);
                }
                halve(256);
            }
#pragma unroll
            for (int half = 128; half > 0; half >>= 1) halve(half);
            return (int)((at + 8u - cur_at) >> 3);
        };
        // (this step's picks, the first unexpanded entries, are marked expanded by now)
        auto unexpanded_above = [&](int b) __attribute__((always_inline)) { return max((int)urank[b] - np, 0); };
        // zeroes behind the candidates, written by each wavefront that reads them
        ckey[nk + lane16] = 0ull;
        // a beam entry with c candidates above it
        auto place_entry = [&](int e, u64 k, int ub, int c) __attribute__((always_inline)) {
            const int ur = c + ub, un = (int)(uint32_t)k & 1;
            place(k, e + c, ur, sr_int<1>{});
            const bool next = (uint32_t)((ur - expand) | (un - 1)) < (uint32_t)expand;           // in line after those picks
            if (__builtin_amdgcn_ballot_w64(next)) touch_row(next ? key_id(k) : e0);
        };
        // Places of the beam entries of this wavefront's 64s; left(h, before) says what stays in the histogram. What is behind
        // the last entry is zero and moves behind the new last one.
        auto place_beam = [&](auto left) __attribute__((always_inline)) {
            const int end = min(bn + 1, ef);
            if constexpr (HSUM) {
                // two of them at a time: the counts of both in one sum
                const int sums = wave_incl_scan(hsum[min(lane, nsum - 1)]);
                for (int base = __builtin_amdgcn_readfirstlane(wv * RA_WAVE); base < end; base += 2 * T) {
                    const int e = base + lane, ec = min(e, ef - 1), f = e + T, fc = min(f, ef - 1);
                    const bool two = base + T < end;
                    int* hp = hist + min(e, ef);
                    int* hq = hist + min(f, ef);
                    const int h = *hp;
                    const u64 k = cur[ec];
                    const int ub = unexpanded_above(ec);
                    int g = 0, uf = 0;
                    u64 kf = 0ull;
                    if (two) {
                        g = *hq;
                        kf = cur[fc];
                        uf = unexpanded_above(fc);
                    }
                    const int both = wave_incl_scan(h | g << 16);
                    const int c = (both & 0xffff) + (base ? __builtin_amdgcn_readlane(sums, base / RA_WAVE - 1) : 0);
                    *hp = left(h, c - h);
                    place_entry(e, k, ub, c);
                    if (two) {
                        const int cf = (int)((uint32_t)both >> 16) + __builtin_amdgcn_readlane(sums, (base + T) / RA_WAVE - 1);
                        *hq = left(g, cf - g);
                        place_entry(f, kf, uf, cf);
                    }
                }
            } else {
                for (int base = __builtin_amdgcn_readfirstlane(wv * RA_WAVE); base < end; base += T) {
                    const int e = base + lane, ec = min(e, ef - 1);
                    int* hp = hist + min(e, ef);
                    const int h = *hp;
                    const u64 k = cur[ec];
                    const int ub = unexpanded_above(ec);
                    int earlier = 0;
                    for (int x = 0; x < base; x += RA_WAVE) earlier += hist[x + lane] & 0xffff;
                    const int c = wave_incl_scan(h) + __builtin_amdgcn_readlane(wave_incl_scan(earlier), RA_WAVE - 1);
                    *hp = left(h, c - h);
                    place_entry(e, k, ub, c);
                }
            }
        };
        constexpr int NARROW = T == 1024 ? 2 * SR_NARROW : SR_NARROW;
        if (__builtin_expect(nk <= NARROW, 1)) {
            // ---- few candidates, one phase: 16 lanes find a candidate's place (its slot by a 16-way search, two or three
            //      dependent reads; the candidates above it by one or two comparisons per lane), and a beam entry is compared
            //      with every candidate, or in a wide beam with those in the range of its wavefront's 64 entries.
            static_assert(SR_NARROW == 16 && NARROW <= RA_WAVE, "a candidate or two per lane of a group, one per lane of a wavefront");
            auto count_group = [&](bool up) __attribute__((always_inline)) {         // lanes of the group of 16 that say so
                const u64 m = __builtin_amdgcn_ballot_w64(up);
                return __popc((lane & 32 ? (uint32_t)(m >> 32) : (uint32_t)m) >> (lane & 16) & 0xffffu);
            };
            for (int c0 = __builtin_amdgcn_readfirstlane((T / RA_WAVE - 1 - wv) * 4); c0 < nk; c0 += T / 16) {
                // (the groups past the last candidate do what the last one's does)
                const u64 k = ckey[min(c0 + (lane >> 4), nk - 1)];
                const u64 other = ckey[lane16], other2 = NARROW > 16 ? ckey[lane16 + 16] : 0ull;
                int b = 0;
                if (bn > 256) b = 256 * count_group(cur[min(lane16 * 256 + 255, ef - 1)] > k);
                b += 16 * count_group(cur[min(b + lane16 * 16 + 15, ef - 1)] > k);
                const u64 e = cur[min(b + lane16, ef - 1)];
                int ub = unexpanded_above(b);
                const bool up = e > k;
                b += count_group(up);
                ub += count_group(up && (e & 1ull));
                int n = count_group(lane16 < nk && other > k);
                if (NARROW > 16 && nk > 16) n += count_group(lane16 + 16 < nk && other2 > k);
                place(k, b + n, n + ub, sr_int<0>{});
                touch_row(key_id(k));
            }
            for (int base = __builtin_amdgcn_readfirstlane(wv * RA_WAVE); base < bn; base += T) {
                const int e = base + lane, ec = min(e, ef - 1);
                const u64 k = cur[ec];
                const int ub = unexpanded_above(ec);
                int c = 0;
                if constexpr (T == 1024) {
                    // (A candidate per lane; those above all 64 entries count for each, those among them are compared in turn. us per
                    // layer, every candidate compared with every entry and, behind the eighth, two phases -> this: 1024 / 12 nodes of
                    // degree 32 per step 230 -> 193, 1500 / 16 280 -> 237, 2048 / 8 719 -> 589, float32 2048 / 16 418 -> 348.)
                    const u64 own = lane < nk ? ckey[lane] : 0ull;
                    const u64 first = lane_key(k, 0), last = lane_key(k, RA_WAVE - 1);
                    const u64 above = __builtin_amdgcn_ballot_w64(own > first);
                    c = __popcll(above);
                    for (u64 among = __builtin_amdgcn_ballot_w64(own > last) & ~above; among; among &= among - 1ull)
                        c += lane_key(own, __builtin_ctzll(among)) > k ? 1 : 0;
                } else {
                    for (int i0 = 0; i0 < nk; i0 += 8) {
                        u64 v[8];
#pragma unroll
                        for (int u = 0; u < 8; ++u) v[u] = ckey[i0 + u];
#pragma unroll
                        for (int u = 0; u < 8; ++u) c += v[u] > k ? 1 : 0;
                    }
                }
                place_entry(e, k, ub, c);
            }
        } else if (nk > SR_DIRECT && nk <= SR_MERGE_REGS * T) {
            // ---- many: dealt into buckets by slot, and counted inside a bucket. (us per layer if from 17, 33, 65 and 129
            //      candidates on: top-2000 165.6, 165.6, 165.8, 173; 64K keys, 16 picks, ef 128 32.1, 30.8, 30.1, 30.1; two sequences
            //      of 50K keys 35.0, 34.9, 34.7, 35.2.)
            u64 mine[SR_MERGE_REGS];
            int at[SR_MERGE_REGS], o[SR_MERGE_REGS];
#pragma unroll
            for (int r = 0; r < SR_MERGE_REGS; ++r)
                if (r * T + tid < nk) {
                    mine[r] = ckey[r * T + tid];
                    touch_row(key_id(mine[r]));
                    at[r] = beam_above(mine[r]);
                    if constexpr (HSUM) atomicAdd(&hsum[at[r] >> 6], 1);
                    o[r] = atomicAdd(&hist[at[r]], 1);
                }
            __syncthreads();
            SR_TICK(8);
            hist_used = true;
            place_beam([&](int h, int before) __attribute__((always_inline)) { return h | before << 16; });
            __syncthreads();
            SR_TICK(9);
#pragma unroll
            for (int r = 0; r < SR_MERGE_REGS; ++r)
                if (r * T + tid < nk) ckey[(hist[at[r]] >> 16) + o[r]] = mine[r];
            __syncthreads();
            SR_TICK(3);
#pragma unroll
            for (int r = 0; r < SR_MERGE_REGS; ++r)
                if (r * T + tid < nk) {
                    const int hb = hist[at[r]], beg = hb >> 16, n = hb & 0xffff;
                    int c = beg, j0 = 0;
                    // (past the bucket's end its last key again, taken off below)
                    do {
                        u64 other[4];
#pragma unroll
                        for (int i = 0; i < 4; ++i) other[i] = ckey[beg + min(j0 + i, n - 1)];
#pragma unroll
                        for (int i = 0; i < 4; ++i) c += other[i] > mine[r] ? 1 : 0;
                        j0 += 4;
                    } while (__builtin_amdgcn_ballot_w64(j0 < n));
                    c -= ckey[beg + n - 1] > mine[r] ? j0 - n : 0;
                    place(mine[r], at[r] + c, c + unexpanded_above(at[r]), sr_int<0>{});
                }
        } else {
            // ---- the candidates above a candidate are counted, 16 at a time for 64 candidates, by the first wavefronts,
            //      while the last ones find the slots
            for (int c = T - 1 - tid; c < nk; c += T) {
                const u64 k = ckey[c];
                touch_row(key_id(k));
                const int b = beam_above(k);
                if constexpr (HSUM) atomicAdd(&hsum[b >> 6], 1);
                atomicAdd(&hist[b], 1);
                atomicAdd(&cnt[c], b << 16);                  // high half: beam entries above it
            }
            const int chunks = (nk + 15) >> 4;
            int t = __builtin_amdgcn_readfirstlane(wv);
            for (int g0 = 0; g0 < nk; g0 += RA_WAVE, t -= chunks)
                for (; t < chunks; t += T / RA_WAVE) {
                    const int c = min(g0 + lane, nk - 1);
                    const u64 k = ckey[c];
                    const int n = count16(t * 16, k, sr_int<0>{});
                    if (g0 + lane < nk && n) atomicAdd(&cnt[c], n);
                }
            __syncthreads();
            SR_TICK(8);
            place_beam([&](int h, int) __attribute__((always_inline)) { return HSUM ? 0 : h; });
            hist_used = hist_used || !HSUM;      // (others read it too)
            SR_TICK(9);
            for (int c = T - 1 - tid; c < nk; c += T) {
                const int both = cnt[c], n = both & 0xffff, b = both >> 16;
                cnt[c] = 0;
                const u64 k = ckey[c];
                place(k, b + n, n + unexpanded_above(b), sr_int<0>{});
            }
        }
        __syncthreads();
        SR_TICK(4);
        bn = bn_new;
        swap_beams();
    }

    if constexpr (Hook::kShareSteps) {
        post(0, 0ull);
        if (tid == 0) xwg_store(hook.area + SR_MSG_LAST, (u64)(last_message + (uint32_t)n_posted));
    }
    if constexpr (Hook::kShareSteps)
        if (ctr[C_MISSED]) {                 // (uniform: written before the last barrier)
            if (tid == 0) hook.steps_missed();
            __syncthreads();
            return -1;
        }
    // ---- result: best-first beam entries outside the static set W = [0,s) u [N-w,N), T entries at a time. (A row of ids has
    //      topk cells; this head returns at most `take` <= topk of them. 100 ids of 256 entries: 900 ticks, 1300 by the first
    //      wavefront alone.)
    int32_t* out = ids + (size_t)head * topk;
    const uint32_t eligible = (uint32_t)max((int)N - w - s, 0);
    int found = 0;
    for (int base = 0; base < bn && found < take; base += T) {          // (uniform)
        const int i = base + tid;
        const int at = i < bn ? key_id(cur[min(i, ef - 1)]) - s : -1;
        const bool ok = (uint32_t)at < eligible;
        const u64 mask = __builtin_amdgcn_ballot_w64(ok);
        if (base) __syncthreads();                                     // (wtot read)
        wtot[wv] = __popcll(mask);                                     // (the same from every lane)
        __syncthreads();
        const int upto = wave_incl_scan(lane < T / RA_WAVE ? wtot[lane] : 0);
        const int before = __builtin_amdgcn_readfirstlane(wv) ? __builtin_amdgcn_readlane(upto, __builtin_amdgcn_readfirstlane(wv) - 1) : 0;
        const int pos = ok ? found + before + __popcll(mask & ((1ull << lane) - 1ull)) : take;
        if (pos < take) {
            out[pos] = at + s;
            if (lds_ids) lds_ids[pos] = at + s;
        }
        found += __builtin_amdgcn_readlane(upto, T / RA_WAVE - 1);
    }
    if (found > take) found = take;
    for (int i = found + tid; i < topk; i += T) {
        out[i] = -1;
        if (lds_ids) lds_ids[i] = -1;
    }
    if (stats && tid == 0) {
        ra_stats st;
        st.n_visited = n_visited;
        st.n_expanded = n_expanded;
        st.n_iters = n_iters;
        st.n_returned = found;
        stats[head] = st;
    }
    __syncthreads();
    SR_TICK(6);
    SR_TICK_FLUSH;
    return found;
}


// Threads per search, of a launch of `heads` searches whose steps read up to `cells` adjacency cells. Merges
// and barriers, which make up a narrow walk's steps, go faster with fewer threads; gathers and merges of wide
// beams with more; and where searches outnumber the compute units (256), several small workgroups share one.
// Measured on the fused launch (us per layer, 32 searches over 128K keys of degree 32 unless said; start sets of 1024
// where a step has 1024 cells or more; 256 / 512 / 1024 threads):
//   ef <= 256, up to 384 searches: 512 threads. ef 256, 2048 cells: 30.6 / 24.5 / 24.8, 256 cells 70.9 / 63.5 / 69.2; ef 128, 2048
//     cells 22.9 / 18.0 / 18.8; 128 searches of 32K keys, ef 256 29.5 / 24.8 / 26.0, 384 of them 38.1 / 38.7 / 52.6.
//   ef <= 256, more searches: 256 threads. 512 searches of 32K keys, ef 128: 40.8 / 47.6 / 63.6, ef 256: 47.0 / 51.7 / 70.1.
//   At most 64 cells and 384 searches (one node per step, mostly): one size down. ef 48: 66.9 / 68.2 / 79.3, ef 128: 159.7 / 161.0 /
//     181.1; ef 300: 397 / 363 / 407, ef 512: 725 / 666 / 698. Over 48 cells 512 threads: degree 64, ef 256: 330 / 319 / 355.
//   ef 257 .. 1024 and at most 256 cells: 512. Four nodes, ef 300: 134 / 120 / 130, ef 384: 172 / 154 / 162.
//   ef 257 .. 1024 and more cells: 1024. ef 1024, 2048 cells: 114 / 84 / 68; ef 512: 52 / 41 / 35, 512 cells 96 / 81 / 78.
//     More than 256 searches, ef up to 512: 512 again, two of which share a compute unit. 320 searches of 32K
//     keys, ef 512: 61 / 57 / 75, ef 384: 45 / 43 / 62; 384 searches 63 / 58 / 82 and 47 / 45 / 64.
//   ef above 1024: 1024. 2048 cells: 320 / 217 / 140; 128 cells: 1672 / 1290 / 1107.
// Where the lines are not the best ones (same measurement, 256 / 512 / 1024 threads): ef 512 and 1024 with up to 256 cells (the
// latter from 32 cells on; 1024: 350 / 294 / 272, 512: 145 / 130 / 125), and ef 2048 with at most 64 (3052 / 2360 / 2068), which 1024 threads
// walk 4 to 14 % faster since they merge up to 32 candidates in one phase; ef 256 with at most 48 cells (322 / 311 / 346); ef 300 with 512 cells
// (57 / 48.5 / 52); 129 to 256 searches with ef 300 to 512, which with their helpers outnumber the compute units (256 of 32K keys, ef
// 384: 43.5 / 41.5 / 51.4); more than 256 searches with ef 1024 (320: 135 / 112 / 152) or with ef 2048 (128 cells: 1813 / 1548 / 2324); 512 searches
// with ef 300 and 384 (57 / 61 / 83).
static inline int search_threads(int heads, int ef, int cells) {
    if (cells <= 64 && heads <= 384) return ef > 256 || cells > 48 ? 512 : 256;
    if (ef > 1024) return 1024;
    if (ef > 256) return cells <= 256 || (heads > 256 && ef <= 512) ? 512 : 1024;
    return heads <= 384 ? 512 : 256;
}

// LDS bytes run_search needs.
static inline size_t search_lds_bytes(int64_t N, int deg, int ef, int expand, bool global_bitset) {
    const int maxc = expand * deg;
    size_t b = SR_TOUCH_BYTES + (size_t)2 * ef * 8 + (size_t)(maxc + 16) * 8 + (size_t)maxc * 4 +
               (size_t)(maxc + ef + 1 + (ef + 64) / 64) * 4 + (expand + C_COUNT) * 4 + (size_t)(ef + 1) * 4;
    if (!global_bitset) b += (size_t)((N + 31) >> 5) * 4;
    return b;
}
