// One launch per layer for the whole decode step of Algorithm 1 (fixed static pattern). A
// workgroup per (sequence, query head) runs the graph search (search_dev.h) and then, without
// leaving the compute unit, Eq. 2 over the retrieved set Omega for its head: the retrieved ids
// are still in LDS, the groups of 16 lanes share the rows round-robin, every group keeps an
// online (max, sum, weighted sum) over its rows, and the groups' partial results are combined
// with the re-scaling factors of Eq. 5 written for many sets (first across the four groups of a
// wavefront by lane exchange, then across the wavefronts through LDS), together with the
// (max, sum, weighted sum) of the static set W: carrying maxima across sets this way is the same
// arithmetic as computing o_W and o_Omega apart and combining them by Eq. 4.
//
// The attention over the static set W does not depend on the search, so it is taken off the
// head's critical path: the launch has one extra "helper" workgroup per (sequence, KV head) that
// reads the rows of W once for the whole GQA group and leaves (max, sum, weighted sums) per query
// head in a hand-over area; the head's workgroup picks its record up after the search and only
// attends to the retrieved rows itself. Helpers have the lowest workgroup ids, never wait for
// anything, and are finished before the first search is. (A launch with few searches has one
// helper per query head instead: see ra_launch_decode.)
//
// The hand-over uses no fence. A variant with agent-scope release/acquire was measured: the part
// has one L2 per XCD, so those fences write back and invalidate L2, about 18 us per launch, more
// than the whole attention. Instead the few words that cross workgroups are written and read with
// relaxed agent-scope atomics, which go around the non-coherent cache levels on their own: the
// helper stores its record in 64-bit words that say themselves whether they have come (a float and a
// 1), and the head polls them, then zeroes them for the next launch: no order between different words
// is needed. The wait is bounded: a head that does not see its record within the limit attends to W
// itself and turns the helpers off for later launches, so words that arrive late are never taken for
// the next launch's. Query heads of a GQA group still run on one XCD (xcd_aware_head) so that the key
// rows their searches have in common are served by that XCD's L2.
//
// A walk that starts from a seed set first scores the whole set, and what bounds that is the rate
// at which one compute unit takes in scattered key rows. A launch with few searches leaves most
// compute units idle, so it has "seed" workgroups as well (between the helpers and the heads):
// each scores one share of one head's set (score_seed_share) and stores the 64-bit keys in a
// hand-over area of their own, one slot per position of the set. A key is never zero and is one
// 64-bit store, so the slot itself says whether its key has come: the head's threads poll their
// slots (bounded), take the keys and zero the slots for the next launch. If a key does not come
// in time the head scores its set itself and switches the shares off for later launches. Same
// relaxed agent-scope accesses as above; no ordering between different words is needed at all.
#include <float.h>

#include "attend_dev.h"
#include "search_dev.h"


struct Softmax8 {          // a lane's share of an online-softmax state: 8 of the 128 outputs
    float m, l, acc[8];
};

// exp for the softmax weights: the hardware exponential for bf16 data (its error, about 1e-6
// relative for the exponents that matter, is far below the bf16 inputs'), the library one for fp32.
template <int DT>
__device__ __forceinline__ float sm_exp(float x) { return DT == RA_BF16 ? __expf(x) : expf(x); }

// One more row for a lane's online-softmax state: logit z, the lane's 8 values of the value row.
// The running maximum settles after a few rows, so the rescaling of the sums is skipped unless
// some lane of the wavefront sees a larger logit. (It starts from the lowest finite number: from -inf, a first row whose logit is
// -inf, which has no weight, would make the sums NaN; tests for that cost 1 % of a batch.)
template <int DT>
__device__ __forceinline__ void sm_row(Softmax8& st, float z, const float* v) {
    if (__builtin_amdgcn_ballot_w64(z > st.m) != 0ull) {
        const float mn = fmaxf(st.m, z);
        const float corr = sm_exp<DT>(st.m - mn);       // 0 on the first row
        st.l *= corr;
#pragma unroll
        for (int e = 0; e < 8; ++e) st.acc[e] *= corr;
        st.m = mn;
    }
    const float p = sm_exp<DT>(z - st.m);
    st.l += p;
#pragma unroll
    for (int e = 0; e < 8; ++e) st.acc[e] = fmaf(p, v[e], st.acc[e]);
}

// The 8 values of a key or value row that a lane owns, as float32.
template <int DT>
__device__ __forceinline__ void row_floats(const RowBits<DT>& r, float* f) {
    if (DT == RA_BF16) {
        f[0] = bf16_lo(r.a.x); f[1] = bf16_hi(r.a.x); f[2] = bf16_lo(r.a.y); f[3] = bf16_hi(r.a.y);
        f[4] = bf16_lo(r.a.z); f[5] = bf16_hi(r.a.z); f[6] = bf16_lo(r.a.w); f[7] = bf16_hi(r.a.w);
    } else {
        f[0] = __uint_as_float(r.a.x); f[1] = __uint_as_float(r.a.y);
        f[2] = __uint_as_float(r.a.z); f[3] = __uint_as_float(r.a.w);
        f[4] = __uint_as_float(r.b.x); f[5] = __uint_as_float(r.b.y);
        f[6] = __uint_as_float(r.b.z); f[7] = __uint_as_float(r.b.w);
    }
}

// a row of zeroes
__device__ static const uint4 no_row[RA_D / 4] = {};

// A lane's 8 query values in the form the attention logits want them: bf16 pairs stay packed and
// go through the two-element dot instruction (exact products, float32 sums), fp32 uses fma.
// (The search scores are not computed here: they decide ids and keep their own fixed order.)
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
template <int DT> struct LaneQuery;
template <> struct LaneQuery<RA_BF16> {
    uint4 q;
    __device__ __forceinline__ void load(const void* qrow, int lane16) {
        q = reinterpret_cast<const uint4*>(qrow)[lane16];
    }
    __device__ __forceinline__ float dot(const RowBits<RA_BF16>& k) const {
        float d = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, q.x), __builtin_bit_cast(bf16x2, k.a.x), 0.f, false);
        d = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, q.y), __builtin_bit_cast(bf16x2, k.a.y), d, false);
        d = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, q.z), __builtin_bit_cast(bf16x2, k.a.z), d, false);
        d = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, q.w), __builtin_bit_cast(bf16x2, k.a.w), d, false);
        return d;
    }
};
template <> struct LaneQuery<RA_F32> {
    float q[8];
    __device__ __forceinline__ void load(const void* qrow, int lane16) { load_q8<RA_F32>(qrow, lane16, q); }
    __device__ __forceinline__ float dot(const RowBits<RA_F32>& k) const {
        float f[8];
        row_floats<RA_F32>(k, f);
        float d = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) d = fmaf(q[e], f[e], d);
        return d;
    }
};

// The largest, or the sum, of x over lanes lane ^ {0, 16, 32, 48}, by the vector unit's row and half exchanges (a shuffle is a trip
// through LDS): of a register swapped with itself one result has the value of each pair's first lane, the other the second's.
__device__ __forceinline__ float rows_max(float x) {
    auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fmaxf(__uint_as_float(p[0]), __uint_as_float(p[1]));
    p = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(p[0]), __uint_as_float(p[1]));
}
__device__ __forceinline__ float rows_sum(float x) {
    auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(p[0]) + __uint_as_float(p[1]);
    p = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(p[0]) + __uint_as_float(p[1]);
}

// Combine the online-softmax states of the lane groups of a workgroup of T threads into one (max,
// sum, weighted sum for output `tid`), valid in threads tid < 128 (T >= 128): first the four
// groups of each wavefront by lane exchange, then the T/64 wavefronts through LDS (T/64 * 130
// floats at `lds`). Two barriers.
template <int T>
__device__ __forceinline__ void sm_combine(Softmax8 st, float* lds, int tid, float& mx, float& l, float& a) {
    const int lane = tid & (RA_WAVE - 1), wv = tid / RA_WAVE;
    // one maximum for the wavefront, one exponential per lane, sums (an empty state has the sum 0 and exp(-inf) = 0)
    const float m = rows_max(st.m);
    const float c = expf(st.m - (m > -INFINITY ? m : 0.f));
    st.l = rows_sum(st.l * c);
#pragma unroll
    for (int e = 0; e < 8; ++e) st.acc[e] = rows_sum(st.acc[e] * c);
    float* sm = lds;                                         // [16]
    float* sl = sm + T / RA_WAVE;                   // [16]
    float* sa = sl + T / RA_WAVE;                   // [16][128]
    __syncthreads();                                         // whatever was in `lds` is dead
    if (lane < 16) {
        if (lane == 0) {
            sm[wv] = m;
            sl[wv] = st.l;
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) sa[wv * RA_D + lane * 8 + e] = st.acc[e];
    }
    __syncthreads();
    mx = -INFINITY;
    a = 0.f;
    l = 0.f;
    if (tid < RA_D) {
#pragma unroll
        for (int j = 0; j < T / RA_WAVE; ++j) mx = fmaxf(mx, sm[j]);
        if (mx > -INFINITY) {
            // (a lane works out the weight of one wavefront's share; each weight is then read from its lane)
            const float own = expf(sm[lane & (T / RA_WAVE - 1)] - mx);
#pragma unroll
            for (int j = 0; j < T / RA_WAVE; ++j) {
                const float wgt = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(own), j));
                a = fmaf(sa[j * RA_D + tid], wgt, a);
                l = fmaf(sl[j], wgt, l);
            }
        }
    }
}

// A word of a helper's record: a float's bits, and in the upper half a 1 that says it has come.
__device__ __forceinline__ u64 rec_word(float v) { return (1ull << 32) | __float_as_uint(v); }
__device__ __forceinline__ bool rec_came(u64 w) { return (w >> 32) != 0ull; }
__device__ __forceinline__ float rec_value(u64 w) { return __uint_as_float((uint32_t)w); }

// Helper workgroup: Eq. 2 over W for NH query heads that share one KV head (heads head0 ..
// head0 + NH - 1), each row of W read once; leaves one record per head.
template <int DT, int NH, int T>
__device__ __forceinline__ void static_helper(unsigned char* lds_raw, const void* q, int head0, const char* Kh,
                                              const char* Vh, int s, int64_t wstart, int64_t N, float scale,
                                              u64* rec, bool off) {
    const int tid = threadIdx.x, grp = tid >> 4, lane16 = tid & 15;
    const size_t esz = DT == RA_BF16 ? 2 : 4;
    constexpr int ROWS = DT == RA_BF16 ? 4 : 2;              // rows in flight per 16-lane group
    LaneQuery<DT> ql[NH];
    Softmax8 st[NH];
#pragma unroll
    for (int h = 0; h < NH; ++h) {
        ql[h].load(reinterpret_cast<const char*>(q) + (size_t)(head0 + h) * RA_D * esz, lane16);
        st[h].m = -FLT_MAX;
        st[h].l = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) st[h].acc[e] = 0.f;
    }
    const int R = s + (int)(N - wstart);
    for (int r0 = 0; r0 < R; r0 += (T / 16) * ROWS) {
        bool live[ROWS];
        RowBits<DT> kb[ROWS], vb[ROWS];
#pragma unroll
        for (int u = 0; u < ROWS; ++u) {
            const int r = r0 + u * (T / 16) + grp;
            live[u] = r < R;
            const int64_t id = !live[u] ? 0 : r < s ? (int64_t)r : wstart + (r - s);   // loads stay unconditional
            kb[u] = load_key<DT>(Kh, id, lane16);
            vb[u] = load_key<DT>(Vh, id, lane16);
        }
#pragma unroll
        for (int u = 0; u < ROWS; ++u) {
            if (!live[u]) continue;
            float v[8];
            row_floats<DT>(vb[u], v);
#pragma unroll
            for (int h = 0; h < NH; ++h) {
                float dot = ql[h].dot(kb[u]);
                dot += at_dpp<0xB1>(dot);
                dot += at_dpp<0x4E>(dot);
                dot += at_dpp<0x141>(dot);
                dot += at_dpp<0x140>(dot);
                sm_row<DT>(st[h], dot * scale, v);
            }
        }
    }
#pragma unroll
    for (int h = 0; h < NH; ++h) {
        float mx, l, a;
        sm_combine<T>(st[h], reinterpret_cast<float*>(lds_raw), tid, mx, l, a);
        if (tid < RA_D && !off) {
            u64* r = rec + (size_t)(head0 + h) * RA_COOP_REC;
            if (tid == 0) {
                xwg_store(r, rec_word(mx));
                xwg_store(r + 1, rec_word(l));
            }
            xwg_store(r + 2 + tid, rec_word(a));
        }
    }
}

// "Helpers off" and "shares off" as this wavefront has read them, and the words in LDS where the workgroup's first thread leaves
// what it has read for all ([1] and [2]). Read back as scalars: with a branch per lane, behind the claims, four layers of 128K
// took 0.7 % longer (95.6 against 94.9 us) and a beam of 2048 0.4 %.
struct OffWords {
    uint32_t helpers, shares;
    uint32_t* lds;
    __device__ __forceinline__ void note() const {
        lds[1] = helpers;
        lds[2] = shares;
    }
};

// What the walk asks of the fused launch (see NoHook): the keys of its start set, scored by other workgroups.
template <int DT> struct SeedHook {
    int spin;
    // this head's keys in the seed hand-over area, the area's "shares off" word, whether the launch
    // has seed workgroups
    u64* seed_keys;
    uint32_t* seed_off;
    bool seed_on;
    OffWords off;
    static constexpr bool kSeedShare = true;
    static constexpr bool kShareSteps = false;
    // value rows
    const char* V;
    static constexpr bool kValues = DT == RA_BF16;
    static constexpr int value_lines = 2;
    __device__ __forceinline__ void touch_value(int id, int line, uint32_t lds) const {
        touch_line_of_halves(V + ((size_t)(uint32_t)id * value_lines + line) * 128, lds);       // (V: aligned to its elements)
    }
    __device__ __forceinline__ void note_off_words() const { off.note(); }
    __device__ __forceinline__ bool seeds_shared() const { return seed_on && __builtin_amdgcn_readfirstlane((int)off.lds[2]) == 0; }
    // Keys c0 and c1 of the head's start set (c1 < 0: only c0, and k1 = k0), polled together a bounded
    // number of times, the slots zeroed for the next launch once the keys are taken; a key that did
    // not come reads 0. A poll is a trip to memory (agent-scope loads go around the caches); more
    // than one in flight per slot was measured and is slower.
    __device__ __forceinline__ void take_seed_keys(int c0, int c1, u64& k0, u64& k1) const {
        u64* p0 = seed_keys + c0;
        u64* p1 = seed_keys + (c1 >= 0 ? c1 : c0);
        k0 = 0ull;
        k1 = 0ull;
        for (int i = 0; i < spin; ++i) {
            if (k0 == 0ull) k0 = xwg_load(p0);               // (a slot whose key has come is not read again)
            if (k1 == 0ull) k1 = xwg_load(p1);
            if (k0 != 0ull && k1 != 0ull) break;
            __builtin_amdgcn_s_sleep(6);
        }
        if (k0 != 0ull) xwg_store(p0, 0ull);
        if (c1 >= 0 && k1 != 0ull) xwg_store(p1, 0ull);
    }
    // a key did not come: later launches score in the head again, so that keys that arrive late
    // are never taken for a later launch's
    __device__ __forceinline__ void seeds_missed() const { xwg_store(seed_off, 1u); }
};

// What a walk that shares its steps asks of the launch.
struct WalkHook {
    int spin, parts_log2;
    u64* area;
    uint32_t* off_word;
    uint32_t* missed;       // in host memory
    OffWords off;
    static constexpr bool kSeedShare = false;
    static constexpr bool kShareSteps = true;
    static constexpr bool kValues = false;
    __device__ __forceinline__ void note_off_words() const { off.note(); }
    __device__ __forceinline__ bool steps_shared() const { return __builtin_amdgcn_readfirstlane((int)off.lds[2]) == 0; }
    __device__ __forceinline__ void steps_missed() const {
        xwg_store(off_word, 1u);
        __hip_atomic_store(missed, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
};

// What the launch adds for walks that share their steps (serve_walk): `heads` of them with 2^parts_log2 workers each, areas from
// `words`, `missed` in host memory. A type of its own, so that the common kernel has neither the arguments nor the code.
struct NoWalk {
    static constexpr bool kShare = false;
};
struct SharedWalk {
    static constexpr bool kShare = true;
    u64* words;
    uint32_t* missed;
    int heads, parts_log2;
    __device__ __forceinline__ uint32_t* off_word() const { return reinterpret_cast<uint32_t*>(words); }
    __device__ __forceinline__ u64* area(int head) const {
        return words + RA_WALK_OFF_WORDS + (size_t)head * (RA_WALK_HEAD_WORDS + ((size_t)RA_WALK_PART_WORDS << parts_log2));
    }
};

// BUDGETS: every head keeps its own number of ids (budgets[head]) instead of topk. A variant of
// its own because the value lives through the whole walk: read in the common kernel, even behind a
// test for a null pointer, it cost 1.5 % of the step.
// With a SharedWalk, workgroup x of the first 8 * ceil(heads / 8) * (1 + workers) runs on the XCD of its head's others (x mod 8, if
// workgroups are dealt round-robin): the workers of a head read the same adjacency rows, and a hand-over inside an XCD is a
// quarter shorter. The heads come first, then the workers; helpers have the highest ids.
template <int DT, int KT, bool GBITS, int T, bool BUDGETS, typename Walk>
__global__ __launch_bounds__(T, SR_WAVES(KT, T)) void decode_kernel(
    const void* __restrict__ q, const int32_t* __restrict__ adj, const int32_t* __restrict__ entry,
    const void* __restrict__ K, const void* __restrict__ V, int n_q, int n_kv, int64_t Ng, int64_t N,
    int64_t kv_stride, int64_t wstart, int deg, int s, int topk, int ef, int expand,
    uint32_t* __restrict__ gbits,
    int32_t* __restrict__ ids, ra_stats* __restrict__ stats, int ids_off, float scale,
    float* __restrict__ out, float* __restrict__ lse, u64* coop, int n_helpers, int coop_mode,
    int coop_spin, const int32_t* __restrict__ roots, int root_cap, const void* __restrict__ Ksearch,
    const float* __restrict__ kscale, const int32_t* __restrict__ budgets, uint32_t* seedx, int seed_parts,
    int seed_stride, int helper_heads, Walk walk) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const int tid = threadIdx.x, grp = tid >> 4, lane16 = tid & 15;
    const size_t esz = DT == RA_BF16 ? 2 : 4;
    const int G = n_q / n_kv;
    int n_heads, helper = (int)blockIdx.x;                   // (helper: in [0, n_helpers) of a helper workgroup)
    if constexpr (Walk::kShare) {
        n_heads = walk.heads;
        helper -= (int)gridDim.x - n_helpers;
    } else {
        n_heads = ((int)gridDim.x - n_helpers) / (1 + seed_parts);
    }
    // hand-over area: records, "helpers off" word (set by a head whose wait ran out); seed hand-over area: [0]
    // the "shares off" word, then (from byte RA_SEEDX_KEYS_OFF) seed_stride 64-bit keys per head, zero
    // between launches. Both words are asked for here, together, and looked at where they are needed: a
    // trip past the caches is a microsecond.
    uint32_t* helpers_off_word = reinterpret_cast<uint32_t*>(coop + (size_t)n_heads * RA_COOP_REC);
    const uint32_t helpers_off = xwg_load(helpers_off_word);
    uint32_t* shares_off_word = seedx ? seedx : helpers_off_word;
    if constexpr (Walk::kShare) shares_off_word = walk.off_word();
    const uint32_t shares_off = xwg_load(shares_off_word);
    if (Walk::kShare ? helper >= 0 : helper < n_helpers) {
        // ---- helper workgroup of (sequence, KV head) blockIdx.x: attention over W for its G heads
        if (coop_mode == RA_HELPERS_SILENT_) return;
        // helper_heads of the group's G query heads per helper workgroup (G: one helper per group, W
        // read once; fewer where the launch leaves compute units idle: the helpers of a group then
        // run side by side on one XCD and share the rows in its L2)
        const int n_groups = n_heads / G;
        const int g = helper % n_groups, part = helper / n_groups;
        const char* Kg = reinterpret_cast<const char*>(K) + (size_t)g * kv_stride * RA_D * esz;
        const char* Vg = reinterpret_cast<const char*>(V) + (size_t)g * kv_stride * RA_D * esz;
        // G is 1, 2, 4 or 8 when helpers are on; 4 heads per pass over W (2 for fp32: registers)
        constexpr int PASS = DT == RA_BF16 ? 4 : 2;
        const int h_end = (part + 1) * helper_heads;
        for (int h0 = part * helper_heads; h0 < h_end; h0 += PASS) {
            const int head0 = g * G + h0;
            if (h_end - h0 >= PASS) static_helper<DT, PASS, T>(lds_raw, q, head0, Kg, Vg, s, wstart, N, scale, coop, helpers_off != 0u);
            else if (h_end - h0 == 2) static_helper<DT, 2, T>(lds_raw, q, head0, Kg, Vg, s, wstart, N, scale, coop, helpers_off != 0u);
            else static_helper<DT, 1, T>(lds_raw, q, head0, Kg, Vg, s, wstart, N, scale, coop, helpers_off != 0u);
        }
        return;
    }
    u64* seed_keys_all = reinterpret_cast<u64*>(reinterpret_cast<char*>(seedx) + RA_SEEDX_KEYS_OFF);
    int head;
    if constexpr (Walk::kShare) {
        // ---- the head (role 0), or one of its workers: all heads, then all first workers, and so on
        const int rows = (n_heads + 7) >> 3, j = (int)blockIdx.x >> 3, role = j / rows;
        head = ((j - role * rows) << 3) + ((int)blockIdx.x & 7);
        if (head >= n_heads || role > 1 << walk.parts_log2) return;
        if (role > 0) {
            if (coop_mode == RA_HELPERS_SILENT_) return;
            serve_walk<DT, KT, T>(lds_raw, head, role - 1, walk.parts_log2, q, adj, entry, Ksearch, n_q, n_kv, Ng, kv_stride, deg, ef, expand,
                                  roots, root_cap, kscale, walk.area(head), shares_off, coop_spin);
            return;
        }
    } else {
        if ((int)blockIdx.x < n_helpers + n_heads * seed_parts) {
            // ---- seed workgroup: one share of one head's start set (on the XCD of the head's workgroup
            //      when the number of heads is a multiple of 8)
            if (coop_mode == RA_HELPERS_SILENT_ || shares_off != 0u) return;
            const int i = (int)blockIdx.x - n_helpers;
            const int part = i / n_heads, hd = xcd_aware_head(i % n_heads, n_heads, G);
            score_seed_share<DT, KT, T>(hd, part, seed_parts, q, Ksearch, n_q, n_kv, kv_stride, roots, root_cap,
                                        seed_stride, expand * deg, kscale, seed_keys_all + (size_t)hd * seed_stride);
            return;
        }
        head = xcd_aware_head((int)blockIdx.x - n_helpers - n_heads * seed_parts, n_heads, G);
    }
    const int seq = head / n_q, h = head % n_q, kvh = h / G;
    int32_t* lds_ids = reinterpret_cast<int32_t*>(lds_raw + ids_off);
    uint32_t* lds_word = reinterpret_cast<uint32_t*>(lds_ids + topk);
    const char* Kh = reinterpret_cast<const char*>(K) + ((size_t)seq * n_kv + kvh) * kv_stride * RA_D * esz;
    const char* Vh = reinterpret_cast<const char*>(V) + ((size_t)seq * n_kv + kvh) * kv_stride * RA_D * esz;
    // The graph covers the first Ng of the N tokens now in the cache; W = [0, s) u [wstart, N) with
    // wstart <= Ng, so every token appended after the build is attended densely.
    // the walk scores Ksearch: K itself, or its 8-bit copy (with kscale)
    // ids kept for this head: topk, or its own budget clamped into [1, topk]
    int take = topk;
    if constexpr (BUDGETS) {
        const int b = budgets[head];
        take = b < 1 ? 1 : b > topk ? topk : b;
    }
    const OffWords off{helpers_off, shares_off, lds_word};
    int cnt;
    if constexpr (Walk::kShare) {
        cnt = run_search<DT, KT, GBITS, T>(lds_raw, head, q, adj, entry, Ksearch, n_q, n_kv, Ng, kv_stride, deg,
                                           s, (int)(Ng - wstart), topk, take, ef, expand, gbits, ids, stats,
                                           lds_ids, roots, root_cap, kscale,
                                           WalkHook{coop_spin, walk.parts_log2, walk.area(head), walk.off_word(), walk.missed, off});
        if (cnt < 0)                                         // alone: the workers have not answered, now or earlier
            cnt = run_search<DT, KT, GBITS, T>(lds_raw, head, q, adj, entry, Ksearch, n_q, n_kv, Ng, kv_stride, deg,
                                               s, (int)(Ng - wstart), topk, take, ef, expand, gbits, ids, stats,
                                               lds_ids, roots, root_cap, kscale, NoHook{});
    } else {
        cnt = run_search<DT, KT, GBITS, T>(lds_raw, head, q, adj, entry, Ksearch, n_q, n_kv, Ng, kv_stride, deg,
                                           s, (int)(Ng - wstart), topk, take, ef, expand, gbits, ids, stats,
                                           lds_ids, roots, root_cap, kscale,
                                           SeedHook<DT>{coop_spin, seed_keys_all + (size_t)head * seed_stride, seedx,
                                                    seed_parts > 0, off, Vh});
    }
#ifdef SR_PHASE_CLOCKS
    const long long t_attn = clock64();
#endif
    // ---- Eq. 2 over Omega (rows [0, cnt): ids in LDS) and, in a launch without helpers, W (the n_w rows after
    //      them). The helper's record is asked for behind the first rows, so that its trip past the caches
    //      is over when they have been attended to (asking for a ready word first, when the walk had
    //      ended, and then for the record took a microsecond of every step).
    const bool helpers = n_helpers > 0 && __builtin_amdgcn_readfirstlane((int)lds_word[1]) == 0;
    u64* rec = coop + (size_t)head * RA_COOP_REC;
    u64 w_mx = 0ull, w_l = 0ull, w_a = 0ull;
    LaneQuery<DT> ql;
    ql.load(reinterpret_cast<const char*>(q) + (size_t)head * RA_D * esz, lane16);
    // rows in flight per 16-lane group: a hundred in one trip with 256 threads, too (16 sequences of 32K 45.6 -> 44.9 us)
    constexpr int DC_ROWS = DT == RA_BF16 ? (T == 256 ? 7 : 6) : 3;
    // attention over the R rows row_id(0 ..) of K and V; `behind` is called once, after the first loads
    auto attend_rows = [&](int R, auto row_id, auto behind) __attribute__((always_inline)) {
        Softmax8 st;
        st.m = -INFINITY;
        st.l = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) st.acc[e] = 0.f;
        if (R <= 0) behind();
        for (int r0 = 0; r0 < R; r0 += (T / 16) * DC_ROWS) {
            RowBits<DT> kb[DC_ROWS], vb[DC_ROWS];
            float z[DC_ROWS];
#pragma unroll
            for (int u = 0; u < DC_ROWS; ++u) {
                if (r0 + u * (T / 16) >= R) break;          // uniform: no group has a row in this slot
                const int64_t id = row_id(min(r0 + u * (T / 16) + grp, R - 1));
                kb[u] = load_key<DT>(Kh, id, lane16);
                // (a group without a row has the weight zero, and values of zero, since 0 * inf is not: clearing what it has loaded took
                // four layers of 128K 1.1 % longer, this 0.1 %)
                vb[u] = load_key<DT>(r0 + u * (T / 16) + grp < R ? Vh + id * (RA_D * (DT == RA_BF16 ? 2 : 4))
                                                                 : reinterpret_cast<const char*>(no_row), 0, lane16);
            }
            if (r0 == 0) behind();
            // the logits, their maximum, then one rescaling of the sums for all of them (row by row, with a branch around the
            // rescaling, 100 rows took 3700 ticks)
            float m = st.m;
#pragma unroll
            for (int u = 0; u < DC_ROWS; ++u) {
                z[u] = -INFINITY;
                if (r0 + u * (T / 16) >= R) continue;
                float dot = ql.dot(kb[u]);
                dot += at_dpp<0xB1>(dot);
                dot += at_dpp<0x4E>(dot);
                dot += at_dpp<0x141>(dot);
                dot += at_dpp<0x140>(dot);
                z[u] = r0 + u * (T / 16) + grp < R ? dot * scale : -INFINITY;
                m = fmaxf(m, z[u]);
            }
            const float m0 = m > -INFINITY ? m : 0.f, corr = sm_exp<DT>(st.m - m0);        // (exp(-inf) = 0: no row yet)
            st.m = m;
            st.l *= corr;
#pragma unroll
            for (int e = 0; e < 8; ++e) st.acc[e] *= corr;
#pragma unroll
            for (int u = 0; u < DC_ROWS; ++u) {
                if (r0 + u * (T / 16) >= R) break;
                const float p = sm_exp<DT>(z[u] - m0);
                float v[8];
                row_floats<DT>(vb[u], v);
                st.l += p;
#pragma unroll
                for (int e = 0; e < 8; ++e) st.acc[e] = fmaf(p, v[e], st.acc[e]);
            }
        }
        return st;
    };
    const int n_w = s + (int)(N - wstart);
    auto w_row = [&](int r) { return r < s ? (int64_t)r : wstart + (r - s); };
    if (tid == 0) *lds_word = 0u;
    const Softmax8 st_om = attend_rows(
        cnt + (helpers ? 0 : n_w), [&](int r) { return r < cnt ? (int64_t)lds_ids[r] : w_row(r - cnt); },
        [&]() {
            if (helpers && tid < RA_D) {
                w_mx = xwg_load(rec);
                w_l = xwg_load(rec + 1);
                w_a = xwg_load(rec + 2 + tid);
            }
        });
    float mx, l, a;
    float* const scratch = reinterpret_cast<float*>(lds_raw + SR_TOUCH_BYTES);       // (touched words may still land in front of it)
    sm_combine<T>(st_om, scratch, tid, mx, l, a);
    // ---- the record, waited for a bounded number of polls; without it, W by this workgroup itself, and
    //      no helpers in later launches
    float mw = -INFINITY, lw = 0.f, aw = 0.f;
    bool have_w = false;
    if (helpers) {
        if (tid < RA_D) {
            for (int i = 0; i < coop_spin && !(rec_came(w_mx) && rec_came(w_l) && rec_came(w_a)); ++i) {
                __builtin_amdgcn_s_sleep(6);
                w_mx = xwg_load(rec);
                w_l = xwg_load(rec + 1);
                w_a = xwg_load(rec + 2 + tid);
            }
            if (rec_came(w_mx) && rec_came(w_l) && rec_came(w_a)) {
                mw = rec_value(w_mx);
                lw = rec_value(w_l);
                aw = rec_value(w_a);
            } else {
                *lds_word = 1u;
            }
        }
        __syncthreads();
        have_w = *lds_word == 0u;
        if (!have_w) {
            if (tid == 0) xwg_store(helpers_off_word, 1u);
            const Softmax8 st_w = attend_rows(n_w, w_row, []() {});
            sm_combine<T>(st_w, scratch, tid, mw, lw, aw);
        }
    }
    // ---- Eq. 4-5: the two sets re-scaled to one maximum
    if (tid < RA_D) {
        const float m2 = fmaxf(mx, mw);
        if (m2 > -INFINITY) {
            const float c1 = expf(mx - m2), c2 = expf(mw - m2);
            a = a * c1 + aw * c2;
            l = l * c1 + lw * c2;
        }
        const bool empty = !(l > 0.f);
        out[(size_t)head * RA_D + tid] = empty ? 0.f : a / l;
        if (tid == RA_WAVE) lse[head] = empty ? -INFINITY : m2 + logf(l);         // (by the second wavefront: the first has the record's last words)
        if (have_w) {                                        // taken: the next launch starts from zero
            xwg_store(rec + 2 + tid, 0ull);
            if (tid < 2) xwg_store(rec + tid, 0ull);
        }
    }
    end_touches();
#ifdef SR_PHASE_CLOCKS
    if (tid == 0 && head < 64) sr_phase_ticks[head * SR_NITER * SR_NPHASE + 7] += clock64() - t_attn;
#endif
}

#ifdef SR_PHASE_CLOCKS
// Tuning builds only: copy the phase clocks of the fused kernel to `host` (64 x SR_NITER x SR_NPHASE values:
// search, step, phase) and clear them.
#ifdef SR_WAVE_CLOCKS
extern "C" int ra_dbg_wave_ticks(long long* host) {
    return hipMemcpyFromSymbol(host, HIP_SYMBOL(sr_wave_ticks), sizeof(long long) * SR_NWAVE) != hipSuccess;
}
#endif
extern "C" int ra_dbg_phase_ticks(long long* host) {
    if (hipMemcpyFromSymbol(host, HIP_SYMBOL(sr_phase_ticks), sizeof(long long) * 64 * SR_NITER * SR_NPHASE) != hipSuccess)
        return 1;
    static long long zeros[64 * SR_NITER * SR_NPHASE];
    return hipMemcpyToSymbol(HIP_SYMBOL(sr_phase_ticks), zeros, sizeof(zeros)) != hipSuccess;
}
#endif

static size_t decode_lds_bytes(int64_t N, int deg, int ef, int expand, int topk, bool gb, int* ids_off) {
    size_t a = search_lds_bytes(N, deg, ef, expand, gb);
    const size_t b = SR_TOUCH_BYTES + (size_t)(SR_THREADS / RA_WAVE) * (RA_D + 2) * sizeof(float);
    if (b > a) a = b;
    a = (a + 15) & ~(size_t)15;
    *ids_off = (int)a;
    return a + (size_t)topk * sizeof(int32_t) + 16;        // ids, then words for the record that did not come and for OffWords
}

bool ra_decode_needs_global_bitset(int64_t N, int deg, int ef, int expand, int topk) {
    int off;
    return (size_t)((N + 31) >> 5) * 4 > SR_BITSET_LDS_MAX ||
           decode_lds_bytes(N, deg, ef, expand, topk, false, &off) > SR_LDS_LIMIT;
}

// helper workgroups in front of the heads' in a decode launch: one per (sequence, KV head), for
// GQA groups of 1, 2, 4 or 8 while the handle has them switched on
static int decode_helper_slots(const unsigned long long* coop, int coop_mode, int n_seq, int n_q, int n_kv) {
    const int G = n_q / n_kv;
    const bool coop_on = coop && coop_mode != RA_HELPERS_OFF && (G == 1 || G == 2 || G == 4 || G == 8);
    return coop_on ? n_seq * n_kv : 0;
}

// compute units of the current device (asked once per device)
static int decode_compute_units() {
    static int cached[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
    if (cached[dev] == 0) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) n = 0;
        cached[dev] = n > 0 ? n : -1;
    }
    return cached[dev] > 0 ? cached[dev] : 0;
}

// (below RA_WALK_MIN_KEYS the visited set of steps of up to RA_WALK_CELLS cells always fits LDS). A head and its workers are on one
// XCD, and one of their workgroups fills a compute unit: of every eighth head an XCD has the head, at most one helper and
// the workers, all of which have to run at once, or heads wait for workers that have no compute unit. On 256 compute units 16
// workers for up to 8 heads, 8 for up to 24. (Counted over the whole device, 9 to 14 heads had 34 workgroups for an XCD's 32
// compute units: their first wait ran out and steps were shared no more.)
int ra_walk_parts(int heads, int64_t N) {
    if (N < RA_WALK_MIN_KEYS) return 0;
    const int room = decode_compute_units() / 8 / ((heads + 7) / 8) - 2;
    return room >= RA_WALK_PARTS_MAX ? RA_WALK_PARTS_MAX : room >= 8 && RA_WALK_PARTS_MAX >= 8 ? 8 : 0;
}

ra_status ra_launch_decode(const void* q, const int32_t* adj, const int32_t* entry, const void* K,
                           const void* V, ra_dtype dt, int n_seq, int n_q, int n_kv, int64_t Ng, int64_t N,
                           int64_t kv_stride, int deg, int sink, int window, int topk, int ef, int expand,
                           uint32_t* bitset, unsigned long long* coop, int coop_mode, int coop_spin,
                           const int32_t* roots, int root_cap, const void* K8, const float* kscale,
                           const int32_t* budgets, uint32_t* seedx, int seed_parts, unsigned long long* walk, int walk_parts,
                           uint32_t* walk_missed, int64_t* walk_launches, hipStream_t st, float* out, float* lse, int32_t* ids, ra_stats* stats) {
    // W = [0, s) u [wstart, N): the sink, the sliding window, and every token appended after the
    // index was built (wstart <= Ng); overlapping ranges make everything static
    int64_t s = sink < 0 ? 0 : sink, ww = window < 0 ? 0 : window;
    if (s > N) s = N;
    if (ww > N) ww = N;
    int64_t wstart = N - ww < Ng ? N - ww : Ng;
    if (s >= wstart) { s = 0; wstart = 0; }
    if (N - wstart + s > 0x3fffffff) RA_FAIL(RA_EUNSUP, "static set too large");
    const int heads = n_seq * n_q;
    const bool gb = ra_decode_needs_global_bitset(Ng, deg, ef, expand, topk);
    int ids_off;
    const size_t lds = decode_lds_bytes(Ng, deg, ef, expand, topk, gb, &ids_off);
    if (lds > SR_LDS_LIMIT)
        RA_FAIL(RA_EUNSUP, "decode state needs %zu B of LDS (limit %d): lower ef or expand", lds,
                SR_LDS_LIMIT);
    if (gb && !bitset) RA_FAIL(RA_EINVAL, "global visited bitset missing");
    const float scale = 1.0f / sqrtf((float)RA_D);
    // one helper workgroup per (sequence, KV head) in front of the heads' (GQA groups of 1, 2, 4 or 8)
    if (!coop) RA_FAIL(RA_EINVAL, "hand-over area missing");
    int n_helpers = decode_helper_slots(coop, coop_mode, n_seq, n_q, n_kv);
    const int threads = search_threads(heads, ef, expand * deg);
    // One helper per query head instead of one per KV head where the launch leaves compute units idle
    // (few searches): with 512 threads a helper's pass over W for a whole group ends later than a
    // short walk does (128K layer: 17.6 against 19.5 us). The helpers of a group run side by side on
    // one XCD and find each other's rows in its L2.
    int helper_heads = n_q / n_kv;
    if (n_helpers > 0 && threads >= 512 && 2 * heads <= decode_compute_units()) {
        n_helpers *= helper_heads;
        helper_heads = 1;
    }
    const void* Ksearch = kscale ? K8 : K;
    // a start set scored in shares by workgroups of their own: only where every workgroup of the
    // launch has a compute unit to itself (few searches, 512 or 1024 threads each); fewer shares when
    // the part has too few compute units, none below two
    int parts = 0;
    if (seedx && seed_parts > 0 && roots && threads >= 512 && coop_mode != RA_HELPERS_OFF) {
        const int room = (decode_compute_units() - n_helpers) / heads - 1;
        parts = seed_parts < room ? seed_parts : room;
        if (parts > RA_SEED_PARTS_MAX) parts = RA_SEED_PARTS_MAX;
        if (parts < 2) parts = 0;
    }
    const int seed_stride = seed_places(root_cap, deg);
    // Steps shared out (serve_walk): walks with the visited set in device memory, where there are compute units for 8 workers each
    // and steps are wide, which takes a beam of some times `expand` entries to pick from. us per layer without -> with, cells of a
    // step / beam: 4 heads of the mixture law, 1M keys, 3072 / 256 to 1024 105 -> 68, 166 -> 101, 292 -> 171; 2M keys, float32, 3072 / 512
    // 260 -> 113. 4 and 16 heads of the Llama-shaped law, whose steps find a hundred new keys, not a thousand: 4096 / 512 and 1024
    // 71 -> 56, 106 -> 80, 16 heads 72 -> 57, 117 -> 85. Below the lines, before the walk's merges were changed: mixture law 1536 / 512 210 ->
    // 182; the other 2048 / 256 to 1024 53 -> 53, 79 -> 80, 135 -> 130, 16 heads 54 -> 55, 81 -> 78, 139 -> 157; 1024 / 1024 165 -> 203; 4096 / 64
    // 32 -> 47. (With the visited set in LDS the head
    // claims faster than workers could be asked to; scores alone shared out there: mixture law, 128K keys, 3072 / 256 104 -> 84, but
    // Llama-shaped walks +5 to +10 %.) 8 workers are 1 to 3 % slower than 16. Inside the lines, both laws, 2 to 24 heads, 0.8 to
    // 1.5M keys, degree 32 and 64, with and without seed sets, no setting of 200 is slower than alone (1.04 to 1.73 times as fast, 24
    // heads 1.04 to 1.63). The upper line, RA_WALK_CELLS, is the size of an answer's place and the number of heads what 8
    // workers each leave room for: wider steps and fewer workers have not been measured.
    int walk_log2 = 0;
    const int cells = expand * deg;
    if (walk && gb && roots && seed_parts > 0 && coop_mode != RA_HELPERS_OFF && !budgets && threads >= 512 && deg >= 2 &&
        deg * (expand < ef / 4 ? expand : ef / 4) >= RA_WALK_MIN_CELLS && cells <= RA_WALK_CELLS) {
        walk_log2 = 31 - __builtin_clz(walk_parts);
        if (serve_lds_bytes(Ng, deg, expand, walk_log2) > lds) walk_log2 = 0;
        else { parts = 0; ++*walk_launches; }
    }
    if (kscale && !K8) RA_FAIL(RA_EINVAL, "8-bit keys missing");
#define RA_DC_GO_AS(DTV, KTV, GB, TV, BU, WALK, GRID, ...)                                         \
    do {                                                                                           \
        RA_LDS_OPT_IN((decode_kernel<DTV, KTV, GB, TV, BU, WALK>), lds);                           \
        hipLaunchKernelGGL((decode_kernel<DTV, KTV, GB, TV, BU, WALK>),                            \
                           dim3((GRID) + n_helpers), dim3(TV),                                     \
                           lds, st, q, adj, entry, K, V, n_q, n_kv, Ng, N, kv_stride, wstart, deg, \
                           (int)s, topk, ef, expand, bitset, ids, stats, ids_off, scale, out, lse, \
                           coop, n_helpers, coop_mode, coop_spin, roots, root_cap, Ksearch,        \
                           kscale, budgets, seedx, parts, seed_stride, helper_heads, __VA_ARGS__); \
    } while (0)
#define RA_DC_GO_TB(DTV, KTV, GB, TV, BU) RA_DC_GO_AS(DTV, KTV, GB, TV, BU, NoWalk, heads * (1 + parts), NoWalk{})
#define RA_DC_GO_T(DTV, KTV, GB, TV)                                                               \
    do {                                                                                           \
        if (walk_log2)                                                                             \
            RA_DC_GO_AS(DTV, KTV, true, (TV < 512 ? 512 : TV), false, SharedWalk,                  \
                        (heads + 7) / 8 * 8 * (1 + (1 << walk_log2)),                              \
                        SharedWalk{walk, walk_missed, heads, walk_log2});                          \
        else                                                                                       \
            RA_DC_GO_TB(DTV, KTV, GB, TV, false);                                                  \
    } while (0)
#define RA_DC_GO(DTV, KTV, GB)                                                                     \
    do {                                                                                           \
        if (threads == 1024) RA_DC_GO_T(DTV, KTV, GB, 1024);                                       \
        else if (threads == 512) RA_DC_GO_T(DTV, KTV, GB, 512);                                    \
        else RA_DC_GO_T(DTV, KTV, GB, 256);                                                        \
    } while (0)
    if (budgets) {
        // per-head budgets: the walk over the keys as stored, visited bitsets in LDS
        if (kscale || gb)
            RA_FAIL(RA_EUNSUP, "per-head budgets go with neither 8-bit keys nor visited bitsets in device "
                               "memory (context too long for LDS at this ef and expand)");
#define RA_DC_GO_B(DTV)                                                                            \
    do {                                                                                           \
        if (threads == 1024) RA_DC_GO_TB(DTV, DTV, false, 1024, true);                             \
        else if (threads == 512) RA_DC_GO_TB(DTV, DTV, false, 512, true);                          \
        else RA_DC_GO_TB(DTV, DTV, false, 256, true);                                              \
    } while (0)
        if (dt == RA_BF16) RA_DC_GO_B(RA_BF16); else RA_DC_GO_B(RA_F32);
#undef RA_DC_GO_B
    } else if (dt == RA_BF16) {
        if (kscale) { if (gb) RA_DC_GO(RA_BF16, RA_KEYS_I8, true); else RA_DC_GO(RA_BF16, RA_KEYS_I8, false); }
        else if (gb) RA_DC_GO(RA_BF16, RA_BF16, true); else RA_DC_GO(RA_BF16, RA_BF16, false);
    } else {
        if (kscale) { if (gb) RA_DC_GO(RA_F32, RA_KEYS_I8, true); else RA_DC_GO(RA_F32, RA_KEYS_I8, false); }
        else if (gb) RA_DC_GO(RA_F32, RA_F32, true); else RA_DC_GO(RA_F32, RA_F32, false);
    }
#undef RA_DC_GO_T
#undef RA_DC_GO_TB
#undef RA_DC_GO_AS
#undef RA_DC_GO
    RA_HIP(hipGetLastError());
    return RA_OK;
}
