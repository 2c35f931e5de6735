// Stand-alone launch of the graph search (ra_search); the search itself is in search_dev.h.
#include "search_dev.h"

template <int DT, int KT, bool GBITS, int T>
__global__ __launch_bounds__(T, SR_WAVES(KT, T)) void search_kernel(
    const void* __restrict__ q, const int32_t* __restrict__ adj, const int32_t* __restrict__ entry,
    const void* __restrict__ K, int n_q, int n_kv, int64_t N, int deg, int s, int w, int topk,
    int ef, int expand, uint32_t* __restrict__ gbits, int32_t* __restrict__ ids,
    ra_stats* __restrict__ stats, const int32_t* __restrict__ roots, int root_cap,
    const float* __restrict__ kscale) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    run_search<DT, KT, GBITS, T>(lds_raw, xcd_aware_head(blockIdx.x, gridDim.x, n_q / n_kv), q, adj, entry, K, n_q, n_kv, N, N, deg, s, w, topk, topk, ef,
                          expand, gbits, ids, stats, nullptr, roots, root_cap, kscale, NoHook());
    end_touches();
}

// Root sets (see run_search): per head [0] the number of ids, [1] 1 + the number of the entry
// point's neighbours, then the ids: the entry point, its distinct valid neighbours in row order,
// then the distinct valid neighbours of those that are not among the former, in row order.
// One workgroup per head. Which of two equal ids comes first is decided in a hash table in LDS: every
// id leaves the smallest place it occurs at (level 1 before level 2), and only the occurrence at that
// place is kept; prefix sums over the kept ones give the order.
#define RT_THREADS 1024
#define RT_SLOTS 8192             // at most RA_MAX_DEG + 1 + RA_MAX_DEG^2 = 4161 ids
__device__ __forceinline__ uint32_t rt_hash(int id) { return ((uint32_t)id * 2654435761u) >> 19; }
__device__ __forceinline__ int rt_slot(int* ids, int id) {
    uint32_t h = rt_hash(id);
    while (true) {                                       // (the table is never more than half full)
        const int seen = atomicCAS(&ids[h], -1, id);
        if (seen == -1 || seen == id) return (int)h;
        h = (h + 1u) & (RT_SLOTS - 1);
    }
}
__global__ __launch_bounds__(RT_THREADS) void roots_kernel(const int32_t* __restrict__ adj,
                                                           const int32_t* __restrict__ entry, int64_t N,
                                                           int deg, int32_t* __restrict__ roots, int cap) {
    __shared__ int l1[RA_MAX_DEG + 1];
    __shared__ int tab_id[RT_SLOTS], tab_at[RT_SLOTS];
    __shared__ int wsum[RT_THREADS / RA_WAVE];
    __shared__ int n1s;
    const int tid = threadIdx.x, head = blockIdx.x, lane = tid & (RA_WAVE - 1), wv = tid / RA_WAVE;
    const int32_t* adj_h = adj + (size_t)head * N * deg;
    int32_t* out = roots + (size_t)head * cap;
    const int e0 = entry[head];
    for (int x = tid; x < RT_SLOTS; x += RT_THREADS) { tab_id[x] = -1; tab_at[x] = 0x7fffffff; }
    __syncthreads();
    // level 1 (one wavefront: deg <= 64): the entry point at place 0, cell j of its row at place 1 + j
    if (wv == 0) {
        const int nb = lane < deg ? adj_h[(size_t)e0 * deg + lane] : -1;
        const bool ok = nb >= 0 && nb < N && nb != e0;
        int slot = 0;
        if (lane == 0) tab_at[rt_slot(tab_id, e0)] = 0;
        if (ok) {
            slot = rt_slot(tab_id, nb);
            atomicMin(&tab_at[slot], 1 + lane);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const bool first = ok && tab_at[slot] == 1 + lane;
        const unsigned long long m = __ballot(first);
        if (first) l1[1 + __popcll(m & ((1ull << lane) - 1ull))] = nb;
        if (lane == 0) { l1[0] = e0; n1s = 1 + __popcll(m); }
    }
    __syncthreads();
    const int n1 = n1s, cells = (n1 - 1) * deg;
    for (int x = tid; x < n1; x += RT_THREADS) out[2 + x] = l1[x];
    // level 2: cell x at place 1 + deg + x
    constexpr int PER = (RA_MAX_DEG * RA_MAX_DEG + RT_THREADS - 1) / RT_THREADS;
    int nb[PER], slot[PER];
#pragma unroll
    for (int r = 0; r < PER; ++r) {
        const int x = r * RT_THREADS + tid;
        nb[r] = x < cells ? adj_h[(size_t)l1[1 + x / deg] * deg + x % deg] : -1;
    }
#pragma unroll
    for (int r = 0; r < PER; ++r) {
        if (nb[r] >= N) nb[r] = -1;
        slot[r] = 0;
        if (nb[r] >= 0) {
            slot[r] = rt_slot(tab_id, nb[r]);
            atomicMin(&tab_at[slot[r]], 1 + deg + r * RT_THREADS + tid);
        }
    }
    __syncthreads();
    int n = n1;
#pragma unroll
    for (int r = 0; r < PER; ++r) {
        if (r * RT_THREADS >= cells) break;              // uniform
        const bool keep = nb[r] >= 0 && tab_at[slot[r]] == 1 + deg + r * RT_THREADS + tid;
        const unsigned long long m = __ballot(keep);
        if (lane == 0) wsum[wv] = __popcll(m);
        __syncthreads();
        int before = n, all = 0;
        for (int y = 0; y < RT_THREADS / RA_WAVE; ++y) {
            if (y < wv) before += wsum[y];
            all += wsum[y];
        }
        if (keep) out[2 + before + __popcll(m & ((1ull << lane) - 1ull))] = nb[r];
        n += all;
        __syncthreads();
    }
    if (tid == 0) {
        out[0] = n;
        out[1] = n1;
    }
}

ra_status ra_launch_roots(const int32_t* adj, const int32_t* entry, int heads, int64_t N, int deg,
                          int32_t* roots, int cap, hipStream_t st) {
    if (deg > RA_MAX_DEG || cap < 3 + deg + deg * deg) RA_FAIL(RA_EINVAL, "root set buffer too small");
    hipLaunchKernelGGL(roots_kernel, dim3(heads), dim3(RT_THREADS), 0, st, adj, entry, N, deg, roots, cap);
    RA_HIP(hipGetLastError());
    return RA_OK;
}

// Seed sets: the first n_seeds positions, breadth first, of the binary tree that slots 0 and 1 of
// every adjacency row span from the entry point (position p has its children at 2p + 1 and 2p + 2;
// for a projected graph this is the head of the popularity order). Positions without a node and
// nodes already listed at an earlier position are dropped, the order kept. Layout of a root set
// with [1] = 0: no id enters the beam as expanded. Behind the ids their masks (seed_masks_kernel). One workgroup per head; a set-up
// step.
#define SD_THREADS 1024
__global__ __launch_bounds__(SD_THREADS) void seeds_kernel(const int32_t* __restrict__ adj,
                                                           const int32_t* __restrict__ entry, int64_t N,
                                                           int deg, int n_seeds, int32_t* __restrict__ seeds,
                                                           int cap) {
    __shared__ int pos[RA_MAX_SEEDS];
    __shared__ int keep[RA_MAX_SEEDS];
    __shared__ int tab_id[RT_SLOTS], tab_at[RT_SLOTS];
    __shared__ int wsum[SD_THREADS / RA_WAVE];
    const int tid = threadIdx.x, head = blockIdx.x;
    const int32_t* adj_h = adj + (size_t)head * N * deg;
    int32_t* out = seeds + (size_t)head * cap;
    for (int x = tid; x < RT_SLOTS; x += SD_THREADS) { tab_id[x] = -1; tab_at[x] = 0x7fffffff; }
    for (int p = tid; p < n_seeds; p += SD_THREADS) {
        // the path from the root to position p: the bits of p + 1 below its leading one, high to low
        int cur = entry[head];
        const unsigned path = (unsigned)p + 1u;
        for (int b = 30 - __clz(path); b >= 0 && cur >= 0; --b) {
            const int slot = (path >> b) & 1u;
            cur = slot < deg ? adj_h[(size_t)cur * deg + slot] : -1;
            if (cur < 0 || cur >= N) cur = -1;
        }
        pos[p] = cur;
    }
    __syncthreads();
    // of equal nodes the one at the lowest position stays
    for (int p = tid; p < n_seeds; p += SD_THREADS) {
        const int id = pos[p];
        if (id < 0) continue;
        const int slot = rt_slot(tab_id, id);
        keep[p] = slot;
        atomicMin(&tab_at[slot], p);
    }
    __syncthreads();
    for (int p = tid; p < n_seeds; p += SD_THREADS) keep[p] = pos[p] >= 0 && tab_at[keep[p]] == p;
    __syncthreads();
    // ordered compaction: RA_MAX_SEEDS <= 2 * SD_THREADS, two rounds of a workgroup-wide prefix sum
    int base = 0;
    for (int p0 = 0; p0 < n_seeds; p0 += SD_THREADS) {
        const int p = p0 + tid;
        const bool k = p < n_seeds && keep[p];
        const unsigned long long m = __ballot(k);
        const int lane = tid & (RA_WAVE - 1), wv = tid / RA_WAVE;
        if (lane == 0) wsum[wv] = __popcll(m);
        __syncthreads();
        int before = base, total = base;
        for (int x = 0; x < SD_THREADS / RA_WAVE; ++x) {
            if (x < wv) before += wsum[x];
            total += wsum[x];
        }
        if (k) out[2 + before + __popcll(m & ((1ull << lane) - 1ull))] = pos[p];
        base = total;
        __syncthreads();
    }
    if (tid == 0) {
        out[0] = base;
        out[1] = 0;
    }
}

// The masks of listed seed sets (seed_mask_words): the set's ids in a table again, a wavefront per row, four rows on their way. A head's
// rows are dealt to gridDim.y workgroups, since one waits for its trips to memory: the call that sets up 32 heads of 2048 seeds of degree 32 takes
// 32 us, 76 with the masks made by the listing's workgroup, and 20 without masks; 512 heads 119, 130 and 36.
__global__ __launch_bounds__(SD_THREADS) void seed_masks_kernel(const int32_t* __restrict__ adj, int64_t N, int deg,
                                                                int32_t* __restrict__ seeds, int cap) {
    __shared__ int tab_id[RT_SLOTS];
    __shared__ int ids[RA_MAX_SEEDS];
    const int tid = threadIdx.x, lane = tid & (RA_WAVE - 1), wv = tid / RA_WAVE, head = blockIdx.x;
    const int32_t* adj_h = adj + (size_t)head * N * deg;
    int32_t* set = seeds + (size_t)head * cap;
    const int n = set[0];
    for (int x = tid; x < RT_SLOTS; x += SD_THREADS) tab_id[x] = -1;
    __syncthreads();
    for (int c = tid; c < n; c += SD_THREADS) {
        ids[c] = set[2 + c];
        (void)rt_slot(tab_id, ids[c]);
    }
    __syncthreads();
    int32_t* masks = set + 2 + seed_places(cap, deg);
    constexpr int ROWS = 4;
    const int W = (int)gridDim.y * (SD_THREADS / RA_WAVE);       // wavefronts of the head
    for (int c0 = (int)blockIdx.y * (SD_THREADS / RA_WAVE) + wv; c0 < n; c0 += W * ROWS) {
        int nb[ROWS];
#pragma unroll
        for (int u = 0; u < ROWS; ++u) nb[u] = lane < deg ? adj_h[(size_t)ids[min(c0 + u * W, n - 1)] * deg + lane] : -1;
#pragma unroll
        for (int u = 0; u < ROWS; ++u) {
            bool fresh = nb[u] >= 0 && nb[u] < N;
            for (uint32_t h = rt_hash(nb[u]); fresh && tab_id[h] != -1; h = (h + 1u) & (RT_SLOTS - 1)) fresh = tab_id[h] != nb[u];
            const unsigned long long m = __ballot(fresh);
            const int c = c0 + u * W;
            if (c < n) {
                if (deg <= 32) { if (lane == 0) masks[c] = (int)(uint32_t)m; }
                else if (lane < 2) masks[2 * c + lane] = (int)(uint32_t)(m >> (32 * lane));
            }
        }
    }
}

int ra_seed_row_words(int n_seeds, int deg) { return seed_row_words(n_seeds, deg); }

ra_status ra_launch_seeds(const int32_t* adj, const int32_t* entry, int heads, int64_t N, int deg,
                          int n_seeds, int32_t* seeds, int cap, hipStream_t st) {
    if (n_seeds < 1 || n_seeds > RA_MAX_SEEDS || seed_places(cap, deg) < n_seeds) RA_FAIL(RA_EINVAL, "seed set buffer too small");
    hipLaunchKernelGGL(seeds_kernel, dim3(heads), dim3(SD_THREADS), 0, st, adj, entry, N, deg, n_seeds, seeds, cap);
    RA_HIP(hipGetLastError());
    // (workgroups that fill the part, up to eight for a head)
    const int parts = heads >= 512 ? 1 : heads <= 64 ? 8 : 512 / heads;
    hipLaunchKernelGGL(seed_masks_kernel, dim3(heads, parts), dim3(SD_THREADS), 0, st, adj, N, deg, seeds, cap);
    RA_HIP(hipGetLastError());
    return RA_OK;
}

size_t ra_search_lds_bytes(int64_t N, int deg, int ef, int expand, bool global_bitset) {
    return search_lds_bytes(N, deg, ef, expand, global_bitset);
}

bool ra_search_needs_global_bitset(int64_t N, int deg, int ef, int expand) {
    return (size_t)((N + 31) >> 5) * 4 > SR_BITSET_LDS_MAX ||
           ra_search_lds_bytes(N, deg, ef, expand, false) > SR_LDS_LIMIT;
}

ra_status ra_launch_search(const void* q, const int32_t* adj, const int32_t* entry, const void* K,
                           ra_dtype dt, int n_seq, int n_q, int n_kv, int64_t N, int deg,
                           int sink, int window, int topk, int ef, int expand, uint32_t* bitset,
                           const int32_t* roots, int root_cap, const float* kscale, hipStream_t st,
                           int32_t* ids, ra_stats* stats) {
    int64_t ss = sink < 0 ? 0 : sink, ww = window < 0 ? 0 : window;
    if (ss > N) ss = N;
    if (ww > N) ww = N;
    if (ss + ww >= N) { ss = N; ww = 0; }
    const bool gb = ra_search_needs_global_bitset(N, deg, ef, expand);
    const size_t lds = ra_search_lds_bytes(N, deg, ef, expand, gb);
    if (lds > SR_LDS_LIMIT)
        RA_FAIL(RA_EUNSUP, "search state needs %zu B of LDS (limit %d): lower ef or expand", lds,
                SR_LDS_LIMIT);
    const int heads = n_seq * n_q;
    if (gb && !bitset) RA_FAIL(RA_EINVAL, "global visited bitset missing");
    const int threads = search_threads(heads, ef, expand * deg);
#define RA_SR_LAUNCH_T(DTV, KTV, GB, TV)                                                          \
    do {                                                                                          \
        RA_LDS_OPT_IN((search_kernel<DTV, KTV, GB, TV>), lds);                                    \
        hipLaunchKernelGGL((search_kernel<DTV, KTV, GB, TV>), dim3(heads), dim3(TV), lds, st, q,  \
                           adj, entry, K, n_q, n_kv, N, deg, (int)ss, (int)ww, topk, ef, expand,  \
                           bitset, ids, stats, roots, root_cap, kscale);                          \
    } while (0)
#define RA_SR_LAUNCH(DTV, KTV, GB)                                                                \
    do {                                                                                          \
        if (threads == 1024) RA_SR_LAUNCH_T(DTV, KTV, GB, 1024);                                  \
        else if (threads == 512) RA_SR_LAUNCH_T(DTV, KTV, GB, 512);                               \
        else RA_SR_LAUNCH_T(DTV, KTV, GB, 256);                                                   \
    } while (0)
    // K holds 8-bit keys when kscale is given (the query keeps its own type dt)
    if (dt == RA_BF16) {
        if (kscale) { if (gb) RA_SR_LAUNCH(RA_BF16, RA_KEYS_I8, true); else RA_SR_LAUNCH(RA_BF16, RA_KEYS_I8, false); }
        else if (gb) RA_SR_LAUNCH(RA_BF16, RA_BF16, true); else RA_SR_LAUNCH(RA_BF16, RA_BF16, false);
    } else {
        if (kscale) { if (gb) RA_SR_LAUNCH(RA_F32, RA_KEYS_I8, true); else RA_SR_LAUNCH(RA_F32, RA_KEYS_I8, false); }
        else if (gb) RA_SR_LAUNCH(RA_F32, RA_F32, true); else RA_SR_LAUNCH(RA_F32, RA_F32, false);
    }
#undef RA_SR_LAUNCH_T
#undef RA_SR_LAUNCH
    RA_HIP(hipGetLastError());
    return RA_OK;
}
