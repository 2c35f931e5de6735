// Projection of the query->key KNN lists into a key-key graph (Sec. 3.2: keys connected to
// the same query vectors are linked and the query vectors are dropped). Integer arithmetic
// only, so identical lists give bit-identical graphs.
//
// Reading implemented (the paper states the step in one sentence):
//   pop(i)  = number of lists holding key i;   c(a,b) = number of lists holding both;
//   pi      = keys by (pop descending, id ascending); entry = pi[0];
//   row(a)  = [pi[2t+1], pi[2t+2]] for a = pi[t] (a binary heap over popularity: every key is
//             reachable from the entry) followed by a's co-listed keys ranked by the Jaccard
//             overlap c / (pop(a) + pop(b) - c), ties by larger c, then lower id, until deg.
//
// Device plan, all stream-ordered, no host round trip:
//   1. pop by atomic histogram over the list cells, through a per-workgroup LDS table so that a
//      hub costs one atomic per workgroup instead of one per list.
//   2. pi: the populated keys are compacted in id order (a count per block of keys, then every block
//      adds up the counts before its own), their [M - pop : id] keys sorted (bitonic, the network of
//      knn_order.hip: as many stages as the number of populated keys needs, which only the device
//      knows), and pi, its inverse pos and the popularity by position written from that. Keys without
//      a list follow in id order.
//   3. inverted lists (key -> the lists that hold it) filled through per-key cursors (ranges
//      reserved per workgroup through the same kind of LDS table), and a copy of the lists with
//      every key replaced by its position in pi, in 16 bits in graphs of at most 8192 populated keys. In such a graph up to
//      128 hubs (keys in more than a 64th of the lists) have a bitmap over the lists instead, and how many lists hold
//      two of them both is counted by and + popcount.
//   4. backbone children and -1 padding for every row.
//   5. rows of the populated keys. For key a: stream the lists that hold a (whole rows of the
//      translated lists, coalesced), count each co-listed key, and select the best 64. Positions
//      stand for ids throughout: among keys of equal overlap and count (which are equally popular)
//      the lower position is the lower id. By the numbers of populated keys and of the key's list cells (lists x knn):
//        - keys of up to 256 lists in a graph of at most 1024 populated keys, and of those the ones with more than 2048 cells
//          in one of at most 4096: one key per wavefront, counts in LDS by position (pj_rows_wave_kernel);
//        - few cells (up to 2048): one key per wavefront, counts in an LDS hash table sized by
//          the key's class, no workgroup barrier (pj_rows_small_kernel);
//        - the rest, in a graph of at most 8192 populated keys: one key per workgroup, counts in an LDS table indexed by
//          position (pj_rows_kernel);
//        - the rest in a larger graph: one key per workgroup, counts in an LDS hash table, in a few
//          passes over the lists where they hold more keys than the table (pj_rows_hash_kernel), and
//          for the keys with most lists in counters in device memory, the low positions still in LDS
//          (pj_rows_hub_kernel);
//        - hubs: from the pairs' counts and from what the other keys counted (c(a, b) = c(b, a)), last (pj_rows_hubs_kernel).
//      A hub's own walk would be most of the work: of the 4.2 M cells of a Llama-shaped graph of 128K lists nine in ten are 128
//      keys' (32 such graphs, whole projection: 5.3 -> 2.5 ms; 64 of 5003 lists: 0.54 -> 0.30).
// No global sort of the M*knn*(knn-1) co-occurrence pairs is needed.
#include <type_traits>

#include "common.h"

#define PJ_ROW_T 256              // threads of the row kernel
#define PJ_LDS_TAB 8192           // words of the workgroup row kernel's table
#define PJ_BLOCK 2048             // keys a workgroup of the compaction kernels owns
#define PJ_CELL_T 256
#define PJ_TOUCH_A 256            // list cells of a key in each class of the wavefront kernel
#define PJ_TOUCH_B 1024
#define PJ_TOUCH_C 2048
#define PJ_HUBS 128               // most keys of a graph whose lists are kept as a bitmap
#define PJ_FEW_HUBS 48            // ... and fewest
#define PJ_SLAB_WORDS 64          // 32-list words of the bitmaps that a workgroup of the pair kernel takes, at least
#define PJ_MOST_SLABS 16
#define PJ_PAIR_T 192             // threads of the pair kernel
#define PJ_HASH_T 512             // threads of the hash kernel
#define PJ_HASH_TAB 16384         // words of its table
#define PJ_HASH_FILL 10240        // list cells one of its passes puts in there
#define PJ_HASH_PASSES 4          // most passes; a key with more cells than they take is the hub kernel's
#define PJ_WAVE_TAB 4096          // words of a wavefront's table in pj_rows_wave_kernel, and the smaller size of it
#define PJ_WAVE_SMALL_TAB 1024
#define PJ_WAVE_LISTS 256         // most lists of a key there: it walks 64 at a time (with 2048: 32 graphs of 4283 lists of 48 1.25 ms instead of
                                  // 1.12, of 128K lists of 32 2.29 instead of 2.24)

// first positions that pj_pi_kernel leaves: a key's lists x knn at most PJ_TOUCH_A, _B, _C, its lists at most what the hash
// kernel takes, at most PJ_WAVE_LISTS
enum { PJ_CLASS_A, PJ_CLASS_B, PJ_CLASS_C, PJ_CLASS_HASH, PJ_CLASS_WAVE, PJ_CLASSES };

typedef unsigned long long u64;

struct ProjWs {                   // per-graph device arrays, carved from one workspace
    int32_t* pop;                 // [N]
    int32_t* cur;                 // [N]   fill cursors
    int32_t* off;                 // [N]   start of each key's inverted list
    int32_t* pos;                 // [N]   position of key in pi
    int32_t* pi;                  // [N]
    int32_t* inv;                 // [M*knn]
    int32_t* lp;                  // [M*knn] the lists with every key replaced by its position in pi (-1: none);
                                  // [M][row16(knn)] of 16 bits (0xffff: none) in graphs of at most PJ_LDS_TAB populated keys
    uint32_t* bits;               // [words][PJ_HUBS] which of 32 lists hold a hub
    uint32_t* pairs;              // [slabs][PJ_HUBS][PJ_HUBS] lists that hold two hubs
    uint32_t* with_hubs;          // [position - hubs][PJ_HUBS] counts of the other keys with the hubs
    u64* keys;                    // [cap padded to a power of two] sort keys of the populated keys
    int32_t* ppop;                // [cap] popularity by position
    int32_t* blk;                 // [blocks] populated keys per block, then [blocks] list cells per block
    int32_t* H;                   // [0] number of populated keys, [1] number of keys in over, [2] number of hubs,
                                  // [3 + class] first position of keys with few enough lists (PJ_CLASS_*)
    int32_t* over;                // [cap] positions whose lists overflowed a hash table
};

static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

struct ProjLayout {
    size_t per_graph, o_pop, o_cur, o_off, o_pos, o_pi, o_inv, o_lp, o_bits, o_pairs, o_with_hubs, o_keys, o_ppop, o_blk, o_H, o_over;
    size_t scratch_per_wg, o_scratch;
    int n_hub_wg, n_blk, n_slabs;     // n_slabs 0: no hubs
    int64_t cap, cap_pad, words, with_hubs;       // with_hubs: rows of that array
};
__host__ __device__ constexpr int row16(int knn) { return (knn + 7) & ~7; }      // (16-byte reads)

// n_graphs: graphs projected at one time; hubs false: without memory for the hubs' arrays (every key by the other kernels)
static ProjLayout proj_layout(int n_graphs, int64_t N, int64_t M, int knn, bool hubs) {
    ProjLayout l;
    const int64_t cells = M * knn;
    l.cap = N < cells ? N : cells;
    l.cap_pad = ra_sort_padded(l.cap);
    l.n_blk = (int)((N + PJ_BLOCK - 1) / PJ_BLOCK);
    size_t o = 0;
    l.o_pop = o; o += align256((size_t)N * 4);
    l.o_cur = o; o += align256((size_t)N * 4);
    l.o_off = o; o += align256((size_t)N * 4);
    l.o_pos = o; o += align256((size_t)N * 4);
    l.o_pi = o; o += align256((size_t)N * 4);
    l.o_inv = o; o += align256((size_t)cells * 4);
    const size_t narrow = (size_t)M * row16(knn) * 2;
    l.o_lp = o; o += align256(l.cap > PJ_LDS_TAB && (size_t)cells * 4 > narrow ? (size_t)cells * 4 : narrow);
    const size_t lp_end = o;
    l.words = (M + 31) / 32;
    l.n_slabs = !hubs || cells < 32768 ? 0 : (int)(l.words / PJ_SLAB_WORDS < 1 ? 1 : l.words / PJ_SLAB_WORDS > PJ_MOST_SLABS ? PJ_MOST_SLABS : l.words / PJ_SLAB_WORDS);
    l.with_hubs = !l.n_slabs ? 0 : cells < 1 << 20 ? cells / 256 : PJ_LDS_TAB;
    if (l.with_hubs > l.cap) l.with_hubs = l.cap;
    l.o_keys = o; o += align256((size_t)l.cap_pad * 8);
    // What the hubs take is no more than the inverted lists (half of them for the counts, 16 bytes a list, a slab of pairs per
    // 2048 lists), and lies where there is room: behind the 16-bit lists, which is where a graph of more populated keys, which
    // has no hubs, has the rest of its 32-bit ones, or in what is not read any more by then, the bitmaps on pop, the pairs on
    // cur and the counts on keys (32 graphs of 128K lists of 32: 1.50 GB in all instead of 1.73).
    size_t behind = l.o_lp + align256(narrow);
    auto hubs_on = [&](size_t at, size_t room, size_t bytes) {
        if (bytes <= room) return at;
        at = behind;
        if (at + align256(bytes) <= lp_end) {
            behind += align256(bytes);
        } else {
            at = o;
            o += align256(bytes);
        }
        return at;
    };
    if (l.n_slabs) {
        l.o_bits = hubs_on(l.o_pop, (size_t)N * 4, (size_t)l.words * PJ_HUBS * 4);
        l.o_pairs = hubs_on(l.o_cur, (size_t)N * 4, (size_t)l.n_slabs * PJ_HUBS * PJ_HUBS * 4);
        l.o_with_hubs = hubs_on(l.o_keys, (size_t)l.cap_pad * 8, (size_t)l.with_hubs * PJ_HUBS * 4);
    } else {
        l.o_bits = l.o_pairs = l.o_with_hubs = o;
    }
    l.o_ppop = o; o += align256((size_t)l.cap * 4);
    l.o_blk = o; o += align256((size_t)l.n_blk * 8);
    l.o_H = o; o += 256;
    l.o_over = o; o += l.cap > PJ_LDS_TAB ? align256((size_t)l.cap * 4) : 0;
    l.per_graph = o;
    // counters of the hub kernel's workgroups (graphs of more than PJ_LDS_TAB populated keys), at most
    // 1 GiB of them
    l.scratch_per_wg = l.cap > PJ_LDS_TAB ? align256((size_t)l.cap * 4) : 0;
    l.n_hub_wg = 64;
    while (l.n_hub_wg > 1 && ((size_t)l.n_hub_wg * n_graphs > 512 ||
                              (size_t)l.n_hub_wg * n_graphs * l.scratch_per_wg > ((size_t)1 << 30)))
        l.n_hub_wg >>= 1;
    l.o_scratch = l.per_graph * n_graphs;
    return l;
}
static size_t proj_bytes(const ProjLayout& l, int n_graphs) { return l.o_scratch + (size_t)l.n_hub_wg * n_graphs * l.scratch_per_wg; }

// How many of the graphs are projected at one time, in `most` bytes (one, where there is no room for more). With 1.5 GiB a launch
// still has the graphs of a layer of 128K, and a batch takes as long as in one piece, ra_project of 512 graphs: 32768 keys,
// 4096 lists of 32 in 1.4 instead of 7.9 GB 5.13 -> 5.12 ms; 20000 keys, 8192 lists of 64 in 1.4 instead of 8.3 GB 10.2 -> 9.9 ms. (The
// driver's own time for pieces of 4 GB and more is anything from half a millisecond to half a second.)
#define PJ_MOST_BYTES ((size_t)3 << 29)
static int proj_graphs_at_once(int n_graphs, int64_t N, int64_t M, int knn, bool hubs, size_t most) {
    const size_t all = proj_layout(1, N, M, knn, hubs).per_graph * n_graphs;
    int64_t calls = all <= most ? 1 : (int64_t)((all - 1) / most) + 1;
    if (calls > n_graphs) calls = n_graphs;
    while (true) {
        const int64_t g = (n_graphs + calls - 1) / calls;
        if (g == 1 || proj_bytes(proj_layout((int)g, N, M, knn, hubs), (int)g) <= most) return (int)g;
        calls = (n_graphs + g - 2) / (g - 1);            // (as many as make it fewer at a time)
    }
}

// least: what it can do with, one graph at a time and without the hubs' arrays
size_t ra_project_workspace_bytes(int n_graphs, int64_t N, int64_t M, int knn, bool least) {
    const int g = least ? 1 : proj_graphs_at_once(n_graphs, N, M, knn, true, PJ_MOST_BYTES);
    return proj_bytes(proj_layout(g, N, M, knn, !least), g);
}

__device__ __forceinline__ ProjWs carve(char* ws, const ProjLayout& l, int g) {
    char* b = ws + (size_t)g * l.per_graph;
    ProjWs w;
    w.pop = (int32_t*)(b + l.o_pop); w.cur = (int32_t*)(b + l.o_cur); w.off = (int32_t*)(b + l.o_off);
    w.pos = (int32_t*)(b + l.o_pos); w.pi = (int32_t*)(b + l.o_pi);
    w.inv = (int32_t*)(b + l.o_inv); w.lp = (int32_t*)(b + l.o_lp);
    w.bits = (uint32_t*)(b + l.o_bits); w.pairs = (uint32_t*)(b + l.o_pairs);
    w.with_hubs = (uint32_t*)(b + l.o_with_hubs);
    w.keys = (u64*)(b + l.o_keys); w.ppop = (int32_t*)(b + l.o_ppop);
    w.blk = (int32_t*)(b + l.o_blk); w.H = (int32_t*)(b + l.o_H);
    w.over = (int32_t*)(b + l.o_over);
    return w;
}

__device__ __forceinline__ void pj_wave_sync() {         // LDS written by one lane, read by another
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// ---- 0. clear --------------------------------------------------------------------------
__global__ void pj_zero_kernel(char* ws, ProjLayout l, int64_t N) {
    ProjWs w = carve(ws, l, blockIdx.y);
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N;
         i += (int64_t)gridDim.x * blockDim.x) {
        w.pop[i] = 0;
        w.cur[i] = 0;
    }
}

// ---- 1. pop ----------------------------------------------------------------------------
// The queries share their favourite keys (a hub is in nearly every list), so plain atomic adds
// would queue up on a handful of addresses. Each workgroup counts in a small direct-mapped table
// in LDS first (a slot is owned by the first key that claims it; a key looks at PJ_PROBE neighbouring
// slots and goes straight to memory when others own them all) and adds every owned slot to memory once
// at the end. Adds to memory are what the counting costs (they go past the per-XCD L2: about 25 per
// ns), so a launch has no more workgroups than fill the part (128K: 1.30 -> 0.32 ms with a
// quarter of them). Slots are read before they are claimed (after the first few lists they are nearly
// always taken) and four cells per thread are in flight.
#define PJ_HOT 2048
#define PJ_PROBE 4
#define PJ_FLY 4
__device__ __forceinline__ int hot_tag(int* s_tag, int x) {
    return __hip_atomic_load(&s_tag[x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
// the slot of key k, claimed if it has none, -1: none; `first` is what its first slot held (read ahead for several keys at once)
__device__ __forceinline__ int hot_slot(int* s_tag, int k, int first) {
    const int x0 = k & (PJ_HOT - 1);
    if (first == k) return x0;
    for (int u = 0; u < PJ_PROBE; ++u) {
        const int x = (x0 + u) & (PJ_HOT - 1);
        int owner = hot_tag(s_tag, x);
        if (owner == -1) {
            owner = atomicCAS(&s_tag[x], -1, k);
            if (owner == -1) owner = k;
        }
        if (owner == k) return x;
    }
    return -1;
}
// The slots of a thread's keys (k < 0: no key), -1: none. The looks are batched over the keys, without a branch per key:
// each is a trip to LDS.
template <int FLY>
__device__ __forceinline__ void hot_find(int* s_tag, const int32_t (&k)[FLY], int (&x)[FLY]) {
    int tag[FLY];
#pragma unroll
    for (int u = 0; u < FLY; ++u) tag[u] = hot_tag(s_tag, k[u] & (PJ_HOT - 1));
    bool lost = false;
#pragma unroll
    for (int u = 0; u < FLY; ++u) {
        x[u] = k[u] >= 0 && tag[u] == k[u] ? k[u] & (PJ_HOT - 1) : -1;
        lost |= k[u] >= 0 && x[u] < 0;
    }
#pragma unroll
    for (int v = 1; v < PJ_PROBE; ++v) {
        if (__ballot(lost) == 0ull) return;
#pragma unroll
        for (int u = 0; u < FLY; ++u) tag[u] = hot_tag(s_tag, (k[u] + v) & (PJ_HOT - 1));
        lost = false;
#pragma unroll
        for (int u = 0; u < FLY; ++u) {
            if (k[u] >= 0 && x[u] < 0 && tag[u] == k[u]) x[u] = (k[u] + v) & (PJ_HOT - 1);
            lost |= k[u] >= 0 && x[u] < 0;
        }
    }
}
__global__ __launch_bounds__(PJ_CELL_T) void pj_pop_kernel(const int32_t* __restrict__ L, char* ws,
                                                           ProjLayout l, int64_t cells, int64_t N) {
    __shared__ int s_tag[PJ_HOT];
    __shared__ int s_num[PJ_HOT];
    ProjWs w = carve(ws, l, blockIdx.y);
    for (int x = threadIdx.x; x < PJ_HOT; x += PJ_CELL_T) { s_tag[x] = -1; s_num[x] = 0; }
    __syncthreads();
    const int32_t* Lg = L + (size_t)blockIdx.y * cells;
    const int64_t stride = (int64_t)gridDim.x * PJ_CELL_T;
    for (int64_t i0 = (int64_t)blockIdx.x * PJ_CELL_T + threadIdx.x; i0 < cells; i0 += PJ_FLY * stride) {
        int32_t k[PJ_FLY], tag[PJ_FLY];
#pragma unroll
        for (int u = 0; u < PJ_FLY; ++u) {
            const int64_t i = i0 + u * stride;
            k[u] = i < cells ? Lg[i] : -1;
        }
#pragma unroll
        for (int u = 0; u < PJ_FLY; ++u) tag[u] = hot_tag(s_tag, k[u] & (PJ_HOT - 1));
#pragma unroll
        for (int u = 0; u < PJ_FLY; ++u) {
            if (k[u] < 0 || k[u] >= N) continue;
            const int x = hot_slot(s_tag, k[u], tag[u]);
            if (x >= 0) atomicAdd(&s_num[x], 1);
            else atomicAdd(&w.pop[k[u]], 1);
        }
    }
    __syncthreads();
    for (int x = threadIdx.x; x < PJ_HOT; x += PJ_CELL_T)
        if (s_tag[x] >= 0) atomicAdd(&w.pop[s_tag[x]], s_num[x]);
}

// ---- 2. ordering -----------------------------------------------------------------------
// exclusive scan of one int per thread over the workgroup; *total receives the sum
__device__ __forceinline__ int block_exscan(int v, int* wsum, int* total) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
    int inc = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int n = __shfl_up(inc, d);
        if (lane >= d) inc += n;
    }
    if (lane == 63) wsum[wv] = inc;
    __syncthreads();
    int base = 0, tot = 0;
    for (int i = 0; i < nw; ++i) {
        const int s = wsum[i];
        if (i < wv) base += s;
        tot += s;
    }
    __syncthreads();
    *total = tot;
    return base + inc - v;
}

// populated keys and list cells of every block of PJ_BLOCK keys
__global__ __launch_bounds__(256) void pj_count_kernel(char* ws, ProjLayout l, int64_t N) {
    __shared__ int wsum[4];
    ProjWs w = carve(ws, l, blockIdx.y);
    int hot = 0, sum = 0;
    for (int x = threadIdx.x; x < PJ_BLOCK; x += 256) {
        const int64_t i = (int64_t)blockIdx.x * PJ_BLOCK + x;
        const int p = i < N ? w.pop[i] : 0;
        hot += p > 0 ? 1 : 0;
        sum += p;
    }
    int th, ts;
    block_exscan(hot, wsum, &th);
    block_exscan(sum, wsum, &ts);
    if (threadIdx.x == 0) {
        w.blk[blockIdx.x] = th;
        w.blk[l.n_blk + blockIdx.x] = ts;
    }
}

// sort keys of the populated keys (compacted in id order), positions of the others, starts of the
// inverted lists. A thread owns PJ_BLOCK / 256 consecutive keys.
__global__ __launch_bounds__(256) void pj_compact_kernel(char* ws, ProjLayout l, int64_t N, int64_t M) {
    __shared__ int wsum[4];
    ProjWs w = carve(ws, l, blockIdx.y);
    const int tid = threadIdx.x;
    int h_before = 0, h_all = 0, c_before = 0;
    for (int b = tid; b < l.n_blk; b += 256) {
        const int h = w.blk[b];
        h_all += h;
        if (b < (int)blockIdx.x) { h_before += h; c_before += w.blk[l.n_blk + b]; }
    }
    int H, hb, cb;
    block_exscan(h_all, wsum, &H);
    block_exscan(h_before, wsum, &hb);
    block_exscan(c_before, wsum, &cb);
    constexpr int PER = PJ_BLOCK / 256;
    const int64_t i0 = (int64_t)blockIdx.x * PJ_BLOCK + tid * PER;
    int p[PER], hot = 0, sum = 0;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        p[u] = i0 + u < N ? w.pop[i0 + u] : 0;
        hot += p[u] > 0 ? 1 : 0;
        sum += p[u];
    }
    int tot;
    int hr = hb + block_exscan(hot, wsum, &tot);
    int off = cb + block_exscan(sum, wsum, &tot);
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int64_t i = i0 + u;
        if (i >= N) break;
        w.off[i] = off;
        off += p[u];
        if (p[u] > 0) {
            w.keys[hr++] = ((u64)(uint32_t)(M - p[u]) << 32) | (u64)(uint32_t)i;    // ascending = descending pop
        } else {
            const int t = H + (int)i - hr;               // after the populated ones, in id order
            w.pos[i] = t;
            w.pi[t] = (int)i;
        }
    }
    if (blockIdx.x == 0 && tid == 0) {
        w.H[0] = H;
        for (int i = 1; i < 3 + PJ_CLASSES; ++i) w.H[i] = 0;
    }
}

// most lists of a key whose list cells (lists x knn) number at most `touch` (a count must fit the 7
// bits of a small table's entry)
__device__ __forceinline__ int small_limit(int touch, int knn) {
    const int lim = touch / knn;
    return lim < 127 ? lim : 127;
}

// bits of a count, and whether position and count share a word
__device__ __forceinline__ bool hash_fits(int pa, int H, int* cb) {
    int b = 1;
    while ((pa >> b) != 0) ++b;
    *cb = b;
    return ((u64)(H + 1) << b) <= 0xffffffffull;
}
// most lists of a key the hash kernel takes (both conditions can only get easier with fewer lists)
__device__ __forceinline__ int hash_limit(int H, int knn) {
    int lim = PJ_HASH_FILL * PJ_HASH_PASSES / knn, cb;
    while (lim > 0 && !hash_fits(lim, H, &cb)) lim >>= 1;
    return lim;
}
// Hubs: the first positions of a graph of at most PJ_LDS_TAB populated keys, those in more than a 64th of the lists (and
// too many for the wavefront kernels), up to PJ_HUBS of them. Fewer than 48 are not worth it, with the other keys' counts to
// write down for them: 8 graphs of 100000 lists of 32 with 8, 16, 32, 48 and 64 such keys, without -> with the bitmaps 2.94 ->
// 2.96, 2.64 -> 2.64, 2.19 -> 2.21, 1.83 -> 1.63, 1.78 -> 1.63 ms.
// pi, pos and popularity by position of the populated keys; the entry point; the number of hubs
__global__ __launch_bounds__(256) void pj_pi_kernel(char* ws, ProjLayout l, int64_t M, int knn,
                                                    int32_t* __restrict__ entry) {
    ProjWs w = carve(ws, l, blockIdx.y);
    const int H = *w.H;
    int hub_floor = small_limit(PJ_TOUCH_C, knn);
    if (M / 64 > hub_floor) hub_floor = (int)(M / 64);
    const int limit[PJ_CLASSES] = {small_limit(PJ_TOUCH_A, knn), small_limit(PJ_TOUCH_B, knn), small_limit(PJ_TOUCH_C, knn),
                                   hash_limit(H, knn), PJ_WAVE_LISTS};
    for (int t = blockIdx.x * 256 + threadIdx.x; t < H; t += gridDim.x * 256) {
        const u64 k = w.keys[t];
        const int id = (int)(uint32_t)k;
        w.pi[t] = id;
        w.pos[id] = t;
        const int pop = (int)(M - (int64_t)(k >> 32)), next = t + 1 < H ? (int)(M - (int64_t)(w.keys[t + 1] >> 32)) : 0;
        w.ppop[t] = pop;
        if (l.n_slabs && H <= PJ_LDS_TAB && H - (t + 1) <= l.with_hubs && t >= PJ_FEW_HUBS - 1 && t < PJ_HUBS && pop > hub_floor &&
            (t + 1 == PJ_HUBS || next <= hub_floor))
            w.H[2] = t + 1;
#pragma unroll
        for (int i = 0; i < PJ_CLASSES; ++i)
            if (pop > limit[i] && next <= limit[i]) w.H[3 + i] = t + 1;
        if (t == 0) entry[blockIdx.y] = id;
    }
    if (H == 0 && blockIdx.x == 0 && threadIdx.x == 0) entry[blockIdx.y] = 0;
}

// ---- 3. inverted lists -----------------------------------------------------------------
// Same trick for the fill cursors: a workgroup first counts its cells per hot key in LDS, takes
// one range of every such key's inverted list with a single atomic add, and hands out the places
// inside its ranges with LDS atomics in a second pass over the same cells. The order of the
// entries inside an inverted list is immaterial (only co-occurrence counts come out of them).
// Lists are read whole, a run of KP (32 or 64) lanes per list, so that no cell divides by knn; a wavefront
// takes 32 consecutive lists, a word of the hubs' bitmaps, PJ_FLY per run at a time. The lists of a hub are that bitmap: nine
// cells in ten of a Llama-shaped graph are hubs', and their places in inverted lists were most of this kernel's time (scattered
// 4-byte writes; 32 graphs of 128K lists of 32: 1.95 ms, with bitmaps 0.88, with looks and positions read for
// several cells at once, without branches, 0.74; a workgroup barrier per word of the bitmaps or none: the same. What is left is
// the two passes' trips to LDS, a fifth of the time, and their instructions.)
template <int KP>
__global__ __launch_bounds__(PJ_CELL_T) void pj_inv_kernel(const int32_t* __restrict__ L, char* ws,
                                                           ProjLayout l, int64_t M, int knn, int64_t N) {
    __shared__ int s_tag[PJ_HOT];
    __shared__ int s_num[PJ_HOT];
    __shared__ int s_base[PJ_HOT];
    __shared__ uint32_t s_bits[PJ_CELL_T / 64][PJ_HUBS];
    constexpr int FLY = PJ_FLY, RUNS = 64 / KP, PASS = FLY * RUNS;      // PASS: lists a wavefront looks at together
    ProjWs w = carve(ws, l, blockIdx.y);
    const int32_t* Lg = L + (size_t)blockIdx.y * M * knn;
    const int lane = threadIdx.x & 63, e = lane & (KP - 1), r = lane / KP;
    uint32_t* bits = s_bits[threadIdx.x / 64];
    const bool has = e < knn;
    const bool narrow = w.H[0] <= PJ_LDS_TAB;
    const int nh = w.H[2], stride = row16(knn);
    uint16_t* lp16 = reinterpret_cast<uint16_t*>(w.lp);
    for (int x = threadIdx.x; x < PJ_HOT; x += PJ_CELL_T) { s_tag[x] = -1; s_num[x] = 0; }
    bits[lane] = bits[64 + lane] = 0u;
    __syncthreads();
    // (the next lists are on their way: without, every turn is a trip to memory for them)
    const int64_t first = ((int64_t)blockIdx.x * (PJ_CELL_T / 64) + threadIdx.x / 64) * 32;
    const int64_t after = ((int64_t)gridDim.x * (PJ_CELL_T / 64) - 1) * 32;    // from the end of a word to the wavefront's next
    auto load = [&](int64_t j0, int32_t (&k)[FLY]) {
#pragma unroll
        for (int u = 0; u < FLY; ++u) {
            const int64_t j = j0 + u * RUNS + r;
            k[u] = Lg[(j < M ? j : M - 1) * knn + (has ? e : 0)];
        }
    };
    auto lists = [&](auto f) {
        int32_t k1[FLY];
        load(first, k1);
        for (int64_t j0 = first; j0 < l.words * 32;) {
            int32_t k[FLY];
#pragma unroll
            for (int u = 0; u < FLY; ++u) k[u] = !has || j0 + u * RUNS + r >= M || k1[u] >= N ? -1 : k1[u];
            const int64_t next = j0 + PASS + ((j0 + PASS) % 32 == 0 ? after : 0);
            load(next, k1);
            f(j0, k);
            j0 = next;
        }
    };
    lists([&](int64_t, const int32_t (&k)[FLY]) {
        int tag[FLY];
#pragma unroll
        for (int u = 0; u < FLY; ++u) tag[u] = hot_tag(s_tag, k[u] & (PJ_HOT - 1));
#pragma unroll
        for (int u = 0; u < FLY; ++u) {
            if (k[u] < 0) continue;
            const int x = hot_slot(s_tag, k[u], tag[u]);
            if (x >= 0) atomicAdd(&s_num[x], 1);
        }
    });
    __syncthreads();
    for (int x = threadIdx.x; x < PJ_HOT; x += PJ_CELL_T) {
        const int k = s_tag[x];
        if (k >= 0) {
            const int p = nh ? w.pos[k] : 0;
            s_base[x] = p < nh ? ~p : w.off[k] + atomicAdd(&w.cur[k], s_num[x]);
        }
        s_num[x] = 0;                                  // now the cursor inside the range
    }
    __syncthreads();
    lists([&](int64_t j0, const int32_t (&k)[FLY]) {
        int p[FLY], at[FLY], slot[FLY];
        hot_find(s_tag, k, slot);                        // (final by now: owners sit where they claimed)
#pragma unroll
        for (int u = 0; u < FLY; ++u) at[u] = s_base[slot[u] >= 0 ? slot[u] : 0];
#pragma unroll
        for (int u = 0; u < FLY; ++u) {
            const bool hub = slot[u] >= 0 && at[u] < 0;
            p[u] = w.pos[hub || k[u] < 0 ? 0 : k[u]];    // (no branch: all in flight)
        }
#pragma unroll
        for (int u = 0; u < FLY; ++u) {
            if (slot[u] >= 0 && at[u] < 0) p[u] = ~at[u];
            if (k[u] < 0) p[u] = -1;
        }
#pragma unroll
        for (int u = 0; u < FLY; ++u) {
            const int64_t j = j0 + u * RUNS + r;
            if (k[u] >= 0) {
                if (p[u] < nh) atomicOr(&bits[p[u]], 1u << ((int)j & 31));
                else w.inv[slot[u] >= 0 ? at[u] + atomicAdd(&s_num[slot[u]], 1) : w.off[k[u]] + atomicAdd(&w.cur[k[u]], 1)] = (int32_t)j;
            }
            if (narrow) {
                if (e < stride && j < M) lp16[j * stride + e] = (uint16_t)p[u];
            } else if (has && j < M) {
                w.lp[j * knn + e] = p[u];
            }
        }
        if (nh && (j0 + PASS) % 32 == 0) {               // (uniform) the word is whole
            pj_wave_sync();
            uint32_t* word = w.bits + j0 / 32 * PJ_HUBS;
            word[lane] = bits[lane];
            word[64 + lane] = bits[64 + lane];
            bits[lane] = bits[64 + lane] = 0u;
            pj_wave_sync();
        }
    });
}

// How many lists hold both of two hubs: and + popcount over their bitmaps, 8 x 8 pairs per thread, a slab of the
// words per workgroup. Two instructions per 32 lists and pair, which is what bounds it: 32 graphs x 128K lists 0.16 ms, 64 x 5003
// lists 29 us (59 with one slab per graph).
// grid: x = slab, y = graph
__global__ __launch_bounds__(PJ_PAIR_T) void pj_pairs_kernel(char* ws, ProjLayout l) {
    constexpr int CH = 32;                               // words in LDS at a time
    __shared__ __align__(16) uint32_t s_bits[CH][PJ_HUBS];
    ProjWs w = carve(ws, l, blockIdx.y);
    const int nh = w.H[2];
    if (nh == 0) return;
    // tile (ti, tj), ti <= tj, of the 16 x 16: thread (r, c) of 8 x 17 takes row r from the diagonal on, then row 15 - r
    const int tid = threadIdx.x, tr = tid / 17, tc = tid % 17;
    const int ti = tc < 16 - tr ? tr : 15 - tr, tj = tc < 16 - tr ? tr + tc : tc - 1;
    const int64_t begin = l.words * blockIdx.x / l.n_slabs, end = l.words * (blockIdx.x + 1) / l.n_slabs;
    const bool mine = tid < 136 && 8 * tj < nh;
    uint32_t acc[8][8] = {};
    for (int64_t w0 = begin; w0 < end; w0 += CH) {
        const int n = (int)(end - w0 < CH ? end - w0 : CH);
        const uint4* src = reinterpret_cast<const uint4*>(w.bits + w0 * PJ_HUBS);
        __syncthreads();
        for (int x = tid; x < n * (PJ_HUBS / 4); x += PJ_PAIR_T) reinterpret_cast<uint4*>(&s_bits[0][0])[x] = src[x];
        __syncthreads();
        if (!mine) continue;
        for (int i = 0; i < n; ++i) {
            uint32_t a[8], b[8];
            *reinterpret_cast<uint4*>(a) = *reinterpret_cast<const uint4*>(&s_bits[i][8 * ti]);
            *reinterpret_cast<uint4*>(a + 4) = *reinterpret_cast<const uint4*>(&s_bits[i][8 * ti + 4]);
            *reinterpret_cast<uint4*>(b) = *reinterpret_cast<const uint4*>(&s_bits[i][8 * tj]);
            *reinterpret_cast<uint4*>(b + 4) = *reinterpret_cast<const uint4*>(&s_bits[i][8 * tj + 4]);
#pragma unroll
            for (int x = 0; x < 8; ++x)
#pragma unroll
                for (int y = 0; y < 8; ++y) acc[x][y] += __popc(a[x] & b[y]);
        }
    }
    if (!mine) return;
    uint32_t* out = w.pairs + (size_t)blockIdx.x * PJ_HUBS * PJ_HUBS;
#pragma unroll
    for (int x = 0; x < 8; ++x)
#pragma unroll
        for (int y = 0; y < 8; ++y) {
            out[(8 * ti + x) * PJ_HUBS + 8 * tj + y] = acc[x][y];
            if (ti < tj) out[(8 * tj + y) * PJ_HUBS + 8 * ti + x] = acc[x][y];
        }
}

// ---- 4. backbone + padding for every row -----------------------------------------------
// V: cells a thread writes at a time (4 where deg allows 16-byte stores)
template <int V>
__global__ __launch_bounds__(256) void pj_backbone_kernel(char* ws, ProjLayout l, int64_t N, int deg,
                                                          int32_t* __restrict__ adj) {
    ProjWs w = carve(ws, l, blockIdx.y);
    const int per = deg / V, rows = 256 / per, slot = (threadIdx.x % per) * V, r = threadIdx.x / per;
    if (r >= rows) return;
    for (int64_t a = (int64_t)blockIdx.x * rows + r; a < N; a += (int64_t)gridDim.x * rows) {
        int32_t v[V];
#pragma unroll
        for (int u = 0; u < V; ++u) v[u] = -1;
        if (slot < 2) {
            const int64_t ch = 2 * (int64_t)w.pos[a] + 1;
#pragma unroll
            for (int u = 0; u < V; ++u)
                if (slot + u < 2 && ch + slot + u < N) v[u] = w.pi[ch + slot + u];
        }
        int32_t* dst = adj + ((size_t)blockIdx.y * N + a) * deg + slot;
        if constexpr (V == 4) *reinterpret_cast<int4*>(dst) = make_int4(v[0], v[1], v[2], v[3]);
        else dst[0] = v[0];
    }
}

// ---- 5. rows of populated keys ---------------------------------------------------------
// A ranked candidate: larger k first, then (WIDE) larger c, then lower position. k holds the Jaccard
// fraction c / d, d = pop(a) + pop(b) - c. Two different fractions with denominators below 2^b differ
// by more than 2^-2b:
//   M <= 2^19: k = [floor(c / d * 2^42) : 43][c : 21]. d < 2^20, so different fractions are four
//     units apart and the rounding of the double division (under 2^-10 of a unit) cannot close the gap;
//     equal fractions round alike, and then the larger c is first.
//   WIDE: k = floor(c / d * 2^62) exactly (d < 2^31), c on its own.
//   PACKED: all of it in k: [floor(c / d * 2^(2b + 1)) : 2b + 2][c][~position], where that is at most 64 bits (d < 2^b: two units
//     apart, and the division's rounding is below 2^-10 of a unit). Comparing and moving it is half the instructions, of which
//     a row of a few hundred candidates is some thousand: with it, and the first 64 not merged into nothing, keys of up to 256
//     cells of 1M x 4 graphs 2.04 -> 1.58 ms, 64 graphs of 350 populated keys 48.6 -> 37.0 us. (The classes of more cells, whose
//     tables leave few wavefronts per compute unit, are as they were: trips to memory.)
// Zero: no candidate (a real one has c >= 1, k > 0).
enum { CAND_NARROW = 0, CAND_WIDE = 1, CAND_PACKED = 2 };
template <int V> struct pj_int { static constexpr int value = V; };      // a compile-time number as an argument
template <int MODE> struct Cand { u64 k; uint32_t pos; };
template <> struct Cand<CAND_WIDE> { u64 k; uint32_t c, pos; };
template <> struct Cand<CAND_PACKED> { u64 k; };
// fields of a packed candidate: whether they fit, for counts of up to c_bits bits
struct CandPack {
    int d_bits, c_bits, pos_bits;
    __device__ __forceinline__ CandPack(int most_pop, int c_bits_, int H)
        : d_bits(33 - __clz(most_pop)), c_bits(c_bits_), pos_bits(32 - __clz(H)) {}      // (d is below twice the largest popularity)
    __device__ __forceinline__ bool fits() const { return d_bits <= 20 && 2 * d_bits + 2 + c_bits + pos_bits <= 64; }
    __device__ __forceinline__ CandPack() : d_bits(0), c_bits(0), pos_bits(0) {}
    __device__ __forceinline__ uint32_t pos_mask() const { return (1u << pos_bits) - 1u; }
};

template <int MODE>
__device__ __forceinline__ Cand<MODE> cand_none() {
    Cand<MODE> x;
    x.k = 0ull;
    if constexpr (MODE != CAND_PACKED) x.pos = 0x7fffffffu;
    if constexpr (MODE == CAND_WIDE) x.c = 0u;
    return x;
}
template <int MODE>
__device__ __forceinline__ Cand<MODE> cand_make(uint32_t c, uint32_t pa, uint32_t pb, uint32_t pos, const CandPack& pack) {
    Cand<MODE> x;
    const uint32_t d = pa + pb - c;
    if constexpr (MODE == CAND_WIDE) {
        const u64 hi = ((u64)c << 31) / d, rem = ((u64)c << 31) % d;
        x.k = (hi << 31) + (rem << 31) / d;
        x.c = c;
    } else if constexpr (MODE == CAND_PACKED) {
        const u64 ratio = (u64)__builtin_amdgcn_ldexp((double)c / (double)d, 2 * pack.d_bits + 1);
        x.k = ratio << (pack.c_bits + pack.pos_bits) | (u64)c << pack.pos_bits | (u64)(pos ^ pack.pos_mask());
    } else {
        x.k = ((u64)((double)c / (double)d * 4398046511104.0) << 21) | (u64)c;
    }
    if constexpr (MODE != CAND_PACKED) x.pos = pos;
    return x;
}
template <int MODE>
__device__ __forceinline__ bool cand_before(const Cand<MODE>& x, const Cand<MODE>& y) {
    if constexpr (MODE == CAND_PACKED) return x.k > y.k;
    else {
        if (x.k != y.k) return x.k > y.k;
        if constexpr (MODE == CAND_WIDE)
            if (x.c != y.c) return x.c > y.c;
        return x.pos < y.pos;
    }
}
// one compare-exchange step of a bitonic network over the 64 lanes: partner lane ^ J; the lane
// keeps the better of the two when keep_best, else the worse
template <int J, int MODE>
__device__ __forceinline__ Cand<MODE> cand_exchange(const Cand<MODE>& v, bool keep_best, int lane) {
    Cand<MODE> o;
    o.k = ((u64)lane_xor32<J>((uint32_t)(v.k >> 32), lane) << 32) | (u64)lane_xor32<J>((uint32_t)v.k, lane);
    if constexpr (MODE != CAND_PACKED) o.pos = lane_xor32<J>(v.pos, lane);
    if constexpr (MODE == CAND_WIDE) o.c = lane_xor32<J>(v.c, lane);
    return (cand_before(o, v) == keep_best) ? o : v;
}
// what lane `from` holds
template <int MODE>
__device__ __forceinline__ Cand<MODE> cand_lane(const Cand<MODE>& v, int from) {
    Cand<MODE> o;
    o.k = __shfl(v.k, from);
    if constexpr (MODE != CAND_PACKED) o.pos = __shfl(v.pos, from);
    if constexpr (MODE == CAND_WIDE) o.c = __shfl(v.c, from);
    return o;
}
// Lanes that keep the better one in the exchange with lane ^ j of runs of k lanes (descending and ascending in turn, the first as
// `desc` says). For packed candidates, whose row's other instructions are few, as a constant of the scalar unit: as comparisons of the
// lane's number, the compiler keeps all 28 of a row's over the loop, in more scalar registers than there are. (In the kernels of
// the other forms, constants, and the test below for the first 64, make the walks over a key's lists 1 to 11 % longer: 2 graphs of 8000 keys
// in 300000 lists of 48 5.20 -> 5.58 ms.)
constexpr u64 cand_keepers(int k, int j, bool desc) {
    u64 m = 0ull;
    for (int l = 0; l < 64; ++l)
        if ((((l & j) == 0) == ((l & k) == 0)) == desc) m |= 1ull << l;
    return m;
}
// 64 candidates, one per lane, into rank order (DESC: lane 0 the best; else lane 63 the best)
template <bool DESC, int MODE>
__device__ __forceinline__ Cand<MODE> cand_sort64(Cand<MODE> v, int lane) {
#define PJ_STEP(K_, J_)                                                                                              \
    if constexpr (MODE == CAND_PACKED)                                                                              \
        v = cand_exchange<J_>(v, __builtin_amdgcn_inverse_ballot_w64(cand_keepers(K_, J_, DESC)), lane);             \
    else                                                                                                            \
        v = cand_exchange<J_>(v, (((lane & J_) == 0) == ((lane & K_) == 0)) == DESC, lane);
    PJ_STEP(2, 1)
    PJ_STEP(4, 2) PJ_STEP(4, 1)
    PJ_STEP(8, 4) PJ_STEP(8, 2) PJ_STEP(8, 1)
    PJ_STEP(16, 8) PJ_STEP(16, 4) PJ_STEP(16, 2) PJ_STEP(16, 1)
    PJ_STEP(32, 16) PJ_STEP(32, 8) PJ_STEP(32, 4) PJ_STEP(32, 2) PJ_STEP(32, 1)
    PJ_STEP(64, 32) PJ_STEP(64, 16) PJ_STEP(64, 8) PJ_STEP(64, 4) PJ_STEP(64, 2) PJ_STEP(64, 1)
#undef PJ_STEP
    return v;
}
// the better 64 of `best` (descending) and of v (ascending), descending
template <int MODE>
__device__ __forceinline__ Cand<MODE> cand_merge64(Cand<MODE> best, const Cand<MODE>& v, int lane) {
    if (cand_before(v, best)) best = v;                // bitonic: the best 64 of the 128
#define PJ_STEP(J_)                                                                                                  \
    best = cand_exchange<J_>(best, MODE == CAND_PACKED ? __builtin_amdgcn_inverse_ballot_w64(cand_keepers(64, J_, true)) \
                                                       : (lane & J_) == 0, lane);
    PJ_STEP(32) PJ_STEP(16) PJ_STEP(8) PJ_STEP(4) PJ_STEP(2) PJ_STEP(1)
#undef PJ_STEP
    return best;
}

// The best 64 of n candidates, merged into `best` (one wavefront; lane l of best: the l-th best).
// get(x, pos, c): position and count of candidate x in [0, n) (count 0: none). Sorting 64 candidates
// costs hundreds of instructions, and of a few hundred candidates most are nowhere near the best 64: up
// to 64 CH of them at a time have their overlap computed in float32 (CH per lane, in registers), a
// bisection over its bits finds a value that at least 64 and hardly more of them reach, and only
// those (a margin of a few units below it covers the float32 division) get the exact key and are
// sorted. `surv` holds 128 ints of LDS.
template <int CH, int MODE, class Get>
__device__ __forceinline__ void select_best(Cand<MODE>& best, int n, uint32_t pa, const int32_t* ppop, int* surv,
                                            int lane, Get get, const CandPack& pack = CandPack()) {
    bool none = __builtin_amdgcn_readfirstlane((int)(best.k != 0ull)) == 0;          // (the first lane holds the best)
    for (int base = 0; base < n; base += 64 * CH) {
        const int m = n - base < 64 * CH ? n - base : 64 * CH;
        uint32_t f[CH];
        int np = 0;
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            f[i] = 0u;
            if (i * 64 < m) {                            // uniform
                const int x = i * 64 + lane;
                uint32_t pos = 0u, c = 0u;
                if (x < m) get(base + x, pos, c);
                const uint32_t pb = (uint32_t)ppop[pos];
                if (c) f[i] = __float_as_uint((float)c * __builtin_amdgcn_rcpf((float)(pa + pb - c)));
            }
        }
#pragma unroll
        for (int i = 0; i < CH; ++i)
            if (i * 64 < m) np += __popcll(__ballot(f[i] != 0u));
        uint32_t floor_ = 1u;
        if (np > 128) {
            uint32_t lo = 1u, hi = 0x3f800100u;          // an overlap is at most 1
            int at_lo = np;
            while (hi - lo > 1u && at_lo > 96) {
                const uint32_t mid = lo + (hi - lo) / 2u;
                int cnt = 0;
#pragma unroll
                for (int i = 0; i < CH; ++i)
                    if (i * 64 < m) cnt += __popcll(__ballot(f[i] >= mid));
                if (cnt >= 64) { lo = mid; at_lo = cnt; } else hi = mid;
            }
            floor_ = lo > 16u ? lo - 16u : 1u;
        }
        int have = 0;
        auto rank = [&](int take) __attribute__((always_inline)) {
            Cand<MODE> v = cand_none<MODE>();
            if (lane < take) {
                uint32_t pos = 0u, c = 0u;
                get(surv[lane], pos, c);
                v = cand_make<MODE>(c, pa, (uint32_t)ppop[pos], pos, pack);
            }
            Cand<MODE> last;
            last.k = ((u64)(uint32_t)__builtin_amdgcn_readlane((int)(best.k >> 32), 63) << 32) |
                     (u64)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)best.k, 63);
            if constexpr (MODE != CAND_PACKED) last.pos = (uint32_t)__builtin_amdgcn_readlane((int)best.pos, 63);
            if constexpr (MODE == CAND_WIDE) last.c = (uint32_t)__builtin_amdgcn_readlane((int)best.c, 63);
            if (__ballot(cand_before(v, last)) == 0ull) return;            // nothing here makes the 64
            v = cand_sort64<false>(v, lane);
            if (MODE == CAND_PACKED && none) {               // (uniform) the first of them: the same, best first
                none = false;
                best = cand_lane(v, 63 - lane);
            } else {
                best = cand_merge64(best, v, lane);
            }
        };
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            if (i * 64 >= m) break;
            const bool in = f[i] >= floor_;
            const u64 mask = __ballot(in);
            if (mask == 0ull) continue;
            if (in) surv[have + __popcll(mask & ((1ull << lane) - 1ull))] = base + i * 64 + lane;
            have += __popcll(mask);
            pj_wave_sync();
            if (have >= 64) {
                rank(64);
                have -= 64;
                const int more = surv[64 + lane];
                pj_wave_sync();
                if (lane < have) surv[lane] = more;
                pj_wave_sync();
            }
        }
        if (have) rank(have);
        pj_wave_sync();
    }
}

// Row of the key at position t: its backbone children pi[2t+1], pi[2t+2], then the ranked
// candidates (lane l of `best` holds the l-th best) that are not among the children, until deg
// entries; -1 beyond. One wavefront.
template <int MODE>
__device__ __forceinline__ void write_row(int32_t* row, const Cand<MODE>& best, int t, const int32_t* pi, int64_t N,
                                          int deg, int lane, const CandPack& pack = CandPack()) {
    const int64_t ch = 2 * (int64_t)t + 1;
    int nk = (int)(N - ch < 0 ? 0 : N - ch < 2 ? N - ch : 2);
    if (nk > deg) nk = deg;
    uint32_t pos;
    if constexpr (MODE == CAND_PACKED) pos = ((uint32_t)best.k & pack.pos_mask()) ^ pack.pos_mask();
    else pos = best.pos;
    const bool keep = best.k != 0ull && lane < deg && ((int64_t)pos < ch || (int64_t)pos >= ch + nk);
    const u64 km = __ballot(keep);
    const int at = nk + __popcll(km & ((1ull << lane) - 1ull));
    const int total = nk + __popcll(km);
    if (lane < nk) row[lane] = pi[ch + lane];
    if (keep && at < deg) row[at] = pi[pos];
    if (lane >= total && lane < deg) row[lane] = -1;
}

// One more co-occurrence of the key at position `key - 1` in an open-addressing table of `slots`
// (a power of two) LDS words, entry = key << cb | count. False when no slot is left.
__device__ __forceinline__ bool lds_table_bump(uint32_t* tab, int slots, uint32_t key, int cb) {
    const uint32_t mask = (uint32_t)slots - 1u;
    uint32_t h = ((key * 2654435761u) >> 12) & mask;
    for (int probe = 0; probe < slots; ++probe) {
        uint32_t v = __hip_atomic_load(&tab[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (v == 0u) {
            v = atomicCAS(&tab[h], 0u, (key << cb) | 1u);
            if (v == 0u) return true;                 // claimed, count 1
        }
        if ((v >> cb) == key) { atomicAdd(&tab[h], 1u); return true; }
        h = (h + 1u) & mask;
    }
    return false;
}

// f(position) for the entries of the lists [begin, end) of a key (inv: its inverted list), U lists in
// flight per run of kp lanes; e: this lane's entry, r0 / rstep: this run's first list and the distance
// to its next
template <int U, class F>
__device__ __forceinline__ void walk_lists(const int32_t* inv, const int32_t* lp, int begin, int end, int knn, int e,
                                           int r0, int rstep, F f) {
    const int ec = e < knn ? e : 0;
    for (int li0 = begin + r0; li0 < end; li0 += U * rstep) {
        int pp[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int li = li0 + u * rstep;
            pp[u] = inv[li < end ? li : end - 1];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) pp[u] = lp[(size_t)pp[u] * knn + ec];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (li0 + u * rstep < end && e < knn && pp[u] >= 0) f(pp[u]);
    }
}

// The same over n lists with rows of 16-bit positions (stride = row16(knn)), by T threads (`at` of them this one): a lane
// takes eight positions of a row, U rows are in flight, and the numbers of the next ones.
template <int U, int T, class F>
__device__ __forceinline__ void walk_narrow(const int32_t* inv, const uint16_t* lp, int n, int stride, int at, F f) {
    const int shift = stride <= 8 ? 0 : stride <= 16 ? 1 : stride <= 32 ? 2 : 3;       // log2 of the lanes of a row
    const int q = 8 * (at & ((1 << shift) - 1)), r = at >> shift, step = T >> shift;
    const bool has = q < stride;
    int j[U];
#pragma unroll
    for (int u = 0; u < U; ++u) j[u] = inv[r + u * step < n ? r + u * step : n - 1];
    for (int i0 = r; i0 < n; i0 += U * step) {
        uint4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = *reinterpret_cast<const uint4*>(lp + (size_t)j[u] * stride + (has ? q : 0));
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int next = i0 + (U + u) * step;
            j[u] = inv[next < n ? next : n - 1];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (!has || i0 + u * step >= n) continue;
            const uint32_t w[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
            for (int x = 0; x < 8; ++x) {
                const int p = (int)((w[x / 2] >> (16 * (x & 1))) & 0xffffu);
                if (p != 0xffff) f(p);
            }
        }
    }
}

#define PJ_SMALL_WAVES 4
#define PJ_HUB_T 1024             // threads of the hub kernel

// Keys with few lists are handled one per wavefront, the others one per workgroup: first position of the former (they
// are pj_rows_small_kernel's; in graphs of at most PJ_WAVE_TAB populated keys pj_rows_wave_kernel's, after the hubs)
__device__ __forceinline__ int large_end(const ProjWs& w, int H) {
    if (H <= PJ_WAVE_TAB) return w.H[2] > w.H[3 + PJ_CLASS_WAVE] ? w.H[2] : w.H[3 + PJ_CLASS_WAVE];
    return H < (1 << 24) ? w.H[3 + PJ_CLASS_C] : H;
}

// the best 64 of a workgroup's wavefronts, and the row of the key at position t
template <int T, int MODE>
__device__ __forceinline__ void finish_row(Cand<MODE> best, Cand<MODE> (*s_best)[64], int32_t* adj_g, int t,
                                           const ProjWs& w, int64_t N, int deg) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    // pairs of wavefronts, then pairs of those
#pragma unroll
    for (int step = 1; step < T / 64; step <<= 1) {
        if ((wv & (2 * step - 1)) == step) s_best[wv][lane] = best;
        __syncthreads();
        if ((wv & (2 * step - 1)) == 0)
            best = cand_merge64(best, s_best[wv + step][63 - lane], lane);          // (descending list, reversed)
    }
    // row = backbone children, then ranked candidates not already present
    if (wv == 0) write_row(adj_g + (size_t)w.pi[t] * deg, best, t, w.pi, N, deg, lane);
    __syncthreads();
}

// Rows of the populated keys but hubs with more list cells than the wavefront kernels take, one per workgroup, of a graph with
// at most PJ_LDS_TAB populated keys. The counters are indexed by position: bumps return nothing and are
// never waited for (a returning add per cell, to notice first touches, was bound by its latency: 7.0
// against 2.9 ms at 128K), and the candidates are the non-zero words.
// grid: x = graph, y = worker of the graph
template <int MODE>
__global__ __launch_bounds__(PJ_ROW_T) void pj_rows_kernel(char* ws, ProjLayout l, int64_t N, int knn, int deg,
                                                           int32_t* __restrict__ adj) {
    constexpr int WV = PJ_ROW_T / 64;
    __shared__ Cand<MODE> s_best[WV][64];
    __shared__ int s_surv[WV][128];
    __shared__ uint32_t tab[PJ_LDS_TAB];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    ProjWs w = carve(ws, l, blockIdx.x);
    int32_t* adj_g = adj + (size_t)blockIdx.x * N * deg;
    const int H = *w.H;
    if (H > PJ_LDS_TAB) return;
    const int t_end = large_end(w, H);
    const int nh = w.H[2];
    if (nh + (int)blockIdx.y >= t_end) return;
    for (int i = tid; i < H; i += PJ_ROW_T) tab[i] = 0u;
    __syncthreads();
    for (int t = nh + blockIdx.y; t < t_end; t += gridDim.y) {
        const int pa = w.ppop[t];
        walk_narrow<4, PJ_ROW_T>(w.inv + w.off[w.pi[t]], reinterpret_cast<const uint16_t*>(w.lp), pa, row16(knn), tid,
                                 [&](int p) { atomicAdd(&tab[p], 1u); });
        __syncthreads();
        if (tid == 0) tab[t] = 0u;                           // the key itself
        __syncthreads();
        if (tid < nh) w.with_hubs[(size_t)(t - nh) * PJ_HUBS + tid] = tab[tid];
        // a wavefront ranks its share of the positions (chunks of 64 dealt in turn)
        Cand<MODE> best = cand_none<MODE>();
        const int chunks = (H + 63) / 64, mine = (chunks - wv + WV - 1) / WV;
        select_best<8>(best, mine * 64, (uint32_t)pa, w.ppop, s_surv[wv], lane,
                       [&](int x, uint32_t& pos, uint32_t& c) {
                           const int p = ((x >> 6) * WV + wv) * 64 + (x & 63);
                           if (p < H) { pos = (uint32_t)p; c = tab[p]; }
                       });
        __syncthreads();
        for (int i = tid; i < H; i += PJ_ROW_T) tab[i] = 0u;
        finish_row<PJ_ROW_T>(best, s_best, adj_g, t, w, N, deg);
    }
}

// The same for graphs with more populated keys: entries are hashed, [position + 1 : count] in one
// word. A key with more cells than the table takes is done in passes over its lists, each counting the
// positions of its own residue. What fits neither way (too many passes, count and position beyond 32
// bits, a crowd in one residue) is left to pj_rows_hub_kernel: its first positions, or the overflow list.
template <int MODE>
__global__ __launch_bounds__(PJ_HASH_T) void pj_rows_hash_kernel(char* ws, ProjLayout l, int64_t N, int knn, int deg,
                                                                 int32_t* __restrict__ adj) {
    constexpr int WV = PJ_HASH_T / 64;
    __shared__ Cand<MODE> s_best[WV][64];
    __shared__ int s_surv[WV][128];
    __shared__ uint32_t tab[PJ_HASH_TAB];
    __shared__ int s_over;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    ProjWs w = carve(ws, l, blockIdx.x);
    int32_t* adj_g = adj + (size_t)blockIdx.x * N * deg;
    const int H = *w.H;
    if (H <= PJ_LDS_TAB) return;
    const int t_begin = w.H[3 + PJ_CLASS_HASH], t_end = large_end(w, H);
    if (t_begin + (int)blockIdx.y >= t_end) return;
    for (int i = tid; i < PJ_HASH_TAB; i += PJ_HASH_T) tab[i] = 0u;
    if (tid == 0) s_over = 0;
    __syncthreads();
    const int kp = knn <= 32 ? 32 : 64;
    const int e = tid & (kp - 1), r0 = tid / kp, rstep = PJ_HASH_T / kp;
    uint32_t* mine = tab + wv * (PJ_HASH_TAB / WV);
    for (int t = t_begin + blockIdx.y; t < t_end; t += gridDim.y) {
        const int pa = w.ppop[t];
        const int32_t* inv = w.inv + w.off[w.pi[t]];
        int cb;
        (void)hash_fits(pa, H, &cb);
        const int passes = (pa * knn + PJ_HASH_FILL - 1) / PJ_HASH_FILL;
        // words the passes spread over: a key with few lists does not clear and scan the whole table
        int slots = 64 * WV;
        while (slots < PJ_HASH_TAB && slots < 2 * pa * knn) slots <<= 1;
        const int quarter = slots / WV;
        uint32_t* part = passes > 1 ? mine : tab + wv * quarter;
        Cand<MODE> best = cand_none<MODE>();
        for (int r = 0; r < passes; ++r) {
            walk_lists<8>(inv, w.lp, 0, pa, knn, e, r0, rstep, [&](int p) {
                // residue classes of a multiplicative hash: neighbouring positions spread out
                if (p == t || (passes > 1 && (int)(((uint32_t)p * 2246822519u >> 16) % (uint32_t)passes) != r)) return;
                if (!lds_table_bump(tab, slots, (uint32_t)p + 1u, cb)) s_over = 1;
            });
            __syncthreads();
            const bool over = s_over != 0;                     // (uniform; set by this pass or one before)
            // every wavefront packs its share of the table in place and ranks it
            int nc = 0;
            for (int q0 = 0; q0 < quarter; q0 += 64) {
                const uint32_t v = part[q0 + lane];
                part[q0 + lane] = 0u;
                const u64 m = __ballot(v != 0u);
                if (v != 0u) part[nc + __popcll(m & ((1ull << lane) - 1ull))] = v;
                nc += __popcll(m);
            }
            pj_wave_sync();
            if (!over)
                select_best<16>(best, nc, (uint32_t)pa, w.ppop, s_surv[wv], lane,
                                [&](int x, uint32_t& pos, uint32_t& c) {
                                    const uint32_t v = part[x];
                                    pos = (v >> cb) - 1u;
                                    c = v & ((1u << cb) - 1u);
                                });
            pj_wave_sync();
            for (int x = lane; x < nc; x += 64) part[x] = 0u;
            __syncthreads();
        }
        if (s_over) {                                          // (uniform)
            __syncthreads();
            if (tid == 0) {
                w.over[atomicAdd(&w.H[1], 1)] = t;
                s_over = 0;
            }
            __syncthreads();
        } else {
            finish_row<PJ_HASH_T>(best, s_best, adj_g, t, w, N, deg);
        }
    }
}

// The keys pj_rows_hash_kernel leaves: counters of positions below PJ_LDS_TAB in LDS, of the others in
// device memory (adds that return nothing), then every counter is looked at.
// grid: x = graph, y = worker
template <int MODE>
__global__ __launch_bounds__(PJ_HUB_T) void pj_rows_hub_kernel(char* ws, ProjLayout l, int64_t N, int knn, int deg,
                                                               int32_t* __restrict__ adj) {
    constexpr int WV = PJ_HUB_T / 64;
    __shared__ Cand<MODE> s_best[WV][64];
    __shared__ int s_surv[WV][128];
    __shared__ uint32_t tab[PJ_LDS_TAB];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    ProjWs w = carve(ws, l, blockIdx.x);
    int32_t* adj_g = adj + (size_t)blockIdx.x * N * deg;
    const int H = *w.H;
    if (H <= PJ_LDS_TAB) return;
    const int t_hub = min(w.H[3 + PJ_CLASS_HASH], large_end(w, H)), n = t_hub + w.H[1];
    if ((int)blockIdx.y >= n) return;
    uint32_t* cnt = (uint32_t*)(ws + l.o_scratch + ((size_t)blockIdx.x * gridDim.y + blockIdx.y) * l.scratch_per_wg);
    for (int i = tid; i < PJ_LDS_TAB; i += PJ_HUB_T) tab[i] = 0u;
    for (int i = tid; i < H; i += PJ_HUB_T)
        __hip_atomic_store(&cnt[i], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    const int kp = knn <= 32 ? 32 : 64;
    const int e = tid & (kp - 1), r0 = tid / kp, rstep = PJ_HUB_T / kp;
    for (int x = blockIdx.y; x < n; x += gridDim.y) {
        const int t = x < t_hub ? x : w.over[x - t_hub];
        const int pa = w.ppop[t];
        walk_lists<8>(w.inv + w.off[w.pi[t]], w.lp, 0, pa, knn, e, r0, rstep, [&](int p) {
            if (p == t) return;
            if (p < PJ_LDS_TAB) atomicAdd(&tab[p], 1u);
            else __hip_atomic_fetch_add(&cnt[p], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        });
        __builtin_amdgcn_s_waitcnt(0);                       // the adds have been made before anyone reads
        __syncthreads();
        Cand<MODE> best = cand_none<MODE>();
        const int chunks = (H + 63) / 64, mine = (chunks - wv + WV - 1) / WV;
        select_best<16>(best, mine * 64, (uint32_t)pa, w.ppop, s_surv[wv], lane,
                        [&](int y, uint32_t& pos, uint32_t& c) {
                            const int p = ((y >> 6) * WV + wv) * 64 + (y & 63);
                            if (p >= H) return;
                            pos = (uint32_t)p;
                            c = p < PJ_LDS_TAB ? tab[p]
                                               : __hip_atomic_load(&cnt[p], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        });
        __syncthreads();
        for (int i = tid; i < PJ_LDS_TAB; i += PJ_HUB_T) tab[i] = 0u;
        for (int i = PJ_LDS_TAB + tid; i < H; i += PJ_HUB_T)
            __hip_atomic_store(&cnt[i], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        finish_row<PJ_HUB_T>(best, s_best, adj_g, t, w, N, deg);
    }
}

// Rows of the keys with few lists, one key per wavefront, no workgroup barrier. Co-occurrence
// counts go into an open-addressing table in LDS (entry = (position + 1) << 7 | count, twice the
// key's list cells at least), which is then packed in place into the candidate list. TOUCH: most
// list cells of a key of this launch's class, more than BELOW: small classes have small tables, and a
// compute unit holds more wavefronts, whose trips to memory (list numbers, lists, popularities) hide
// behind each other.
// grid: x = graph, y = worker
template <int TOUCH, int BELOW, int MODE>
__global__ __launch_bounds__(PJ_SMALL_WAVES * 64) void pj_rows_small_kernel(
    char* ws, ProjLayout l, int64_t N, int knn, int deg, int32_t* __restrict__ adj) {
    constexpr int SLOTS = 2 * TOUCH;
    __shared__ uint32_t s_slot[PJ_SMALL_WAVES][SLOTS];
    __shared__ int s_surv[PJ_SMALL_WAVES][128];
    const int g = blockIdx.x;
    ProjWs w = carve(ws, l, g);
    int32_t* adj_g = adj + (size_t)g * N * deg;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    uint32_t* slot = s_slot[wv];
    const int H = *w.H;
    if (H <= PJ_WAVE_SMALL_TAB) return;                  // pj_rows_wave_kernel's
    if (H >= (1 << 24)) return;                          // a position must fit the other 25 bits: pj_rows_kernel's
    const int nh = w.H[2];
    const int kp = knn <= 32 ? 32 : 64, e = lane & (kp - 1), lpp = 64 / kp;     // lists per pass
    for (int x = lane; x < SLOTS; x += 64) slot[x] = 0u;
    pj_wave_sync();
    const int t0 = w.H[3 + (TOUCH == PJ_TOUCH_A ? PJ_CLASS_A : TOUCH == PJ_TOUCH_B ? PJ_CLASS_B : PJ_CLASS_C)];
    const int t1 = BELOW == 0 ? H : w.H[3 + (BELOW == PJ_TOUCH_A ? PJ_CLASS_A : PJ_CLASS_B)];
    auto rows = [&](auto mode_c, const CandPack& pack) __attribute__((always_inline)) {
        constexpr int M = decltype(mode_c)::value;
        for (int t = t0 + blockIdx.y * PJ_SMALL_WAVES + wv; t < t1; t += gridDim.y * PJ_SMALL_WAVES) {
            const int a = w.pi[t];
            const int pa = w.ppop[t];
            int slots = 128;
            while (slots < 2 * pa * knn) slots <<= 1;        // <= SLOTS by small_limit()
            auto bump = [&](int p) {
                if (p != t) lds_table_bump(slot, slots, (uint32_t)p + 1u, 7);
            };
            if (H <= PJ_LDS_TAB)
                walk_narrow<4, 64>(w.inv + w.off[a], reinterpret_cast<const uint16_t*>(w.lp), pa, row16(knn), lane, bump);
            else
                walk_lists<4>(w.inv + w.off[a], w.lp, 0, pa, knn, e, lane / kp, lpp, bump);
            pj_wave_sync();
            // pack the table in place: entry q moves to the number of entries before it
            int nc = 0;
            for (int q0 = 0; q0 < slots; q0 += 64) {
                const uint32_t v = slot[q0 + lane];
                slot[q0 + lane] = 0u;
                const u64 m = __ballot(v != 0u);
                if (v != 0u) slot[nc + __popcll(m & ((1ull << lane) - 1ull))] = v;
                nc += __popcll(m);
            }
            pj_wave_sync();
            if (nh) {                                            // (uniform)
                int* row = s_surv[wv];
                row[lane] = row[64 + lane] = 0;
                pj_wave_sync();
                for (int x = lane; x < nc; x += 64) {
                    const uint32_t v = slot[x];
                    if ((int)(v >> 7) <= nh) row[(v >> 7) - 1u] = (int)(v & 127u);
                }
                pj_wave_sync();
                for (int x = lane; x < nh; x += 64) w.with_hubs[(size_t)(t - nh) * PJ_HUBS + x] = (uint32_t)row[x];
                pj_wave_sync();
            }
            Cand<M> best = cand_none<M>();
            select_best<(TOUCH + 63) / 64 < 16 ? (TOUCH + 63) / 64 : 16>(
                best, nc, (uint32_t)pa, w.ppop, s_surv[wv], lane, [&](int x, uint32_t& pos, uint32_t& c) {
                    const uint32_t v = slot[x];
                    pos = (v >> 7) - 1u;
                    c = v & 127u;
                }, pack);
            pj_wave_sync();
            for (int x = lane; x < nc; x += 64) slot[x] = 0u;       // the table is empty again
            pj_wave_sync();
            write_row(adj_g + (size_t)a * deg, best, t, w.pi, N, deg, lane, pack);
        }
    };
    if (t0 >= t1) return;
    const CandPack pack(w.ppop[0], 7, H);
    if (pack.fits()) rows(pj_int<CAND_PACKED>{}, pack);
    else rows(pj_int<MODE>{}, pack);
}

// Rows of the keys with at most PJ_WAVE_LISTS lists in a graph of at most PJ_WAVE_TAB populated keys, one per wavefront,
// without a barrier; the counters are indexed by position. (With a workgroup per key, its four wavefronts' rankings
// and their merges were most of a row: 64 graphs of about 350 populated keys 76 us, now 55 with all their smaller keys, which
// the small kernels took another 90 for; 32 graphs of 1000 to 3000, the larger keys but hubs 0.65 -> 0.58 ms.) Above
// PJ_WAVE_SMALL_TAB the smaller keys stay the small kernels': looking through a table of H counters for a key of a few
// lists costs more than a hash table (the same 32 graphs: 0.60 ms here, without them 0.30, and 0.22 there).
// grid: x = graph, y = worker
template <int TAB, int ABOVE, int MODE>
__global__ __launch_bounds__(PJ_SMALL_WAVES * 64) void pj_rows_wave_kernel(char* ws, ProjLayout l, int64_t N, int knn,
                                                                           int deg, int32_t* __restrict__ adj) {
    __shared__ uint32_t s_tab[PJ_SMALL_WAVES][TAB];
    __shared__ int s_surv[PJ_SMALL_WAVES][128];
    ProjWs w = carve(ws, l, blockIdx.x);
    int32_t* adj_g = adj + (size_t)blockIdx.x * N * deg;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    uint32_t* tab = s_tab[wv];
    const int H = *w.H;
    if (H > TAB || H <= ABOVE) return;
    const int nh = w.H[2];
    for (int x = lane; x < H; x += 64) tab[x] = 0u;
    pj_wave_sync();
    const int t_end = TAB == PJ_WAVE_SMALL_TAB ? H : w.H[3 + PJ_CLASS_C];
    auto rows = [&](auto mode_c, const CandPack& pack) __attribute__((always_inline)) {
        constexpr int M = decltype(mode_c)::value;
        for (int t = large_end(w, H) + blockIdx.y * PJ_SMALL_WAVES + wv; t < t_end; t += gridDim.y * PJ_SMALL_WAVES) {
            const int a = w.pi[t];
            const int pa = w.ppop[t];
            walk_narrow<4, 64>(w.inv + w.off[a], reinterpret_cast<const uint16_t*>(w.lp), pa, row16(knn), lane,
                               [&](int p) { atomicAdd(&tab[p], 1u); });
            pj_wave_sync();
            if (lane == 0) tab[t] = 0u;                          // the key itself
            pj_wave_sync();
            for (int x = lane; x < nh; x += 64) w.with_hubs[(size_t)(t - nh) * PJ_HUBS + x] = tab[x];
            // pack the table in place, position and count in a word (a count is at most PJ_WAVE_LISTS x 64)
            static_assert(PJ_WAVE_TAB <= 1 << 12 && PJ_WAVE_LISTS * 64 < 1 << 20, "a position and a count share a word");
            int nc = 0;
            for (int q0 = 0; q0 < H; q0 += 64) {
                const int q = q0 + lane;
                const uint32_t c = q < H ? tab[q] : 0u;
                if (q < H) tab[q] = 0u;
                const u64 m = __ballot(c != 0u);
                if (c != 0u) tab[nc + __popcll(m & ((1ull << lane) - 1ull))] = (uint32_t)q << 20 | c;
                nc += __popcll(m);
            }
            pj_wave_sync();
            Cand<M> best = cand_none<M>();
            select_best<8>(best, nc, (uint32_t)pa, w.ppop, s_surv[wv], lane, [&](int x, uint32_t& pos, uint32_t& c) {
                const uint32_t v = tab[x];
                pos = v >> 20;
                c = v & 0xfffffu;
            }, pack);
            pj_wave_sync();
            for (int x = lane; x < nc; x += 64) tab[x] = 0u;
            pj_wave_sync();
            write_row(adj_g + (size_t)a * deg, best, t, w.pi, N, deg, lane, pack);
        }
    };
    const CandPack pack(w.ppop[0], 15, H);                  // (a count is at most PJ_WAVE_LISTS x 64)
    if (pack.fits()) rows(pj_int<CAND_PACKED>{}, pack);
    else rows(pj_int<MODE>{}, pack);
}

// Rows of the hubs, one per wavefront: their counts with each other are pj_pairs_kernel's, those with the other keys what
// these found on their own walks. 32 graphs of 128K lists 0.08 ms; a walk per hub, over the front of each of its lists' rows
// only, and only where the other hubs did not settle its row, 1.0 ms; over whole rows 1.7.
// grid: x = graph, y = workers
template <int MODE>
__global__ __launch_bounds__(PJ_ROW_T) void pj_rows_hubs_kernel(char* ws, ProjLayout l, int64_t N, int knn, int deg,
                                                                int32_t* __restrict__ adj) {
    constexpr int WV = PJ_ROW_T / 64;
    __shared__ uint32_t s_with[WV][PJ_HUBS];
    __shared__ int s_surv[WV][128];
    __shared__ int s_n, s_twice;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    ProjWs w = carve(ws, l, blockIdx.x);
    const int H = *w.H, nh = w.H[2], t0 = blockIdx.y * WV, t = t0 + wv;
    if (t0 >= nh) return;
    if (tid == 0) s_twice = 0;
    __syncthreads();
    for (int x = lane; x < nh; x += 64) {
        uint32_t c = 0u, own = 0u;
#pragma unroll 4
        for (int i = 0; i < l.n_slabs; ++i) {
            const uint32_t* slab = w.pairs + (size_t)i * PJ_HUBS * PJ_HUBS;
            c += slab[(t < nh ? t : t0) * PJ_HUBS + x];
            own += slab[x * PJ_HUBS + x];
        }
        s_with[wv][x] = c;
        if ((int)own != w.ppop[x]) s_twice = 1;
    }
    __syncthreads();
    if (s_twice) {
        // A list holds a hub more than once, and every pair of places counts: the lists of this workgroup's hubs are
        // looked at one by one, their numbers written to where the hub's inverted list would be.
        const uint16_t* lp = reinterpret_cast<const uint16_t*>(w.lp);
        const int kp = knn <= 32 ? 32 : 64, e = tid & (kp - 1), rstep = PJ_ROW_T / kp, stride = row16(knn);
        for (int h = t0; h < t0 + WV && h < nh; ++h) {
            int32_t* inv = w.inv + w.off[w.pi[h]];
            __syncthreads();
            if (tid == 0) s_n = 0;
            if (tid < nh) s_with[h - t0][tid] = 0u;
            __syncthreads();
            for (int64_t word = tid; word < l.words; word += PJ_ROW_T) {
                uint32_t b = w.bits[word * PJ_HUBS + h];
                for (int at = b ? atomicAdd(&s_n, __popc(b)) : 0; b != 0u; b &= b - 1u) inv[at++] = (int)(word * 32) + __ffs(b) - 1;
            }
            __syncthreads();
            const int n = s_n;
            for (int i0 = 0; i0 < n; i0 += rstep) {          // (uniform)
                const int i = i0 + tid / kp;
                uint32_t p = 0xffffu;
                if (i < n && e < knn) p = lp[(size_t)inv[i] * stride + e];
                const u64 same = __ballot(p == (uint32_t)h);
                const int times = __popcll(kp == 64 ? same : same >> (lane & 32) & 0xffffffffull);
                if (p < (uint32_t)nh) atomicAdd(&s_with[h - t0][p], (uint32_t)times);
            }
        }
        __syncthreads();
    }
    if (t >= nh) return;
    if (lane == 0) s_with[wv][t] = 0u;                       // the key itself
    pj_wave_sync();
    Cand<MODE> best = cand_none<MODE>();
    select_best<8>(best, H, (uint32_t)w.ppop[t], w.ppop, s_surv[wv], lane, [&](int x, uint32_t& pos, uint32_t& c) {
        pos = (uint32_t)x;
        c = x < nh ? s_with[wv][x] : w.with_hubs[(size_t)(x - nh) * PJ_HUBS + t];
    });
    write_row(adj + ((size_t)blockIdx.x * N + w.pi[t]) * deg, best, t, w.pi, N, deg, lane);
}

template <int MODE>
static void project_rows(const ProjLayout& l, char* ws, int n_graphs, int64_t N, int knn, int deg, hipStream_t st,
                         int32_t* adj) {
    // workgroups that fill the part: 4 per compute unit by position, 2 of the hash kernel, 2, 4 and 8 of the small
    // classes (LDS), all with a share of keys each; twice as many of the wavefront kernels, which not every graph needs
    auto wgs = [&](int all) { return (unsigned)(n_graphs >= all ? 1 : all / n_graphs); };
    // (a key of many lists takes its workgroup long: enough workers that no other key waits behind one)
    const dim3 threads(PJ_SMALL_WAVES * 64);
    hipLaunchKernelGGL(pj_rows_kernel<MODE>, dim3(n_graphs, wgs(4096) < 128 ? wgs(4096) : 128u), dim3(PJ_ROW_T), 0, st,
                       ws, l, N, knn, deg, adj);
    hipLaunchKernelGGL((pj_rows_wave_kernel<PJ_WAVE_SMALL_TAB, 0, MODE>), dim3(n_graphs, wgs(4096)), threads, 0, st, ws, l,
                       N, knn, deg, adj);
    if (l.cap > PJ_WAVE_SMALL_TAB)
        hipLaunchKernelGGL((pj_rows_wave_kernel<PJ_WAVE_TAB, PJ_WAVE_SMALL_TAB, MODE>), dim3(n_graphs, wgs(1024)), threads, 0,
                           st, ws, l, N, knn, deg, adj);
    if (l.cap > PJ_LDS_TAB) {
        hipLaunchKernelGGL(pj_rows_hash_kernel<MODE>, dim3(n_graphs, wgs(2048)), dim3(PJ_HASH_T), 0, st, ws, l, N,
                           knn, deg, adj);
        hipLaunchKernelGGL(pj_rows_hub_kernel<MODE>, dim3(n_graphs, l.n_hub_wg), dim3(PJ_HUB_T), 0, st, ws, l, N,
                           knn, deg, adj);
    }
    if (l.cap > PJ_WAVE_SMALL_TAB) {
        hipLaunchKernelGGL((pj_rows_small_kernel<PJ_TOUCH_C, PJ_TOUCH_B, MODE>), dim3(n_graphs, wgs(512)), threads, 0, st,
                           ws, l, N, knn, deg, adj);
        hipLaunchKernelGGL((pj_rows_small_kernel<PJ_TOUCH_B, PJ_TOUCH_A, MODE>), dim3(n_graphs, wgs(1024)), threads, 0, st,
                           ws, l, N, knn, deg, adj);
        hipLaunchKernelGGL((pj_rows_small_kernel<PJ_TOUCH_A, 0, MODE>), dim3(n_graphs, wgs(4096)), threads, 0, st, ws, l,
                           N, knn, deg, adj);
    }
    // (after the other rows: it reads their counts)
    if (l.n_slabs)
        hipLaunchKernelGGL(pj_rows_hubs_kernel<MODE>, dim3(n_graphs, PJ_HUBS * 64 / PJ_ROW_T), dim3(PJ_ROW_T), 0, st, ws, l, N,
                           knn, deg, adj);
}

// n_graphs graphs, no more than the layout is for
static ra_status project_group(const ProjLayout& l, char* ws, const int32_t* L, int n_graphs, int64_t N, int64_t M, int knn,
                               int deg, hipStream_t st, int32_t* adj, int32_t* entry) {
    const int64_t cells = M * knn;
    const unsigned gx = 256;
    const unsigned zx = N < 256 * 256 ? (unsigned)((N + 255) / 256) : gx;
    hipLaunchKernelGGL(pj_zero_kernel, dim3(zx, n_graphs), dim3(256), 0, st, ws, l, N);
    // a workgroup of the cell kernels has at least a few thousand cells, so that its table pays
    unsigned cx = (unsigned)((cells + 8191) / 8192);
    const unsigned fill = n_graphs >= 2048 ? 1u : (unsigned)(2048 / n_graphs);
    if (cx > fill) cx = fill;
    hipLaunchKernelGGL(pj_pop_kernel, dim3(cx, n_graphs), dim3(PJ_CELL_T), 0, st, L, ws, l, cells, N);
    hipLaunchKernelGGL(pj_count_kernel, dim3(l.n_blk, n_graphs), dim3(256), 0, st, ws, l, N);
    hipLaunchKernelGGL(pj_compact_kernel, dim3(l.n_blk, n_graphs), dim3(256), 0, st, ws, l, N, M);
    ra_status rc = ra_launch_sort(ws + l.o_keys, l.per_graph / 8, n_graphs, l.cap_pad, (const int32_t*)(ws + l.o_H),
                                  l.per_graph / 4, st);
    if (rc != RA_OK) return rc;
    const unsigned px = l.cap < 64 * 256 ? (unsigned)((l.cap + 255) / 256) : 64u;
    hipLaunchKernelGGL(pj_pi_kernel, dim3(px, n_graphs), dim3(256), 0, st, ws, l, M, knn, entry);
    // (24 KB of LDS: six of these workgroups per compute unit)
    const unsigned fill_inv = n_graphs >= 1536 ? 1u : (unsigned)(1536 / n_graphs);
    const dim3 inv_grid(cx < fill_inv ? cx : fill_inv, n_graphs);
    if (knn <= 32) hipLaunchKernelGGL(pj_inv_kernel<32>, inv_grid, dim3(PJ_CELL_T), 0, st, L, ws, l, M, knn, N);
    else hipLaunchKernelGGL(pj_inv_kernel<64>, inv_grid, dim3(PJ_CELL_T), 0, st, L, ws, l, M, knn, N);
    if (l.n_slabs) hipLaunchKernelGGL(pj_pairs_kernel, dim3(l.n_slabs, n_graphs), dim3(PJ_PAIR_T), 0, st, ws, l);
    if (deg % 4 == 0)
        hipLaunchKernelGGL(pj_backbone_kernel<4>, dim3(zx, n_graphs), dim3(256), 0, st, ws, l, N, deg, adj);
    else
        hipLaunchKernelGGL(pj_backbone_kernel<1>, dim3(zx, n_graphs), dim3(256), 0, st, ws, l, N, deg, adj);
    if (M <= (1 << 19)) project_rows<CAND_NARROW>(l, ws, n_graphs, N, knn, deg, st, adj);
    else project_rows<CAND_WIDE>(l, ws, n_graphs, N, knn, deg, st, adj);
    RA_HIP(hipGetLastError());
    return RA_OK;
}

// workspace: what ra_project_workspace_bytes says. (With less, as many graphs at a time as fit, if need be without the
// hubs' arrays: the same rows.)
ra_status ra_launch_project(const int32_t* L, int n_graphs, int64_t N, int64_t M, int knn, int deg,
                            void* workspace, size_t workspace_bytes, hipStream_t st, int32_t* adj, int32_t* entry) {
    if (M * (int64_t)knn >= ((int64_t)1 << 31))
        RA_FAIL(RA_EUNSUP, "M * knn must stay below 2^31 list cells");
    if (n_graphs > 65535) RA_FAIL(RA_EUNSUP, "more than 65535 graphs");
    const size_t most = workspace_bytes < PJ_MOST_BYTES ? workspace_bytes : PJ_MOST_BYTES;
    const bool hubs = proj_bytes(proj_layout(1, N, M, knn, true), 1) <= workspace_bytes;
    const int at_once = proj_graphs_at_once(n_graphs, N, M, knn, hubs, most);
    const ProjLayout l = proj_layout(at_once, N, M, knn, hubs);
    ra_status rc = RA_OK;
    for (int g = 0; g < n_graphs && rc == RA_OK; g += at_once)
        rc = project_group(l, (char*)workspace, L + (size_t)g * M * knn, n_graphs - g < at_once ? n_graphs - g : at_once, N, M,
                           knn, deg, st, adj + (size_t)g * N * deg, entry + g);
    return rc;
}
