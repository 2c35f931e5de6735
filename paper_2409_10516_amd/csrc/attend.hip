// Stand-alone attention launches (ra_attend); the device code is in attend_dev.h.
#include "attend_dev.h"
#include "ticket.h"

// Folds the slices' (max, sum, weighted sum) of a head through LDS, in slice order, and closes it (called by
// all threads; slice 0 writes).
#define AT_MERGE_SLICES 8
__device__ __forceinline__ void merge_slices(float* part, int slice, int n_slices, int t, float (&M)[2], float (&L)[2],
                                             float (&A)[2], size_t head, float* out, float* lse, float* o_om,
                                             float* lse_om, float* o_w, float* lse_w) {
    if (n_slices > 1) {
        auto at = [&](int sl, int set, int what) -> float& { return part[((sl * 2 + set) * 3 + what) * RA_D + t]; };
#pragma unroll
        for (int set = 0; set < 2; ++set) {
            at(slice, set, 0) = M[set];
            at(slice, set, 1) = L[set];
            at(slice, set, 2) = A[set];
        }
        __syncthreads();
        if (slice == 0)
            for (int b = 1; b < n_slices; ++b)
#pragma unroll
                for (int set = 0; set < 2; ++set)
                    merge_fold(M[set], L[set], A[set], at(b, set, 0), at(b, set, 1), at(b, set, 2));
    }
    if (slice == 0) merge_finish(M, L, A, t, head, out, lse, o_om, lse_om, o_w, lse_w);
}

// Where a partial launch's records are combined: by the launch itself (tickets: one word per query head, see
// ticket.h), or, with tickets null, by attend_merge_kernel afterwards.
struct AttendOut {
    uint32_t* tickets;
    float *out, *lse, *o_om, *lse_om, *o_w, *lse_w;
};

// grid: x = record slot (nS static chunks, then G x nG gathered chunks), y = G query heads, z = seq.
// kv_div consecutive grid rows share a KV head (a GQA group of more heads than a workgroup takes).
// TICKETS: whoever writes a head's last record combines them all: a workgroup stores its records past the
// L2, waits for the stores, and takes a ticket of each of its heads; the one that gets the last ticket
// reads the P records back the same way. That saves a launch (4 us of 13.5 us for the decode step's sets).
// LONG: a static workgroup has several chunks (sub of them, step apart). The decode step's sets, where that is one, have
// instances of their own, in which the run-ahead over chunks is gone: 61 registers instead of 110 (bf16, one head, no
// tickets), and in us per call, 32 query heads on 8, 100 retrieved rows: one sequence 10.55 -> 10.32, 4 16.5 -> 16.2, 16 30.4 -> 28.0;
// float32, 16 sequences 48.9 -> 41.6.
template <int DT, int G, bool TICKETS, bool LONG>
__global__ __launch_bounds__(AT_THREADS) void attend_partial_kernel(
    const void* __restrict__ q, const void* __restrict__ K, const void* __restrict__ V,
    const int32_t* __restrict__ ids, float* __restrict__ partials, int n_q, int n_kv, int64_t N,
    int s, int w, int topk, int nS, int nG, int sub, int front, float scale, int kv_div, AttendOut o) {
    extern __shared__ float smem[];
    const int kvh = blockIdx.y / kv_div, seq = blockIdx.z, x = blockIdx.x;
    const int P = nS + nG;
    const size_t esz = DT == RA_BF16 ? 2 : 4;
    const char* Kh = reinterpret_cast<const char*>(K) + ((size_t)seq * n_kv + kvh) * N * RA_D * esz;
    const char* Vh = reinterpret_cast<const char*>(V) + ((size_t)seq * n_kv + kvh) * N * RA_D * esz;
    const int h0 = blockIdx.y * G;
    const char* qg = reinterpret_cast<const char*>(q) + ((size_t)seq * n_q + h0) * RA_D * esz;
    float* rec_g = partials + ((size_t)seq * n_q + h0) * P * AT_RS;
    const int n_sub = LONG ? sub : 1, step = LONG && front ? nS : 1, first_chunk = LONG && !front ? x * sub : x;
    int first = 0, n_mine = G, slot = x;        // heads of the group this workgroup has a record of, and which
    if (x < nS) {
        RowSrc src{nullptr, N, s, w, s + w};
        if constexpr (LONG && DT == RA_BF16 && G <= 4)      // a long dense range (full attention): logits on the matrix cores
            attend_chunk_mfma<G, TICKETS>(threadIdx.x, qg, Kh, Vh, src, first_chunk, n_sub, step, scale, rec_g + (size_t)x * AT_RS,
                                          (int64_t)P * AT_RS, smem);
        else
            attend_chunk<DT, G, TICKETS, LONG>(threadIdx.x, qg, Kh, Vh, src, first_chunk, n_sub, step, scale, rec_g + (size_t)x * AT_RS,
                                         (int64_t)P * AT_RS, smem);
    } else {
        const int t = x - nS, g = t / nG, c = t % nG;
        RowSrc src{ids + ((size_t)seq * n_q + h0 + g) * topk, N, 0, 0, topk};
        attend_chunk<DT, 1, TICKETS, false>(threadIdx.x, qg + (size_t)g * RA_D * esz, Kh, Vh, src, c, 1, 1, scale,
                                     rec_g + ((size_t)g * P + nS + c) * AT_RS, 0, smem);
        first = g;
        n_mine = 1;
        slot = nS + c;
    }
    if constexpr (TICKETS) {
        __builtin_amdgcn_s_waitcnt(0x0F70);     // vmcnt(0): this wavefront's record stores have completed
        __syncthreads();                        // ... and every other's (and the LDS of the chunk is free)
        uint32_t* last = reinterpret_cast<uint32_t*>(smem);
        const size_t head0 = (size_t)seq * n_q + h0 + first;
        if ((int)threadIdx.x < n_mine) {
            const uint32_t step = ticket_step(slot, P);
            last[threadIdx.x] = ticket_last(__hip_atomic_fetch_add(o.tickets + head0 + threadIdx.x, step, __ATOMIC_RELAXED,
                                                                   __HIP_MEMORY_SCOPE_AGENT), step);
        }
        __syncthreads();
        bool mine[G];
#pragma unroll
        for (int g = 0; g < G; ++g) mine[g] = g < n_mine && last[g] != 0u;
        __syncthreads();                        // (read before the merge reuses the LDS)
        constexpr int SL = AT_THREADS / RA_D;
        const int t = threadIdx.x % RA_D, slice = threadIdx.x / RA_D;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            if (!mine[g]) continue;             // (uniform)
            const size_t head = head0 + g;
            float M[2] = {-INFINITY, -INFINITY}, L[2] = {0.f, 0.f}, A[2] = {0.f, 0.f};
            merge_accumulate<true>(partials + head * P * AT_RS, nS, nG, t, slice, SL, M, L, A);
            merge_slices(smem, slice, SL, t, M, L, A, head, o.out, o.lse, o.o_om, o.lse_om, o.o_w, o.lse_w);
            if (g + 1 < G) __syncthreads();
        }
    }
}

// grid: x = query head, y = seq; block = n_slices x 128 threads (one per slice of the records and
// output dimension). A head with more than sixteen records (a long static range: full attention)
// has its batches of sixteen dealt to up to AT_MERGE_SLICES slices that run side by side and are
// folded through LDS, in slice order, by the first.
__global__ __launch_bounds__(AT_MERGE_SLICES * RA_D) void attend_merge_kernel(
    const float* __restrict__ partials, int n_q, int nS, int nG, AttendOut o) {
    __shared__ float part[AT_MERGE_SLICES * 2 * 3 * RA_D];       // [slice][set][M, L, A][dimension]
    const size_t head = (size_t)blockIdx.y * n_q + blockIdx.x;
    const int t = threadIdx.x % RA_D, slice = threadIdx.x / RA_D, n_slices = blockDim.x / RA_D;
    float M[2] = {-INFINITY, -INFINITY}, L[2] = {0.f, 0.f}, A[2] = {0.f, 0.f};
    merge_accumulate<false>(partials + head * (nS + nG) * AT_RS, nS, nG, t, slice, n_slices, M, L, A);
    merge_slices(part, slice, n_slices, t, M, L, A, head, o.out, o.lse, o.o_om, o.lse_om, o.o_w, o.lse_w);
}

// Static chunks: 64 rows each for the decode step's few hundred static rows; a long static range (full
// attention) is cut so that its workgroups are about two per compute unit (the kernel's vector
// registers allow two side by side; one for the float32 kernel of eight heads), all running from start
// to end. Measured for full attention over 131072 tokens, 8 KV heads (us per layer): 32 records per
// head 178, 64 records 115, 128 records 123, 256 records 136; with the number of sub-chunks rounded up to
// a power of two a context of 100003 tokens had 392 workgroups on 512 places (88 us; 74 us with 504).
#define AT_MAX_STATIC_CHUNKS 64     // most chunks of 64 rows that get a record each

// Query heads that one workgroup of a long static range serves, of a group of G. bf16 goes through the
// matrix cores, which the kernel does for up to four heads: a group of eight takes two workgroups, which
// find each other's rows in the L2 (131072 tokens, 32 heads on 4: 110 us with eight heads on the vector
// units, 81 us); float32 is bound by the loads (180 us with four heads, 145 us with eight).
static int long_heads(ra_dtype dt, int G) { return G == 2 || G == 4 ? G : G == 8 ? (dt == RA_BF16 ? 4 : 8) : 1; }

// The same for the decode step's sets, in a launch of `records` records. A launch of few workgroups is
// bound by its latency, and a static chunk for g heads takes g times the arithmetic and closes g
// records one after the other: every query head reads its static rows itself then (the heads of a
// group find them in the L2). Beyond, bf16 takes two heads, float32, with rows twice as wide, two and then four.
// Measured (us per call, 32 query heads, 100 retrieved rows; 1 / 2 / 4 / 8 heads):
//   bf16, 640 static rows, G 4: 416 records 10.7 / 12.9 / 21.0, 832 10.4 / 10.7 / 14.0, 1664 15.8 / 14.7 / 16.3,
//     3328 22.2 / 21.1 / 24.5, 13312 63 / 56 / 68; G 2 and 8 within 3 % of these; G 8 with eight heads 38, 17, 22, 34, 108.
//   float32, 640 static rows, G 4: 416 records 11.1 / 13.3 / 21.4, 832 16.4 / 11.7 / 15.0, 1664 23.0 / 19.8 / 18.6,
//     3328 36 / 28.5 / 28.1, 13312 119 / 89 / 84; G 8: 832 16.4 / 11.6 / 14.9 / 18.5, 1664 22.9 / 19.4 / 18.7 / 24.5.
// What the lines rest on is the number of records alone: one head up to about 1000 (bf16) and 500 (float32), whatever G
// is. The lines below grow with G, so some launches between are not served best: bf16, G 4 and 8, 1664 records (15.8
// where two heads take 14.7); float32, G 2, 192 to 416 records (12.3 to 13.4 where one head takes 8.7 to 11.2), and G 8,
// 832 and 1664 records (16.4 and 22.9 where two take 11.6 and four 18.7).
static int short_heads(ra_dtype dt, int G, int64_t records) {
    if (G != 2 && G != 4 && G != 8) return 1;
    if (records <= (dt == RA_BF16 ? 512 * G : 32 * G * G)) return 1;
    if (dt == RA_BF16 || G == 2) return 2;
    return G == 4 && records <= 1024 ? 2 : 4;
}

static int static_sub(ra_dtype dt, int rows, int n_seq, int n_q, int n_kv) {
    const int chunks = (rows + AT_CH - 1) / AT_CH;
    if (chunks <= AT_MAX_STATIC_CHUNKS) return 1;
    const int g = long_heads(dt, n_q / n_kv);
    int records = (g == 8 ? 256 : 512) / (n_seq * n_q / g);
    if (records < 4) records = 4;
    if (records > chunks / 2) records = chunks / 2;
    return (chunks + records - 1) / records;
}

size_t ra_attend_partial_floats(ra_dtype dt, int n_seq, int n_q, int n_kv, int64_t N, int sink, int window,
                                int topk) {
    int s, w;
    static_ranges(N, sink, window, &s, &w);
    const int sub = static_sub(dt, s + w, n_seq, n_q, n_kv);
    const int nS = (s + w + AT_CH * sub - 1) / (AT_CH * sub), nG = (topk + AT_CH - 1) / AT_CH;
    return (size_t)n_seq * n_q * (nS + nG) * AT_RS;
}

// Up to so many records the last workgroup of a head combines them (13 records of 32 heads: 12.4 -> 10.3 us).
// Storing records past the L2 and taking tickets costs each workgroup more than a launch costs all
// of them when there are many: 2900 records took twice as long that way.
#define AT_TICKET_RECORDS 512

ra_status ra_launch_attend(const void* q, const void* K, const void* V, ra_dtype dt, int n_seq,
                           int n_q, int n_kv, int64_t N, int sink, int window, int topk,
                           const int32_t* ids, float* partials, uint32_t* tickets, hipStream_t st, float* out,
                           float* lse, float* o_omega, float* lse_omega, float* o_w,
                           float* lse_w) {
    int s, w;
    static_ranges(N, sink, window, &s, &w);
    const int G = n_q / n_kv;
    const int sub = static_sub(dt, s + w, n_seq, n_q, n_kv);
    const int nS = (s + w + AT_CH * sub - 1) / (AT_CH * sub), nG = ids ? (topk + AT_CH - 1) / AT_CH : 0;
    const float scale = 1.0f / sqrtf((float)RA_D);
    const size_t lds = (size_t)AT_CHUNK_LDS_FLOATS * sizeof(float);
    const int64_t records = (int64_t)(nS + nG) * n_q * n_seq;
    if (records > AT_TICKET_RECORDS) tickets = nullptr;
    // Workgroups of a long static range that take its chunks in turn read side by side, as one front per head, which the
    // memory serves better than a stream of its own for each, unless the heads lie a multiple of 1 MB apart, where their fronts meet
    // in the same channels; one head by itself meets none. Layers in turn, us per layer, streams of their own -> fronts. bf16, 8 KV
    // heads: 60001 tokens 54.6 -> 53.0, 100003 79.0 -> 75.3, 200000 140.7 -> 137.5; near a multiple, 65537 56.6 -> 56.6, 66048
    // 59.4 -> 58.2, 131200 97.8 -> 98.2; at one, 65536 54.2 -> 53.8, 131072 96.4 -> 96.7, 8 heads without groups 87.4 -> 89.0, 16
    // sequences of 32768 339 -> 342. 16 sequences of other lengths go either way by 3 %, with where their tensors lie. One
    // head: 131072 38.7 -> 38.3, 1M 105.6 -> 103.2, float32 262144 67.6 -> 65.5.
    const bool apart = n_seq * n_kv == 1 || ((size_t)N * RA_D * (dt == RA_BF16 ? 2 : 4)) % ((size_t)1 << 20) != 0;
    const int front = sub > 1 && apart;
    const AttendOut o{tickets, out, lse, o_omega, lse_omega, o_w, lse_w};
    const int g = sub > 1 ? long_heads(dt, G) : short_heads(dt, G, records);
    const dim3 grid(nS + g * nG, n_q / g, n_seq);
    if (nS + nG > 0) {
#define RA_AT_GO(DTV, GG, LG, TK)                                                                                 \
    hipLaunchKernelGGL((attend_partial_kernel<DTV, GG, TK, LG>), grid, dim3(AT_THREADS), lds, st, q, K, V, ids, partials, \
                       n_q, n_kv, N, s, w, topk, nS, nG, sub, front, scale, G / g, o)
#define RA_AT_TK(DTV, GG, LG)                                                                                     \
    do { if (tickets) RA_AT_GO(DTV, GG, LG, true); else RA_AT_GO(DTV, GG, LG, false); } while (0)
#define RA_AT_LG(DTV, GG)                                                                                         \
    do { if (sub > 1) RA_AT_TK(DTV, GG, true); else RA_AT_TK(DTV, GG, false); } while (0)
        // (long_heads and short_heads say which of these there are)
        if (dt == RA_BF16) {
            if (g == 1) RA_AT_LG(RA_BF16, 1);
            else if (g == 2) RA_AT_LG(RA_BF16, 2);
            else RA_AT_TK(RA_BF16, 4, true);
        } else {
            if (g == 1) RA_AT_LG(RA_F32, 1);
            else if (g == 2) RA_AT_LG(RA_F32, 2);
            else if (g == 4) RA_AT_LG(RA_F32, 4);
            else RA_AT_TK(RA_F32, 8, true);
        }
#undef RA_AT_LG
#undef RA_AT_TK
#undef RA_AT_GO
        RA_HIP(hipGetLastError());
    }
    if (tickets && nS + nG > 0) return RA_OK;
    int slices = (nS + nG + 15) / 16;                     // one per batch of sixteen records, at most 8
    if (slices > AT_MERGE_SLICES) slices = AT_MERGE_SLICES;
    if (slices < 1) slices = 1;
    hipLaunchKernelGGL(attend_merge_kernel, dim3(n_q, n_seq), dim3(slices * RA_D), 0, st, partials, n_q, nS,
                       nG, o);
    RA_HIP(hipGetLastError());
    return RA_OK;
}


// ---- ra_attend for callers that cannot allocate ---------------------------------------------------
// The partial records live in a file-scope device array instead of memory the handle allocates on
// first use. Every device the library runs on holds its own copy of the array at its own address;
// host code never passes the array's name to a kernel, only the address hipGetSymbolAddress gives
// for the current device (looked up once per device and kept).
static __device__ __align__(256) unsigned char scratch[RA_ATTEND_NOALLOC_SCRATCH_BYTES];
// one ticket per head that fits (a head has a record at least); they bring themselves back to zero (ticket.h)
static __device__ uint32_t scratch_tickets[RA_ATTEND_NOALLOC_SCRATCH_BYTES / (AT_RS * 4)];
static void* g_scratch_addr[RA_MAX_DEVICES];
static uint32_t* g_ticket_addr[RA_MAX_DEVICES];

static ra_status scratch_address(void** out, uint32_t** tickets) {
    int dev = 0;
    RA_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= RA_MAX_DEVICES) RA_FAIL(RA_EUNSUP, "device %d out of range", dev);
    if (!g_scratch_addr[dev]) {
        void* p = nullptr;
        RA_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) RA_FAIL(RA_EHIP, "the scratch array has no address on device %d", dev);
        void* t = nullptr;
        RA_HIP(hipGetSymbolAddress(&t, HIP_SYMBOL(scratch_tickets)));
        g_ticket_addr[dev] = reinterpret_cast<uint32_t*>(t);
        g_scratch_addr[dev] = p;
    }
    *out = g_scratch_addr[dev];
    *tickets = g_ticket_addr[dev];
    return RA_OK;
}

ra_status ra_launch_attend_noalloc(const void* q, const void* K, const void* V, ra_dtype dt, int n_seq,
                                   int n_q, int n_kv, int64_t N, int sink, int window, int topk,
                                   const int32_t* ids, hipStream_t st, float* out, float* lse,
                                   float* o_omega, float* lse_omega, float* o_w, float* lse_w) {
    const size_t need = ra_attend_partial_floats(dt, n_seq, n_q, n_kv, N, sink, window, topk) * sizeof(float);
    if (need > RA_ATTEND_NOALLOC_SCRATCH_BYTES)
        RA_FAIL(RA_EUNSUP, "the partial records of this call take %zu bytes, above the %u bytes "
                "ra_attend_noalloc keeps (use ra_attend)", need, (unsigned)RA_ATTEND_NOALLOC_SCRATCH_BYTES);
    void* ptr = nullptr;
    uint32_t* tickets = nullptr;
    ra_status rc = scratch_address(&ptr, &tickets);
    if (rc != RA_OK) return rc;
    // nothing to clear: every record the merge reads is written by this call, and the tickets are zero
    // whenever no call is running, also after calls that overlapped
    return ra_launch_attend(q, K, V, dt, n_seq, n_q, n_kv, N, sink, window, topk, ids,
                            reinterpret_cast<float*>(ptr), tickets, st, out, lse, o_omega, lse_omega, o_w, lse_w);
}
