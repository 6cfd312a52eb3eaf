// Upper bounds of the fused scores of a batch of queries against every document: what lets a search drop a neighbour
// that cannot enter its pool on one 4-byte read, instead of reading its record (1.3 KB) and often its dense row (3 KB),
// and lets the exact top-k score a few hundred documents per query instead of all.
//
//   table[q][d] >= w_d <q_d,d_d> + w_s <q_s,d_s> + w_f <q_f,d_f>   as the scoring kernels round it.
//
// The dense part and the most frequent terms of both vocabularies (the "head": at most AP_BOUND_HEAD columns) are one
// bf16 matrix product; the remaining terms (the "tail") are added to a tile of it from postings of the tile's documents.  Rounding to bf16 is paid for by a
// slack per pair, made of what it took off the two sides, so nothing that decides a result depends on the product's precision: a candidate the bound lets
// through is scored as ever, and one it stops could not have entered.
#include <math.h>
#include <algorithm>
#include <new>
#include "ap_tiles.hpp"

int ap_validate_queries(const ap_queries *q);

#define AP_BOUND_HEAD 512
#define AP_BOUND_QMAX 1e14f
#define AP_BOUND_DMAX 1e15f
#define AP_BOUND_QT 256              // queries and documents of a tile
#define AP_BOUND_VOCAB ((int64_t)1 << 24)   // terms of both vocabularies together a table of columns is kept for
#define AP_BOUND_BITS_MIN 8          // buckets of a tile's postings: 2^8 to 2^13, for long lists up to 2^15 (128 KB of LDS at ingest)
#define AP_BOUND_BITS 13
#define AP_BOUND_BITS_LONG 15
#define AP_BOUND_TERMS 4             // terms of a query that a lane looks up at once
#define AP_BOUND_LIST (1 + 128)      // a query's tail as the product's kernel reads it: (entries, AP_BOUND_NONE or the first term of the lists that found no place), then (term, weighted value)
#define AP_BOUND_NONE 0xffffffffu
#define AP_BOUND_MUCH 16             // entries of a bucket beyond those for which a query's eight lanes read it together
#define AP_BOUND_AHEAD 4             // postings of a bucket that are read at once, and entries behind the last one for it

// The workspaces of an index: one per stream that searches it (at most AP_BOUND_STREAMS; insertion and large exact top-k
// give theirs back, the others only grow), so that searches
// of one index on several streams do not share a table.  A further stream gets the one that has been idle longest; while all
// of them are at work it goes without.  `done` is recorded behind a workspace's last use.
#define AP_BOUND_STREAMS 4
struct ApBoundPool {
    std::mutex lock;
    struct { hipStream_t stream; void *mem; size_t bytes; hipEvent_t done; uint64_t last; } ws[AP_BOUND_STREAMS];
    int used = 0;
    uint64_t uses = 0;
};

// ------------------------------------------------------------------ ingest
__global__ __launch_bounds__(256) void k_bd_hist(const int32_t *__restrict__ df_sp, int32_t nsp, const int32_t *__restrict__ df_tx, int32_t ntx,
                                                 int32_t *__restrict__ hist) {
    __shared__ int32_t h[256];
    h[threadIdx.x] = 0;
    __syncthreads();
    for (int64_t t = blockIdx.x * (int64_t)256 + threadIdx.x; t < (int64_t)nsp + ntx; t += (int64_t)gridDim.x * 256) {
        const int b = ap_df_bin(t < nsp ? df_sp[t] : df_tx[t - nsp]);
        if (b >= 0) atomicAdd(&h[b], 1);
    }
    __syncthreads();
    if (h[threadIdx.x]) atomicAdd(&hist[threadIdx.x], h[threadIdx.x]);
}
int ap_df_histogram(const int32_t *df_sp, int32_t nsp, const int32_t *df_tx, int32_t ntx, int32_t *hist, hipStream_t st) {
    const int64_t all = (int64_t)nsp + ntx;
    hipLaunchKernelGGL(k_bd_hist, dim3((unsigned)std::min<int64_t>((all + 255) / 256, 256)), dim3(256), 0, st, df_sp, nsp, df_tx, ntx, hist);
    AP_CHECK_HIP(hipGetLastError());
    return AP_OK;
}
// The head is every term of the top bins that fit kh columns together.  *taken counts columns.
__global__ __launch_bounds__(1024) void k_bd_pick(const int32_t *__restrict__ df_sp, int32_t nsp, const int32_t *__restrict__ df_tx, int32_t ntx,
                                                  const int32_t *__restrict__ hist, int32_t kh, int32_t *__restrict__ col, uint32_t *__restrict__ taken) {
    __shared__ int32_t s_low, s_hist[256];
    if (threadIdx.x < 256) s_hist[threadIdx.x] = hist[threadIdx.x];
    __syncthreads();
    if (threadIdx.x == 0) {
        int32_t low = 256, sum = 0;
        while (low > 0 && sum + s_hist[low - 1] <= kh) sum += s_hist[--low];
        s_low = low;
    }
    __syncthreads();
    const int64_t t = blockIdx.x * (int64_t)1024 + threadIdx.x;
    if (t >= (int64_t)nsp + ntx) return;
    const int32_t df = t < nsp ? df_sp[t] : df_tx[t - nsp];
    col[t] = df > 0 && ap_df_bin(df) >= s_low ? (int32_t)atomicAdd(taken, 1u) : -1;
}

// A tile's postings: the tail entries of AP_BOUND_QT consecutive documents, grouped by a hash of their terms.  An entry is
// (term << 8 | document in the tile, value bits); terms of both vocabularies count through and stay below AP_BOUND_VOCAB.
// The tile's entries begin where its documents' lists do (both vocabularies' offsets together), start[b] is where those of
// bucket b do behind that.  One block per tile; the order within a bucket is left to chance, and with it the order in which the terms of a query are
// added to a document's entry: bounds, and the counters of what they keep from being scored, may differ by a last place between two ingests of a corpus.
// That an entry is an upper bound does not depend on it, so ids and scores do not.
static_assert(AP_BOUND_VOCAB <= (int64_t)1 << 24 && AP_BOUND_QT == 256, "a term and a document of a tile share a word");
__device__ __forceinline__ uint32_t ap_bound_bucket(uint32_t t, int bits) { return (t * 0x9E3779B1u) >> (32 - bits); }
__device__ __forceinline__ void ap_bd_post(const ApVecs &D, int64_t tile, int32_t nsp, const int32_t *__restrict__ col, int bits, uint32_t *__restrict__ start,
                                           uint2 *__restrict__ post, uint32_t *post_cnt /* 1 << bits */) {
    __shared__ uint32_t part[16], begin[2][AP_BOUND_QT];   // where the documents' lists begin (past the end: behind all entries)
    const int lane = threadIdx.x & 63, wave = ap_wave_id(), buckets = 1 << bits;
    const int64_t d0 = tile * AP_BOUND_QT, d1 = d0 + AP_BOUND_QT < D.n ? d0 + AP_BOUND_QT : D.n;
    const int64_t from[2] = {D.sp_indptr[d0], D.tx_indptr[d0]};
    uint2 *to = post + from[0] + from[1];
    if (threadIdx.x < 2 * AP_BOUND_QT) {
        const int64_t v = d0 + threadIdx.x % AP_BOUND_QT;
        const int p = threadIdx.x / AP_BOUND_QT;
        begin[p][threadIdx.x % AP_BOUND_QT] = v < d1 ? (uint32_t)((p ? D.tx_indptr[v] : D.sp_indptr[v]) - from[p]) : 0xffffffffu;
    }
    uint32_t *first = start + tile * (buckets + 1);
    for (int b = threadIdx.x; b < buckets; b += 1024) post_cnt[b] = 0;
    __syncthreads();
    // four entries a thread at once, term by term and vocabulary by vocabulary
    auto each = [&](auto &&f) {
        for (int p = 0; p < 2; p++) {
            const int32_t *idx = p ? D.tx_idx : D.sp_idx;
            const int64_t e = p ? D.tx_indptr[d1] : D.sp_indptr[d1];
            for (int64_t i0 = (p ? D.tx_indptr[d0] : D.sp_indptr[d0]) + threadIdx.x; i0 < e; i0 += 4096) {
                int32_t t[4], c[4];
#pragma unroll
                for (int j = 0; j < 4; j++) t[j] = (p ? nsp : 0) + idx[i0 + 1024 * j < e ? i0 + 1024 * j : i0];
#pragma unroll
                for (int j = 0; j < 4; j++) c[j] = i0 + 1024 * j < e ? col[t[j]] : 0;
                f(p, i0, t, c);
            }
        }
    };
    each([&](int, int64_t, const int32_t (&t)[4], const int32_t (&c)[4]) {
#pragma unroll
        for (int j = 0; j < 4; j++)
            if (c[j] < 0) atomicAdd(&post_cnt[ap_bound_bucket((uint32_t)t[j], bits)], 1u);
    });
    __syncthreads();
    const int per = (buckets + 1023) / 1024, b0 = (int)threadIdx.x * per;
    uint32_t sum = 0;
    for (int b = b0; b < b0 + per && b < buckets; b++) sum += post_cnt[b];
    uint32_t upto = sum;
    for (int o = 1; o < 64; o <<= 1) { const uint32_t up = __shfl_up(upto, o, 64); if (lane >= o) upto += up; }
    if (lane == 63) part[wave] = upto;
    __syncthreads();
    uint32_t at = upto - sum;
    for (int w = 0; w < wave; w++) at += part[w];
    for (int b = b0; b < b0 + per && b < buckets; b++) {
        const uint32_t c = post_cnt[b];
        post_cnt[b] = first[b] = at;
        at += c;
    }
    if (threadIdx.x == 1023) first[buckets] = at;
    __syncthreads();
    each([&](int p, int64_t i0, const int32_t (&t)[4], const int32_t (&c)[4]) {
        const float *val = p ? D.tx_val : D.sp_val;
        float x[4];
#pragma unroll
        for (int j = 0; j < 4; j++) x[j] = c[j] < 0 ? val[i0 + 1024 * j] : 0.f;
#pragma unroll
        for (int j = 0; j < 4; j++)
            if (c[j] < 0) {
                int d = 0;   // the last document whose list begins at or before the entry
                for (int o = AP_BOUND_QT / 2; o > 0; o >>= 1)
                    if (begin[p][d + o] <= (uint32_t)(i0 + 1024 * j - from[p])) d += o;
                to[atomicAdd(&post_cnt[ap_bound_bucket((uint32_t)t[j], bits)], 1u)] = make_uint2((uint32_t)t[j] << 8 | (uint32_t)d, __float_as_uint(x[j]));
            }
    });
}

__device__ __forceinline__ uint32_t ap_bf16_bits(float f) { return (uint32_t)__builtin_bit_cast(uint16_t, (__bf16)f); }   // to nearest even

__device__ __forceinline__ float ap_bf16_value(uint32_t bits) { return __uint_as_float(bits << 16); }

// The first blocks take a tile's postings each (one launch, since a few tiles leave the chip idle: 2,000 documents 42 -> 26 us), the others a wave
// per document: its bound row (dense part rounded to bf16 if kd > 0, then the head columns), what the slack of its
// column is made of, and its bit in the bitmaps of the lexical head terms it holds.  norms: planes of n
// entries for the dense part and the head columns of either vocabulary, each the norm of what rounding to bf16 took off the
// part (exact differences: a value and its rounding lie within a factor of two) and the part's own norm.
template <int DT>
__global__ __launch_bounds__(1024) void k_bd_rows(ApVecs D, int32_t nsp, const int32_t *__restrict__ col, int32_t kd, int32_t kh, uint16_t *__restrict__ rows,
                                                  const float *__restrict__ dnorm, float2 *__restrict__ norms, uint32_t *__restrict__ bits, int64_t words,
                                                  uint32_t tiles, int bucket_bits, uint32_t *__restrict__ start, uint2 *__restrict__ post) {
    extern __shared__ __attribute__((aligned(16))) uint32_t bd_lds[];   // a tile's buckets, or a head row per wave
    if (blockIdx.x < tiles) {   // uniform
        ap_bd_post(D, blockIdx.x, nsp, col, bucket_bits, start, post, bd_lds);
        return;
    }
    const int lane = threadIdx.x & 63, wave = ap_wave_id();
    uint16_t *head = reinterpret_cast<uint16_t *>(bd_lds) + wave * AP_BOUND_HEAD;
    const int32_t ld = kd + kh;
    for (int64_t v = (int64_t)(blockIdx.x - tiles) * 16 + wave; v < D.n; v += (int64_t)(gridDim.x - tiles) * 16) {
        uint16_t *row = rows + v * ld;
        float sum[2] = {0.f, 0.f}, lost[3] = {0.f, 0.f, 0.f};
        for (int32_t c = lane * 4; c < kd; c += 256) {
            float x[4] = {0.f, 0.f, 0.f, 0.f};
            uint32_t y16[4];
            if (c < D.dim) {   // dim is a multiple of 4
                if (DT == AP_F32) {
                    const float4 y = *reinterpret_cast<const float4 *>(static_cast<const float *>(D.dense) + v * D.dim + c);
                    x[0] = y.x; x[1] = y.y; x[2] = y.z; x[3] = y.w;
                } else {
                    for (int e = 0; e < 4; e++) x[e] = __uint_as_float((uint32_t)static_cast<const uint16_t *>(D.dense)[v * D.dim + c + e] << 16);
                }
            }
#pragma unroll
            for (int e = 0; e < 4; e++) {
                y16[e] = ap_bf16_bits(x[e]);
                const float off = x[e] - ap_bf16_value(y16[e]);
                lost[0] = fmaf(off, off, lost[0]);
            }
            *reinterpret_cast<uint2 *>(row + c) = make_uint2(y16[0] | (y16[1] << 16), y16[2] | (y16[3] << 16));
        }
        for (int32_t c = lane * 8; c < kh; c += 512) *reinterpret_cast<uint4 *>(head + c) = make_uint4(0, 0, 0, 0);
        ap_wave_sync();
        for (int part = 0; part < 2; part++) {
            const int64_t b = part ? D.tx_indptr[v] : D.sp_indptr[v], e = part ? D.tx_indptr[v + 1] : D.sp_indptr[v + 1];
            for (int64_t p = b + lane; p < e; p += 64) {
                const int32_t t = part ? nsp + D.tx_idx[p] : D.sp_idx[p];
                const float x = part ? D.tx_val[p] : D.sp_val[p];
                const int32_t c = col[t];
                if (c >= 0) {
                    const uint32_t h = ap_bf16_bits(x);
                    const float off = x - ap_bf16_value(h);
                    head[c] = (uint16_t)h; sum[part] = fmaf(x, x, sum[part]); lost[1 + part] = fmaf(off, off, lost[1 + part]);
                    if (part) atomicOr(&bits[c * words + (v >> 5)], 1u << (v & 31));
                }
            }
        }
        ap_wave_sync();
        for (int32_t c = lane * 8; c < kh; c += 512) *reinterpret_cast<uint4 *>(row + kd + c) = *reinterpret_cast<const uint4 *>(head + c);
        const float hs = ap_wave_sum(sum[0]), hf = ap_wave_sum(sum[1]);
        for (int p = 0; p < 3; p++) lost[p] = ap_wave_sum(lost[p]);
        if (lane == 0) {
            norms[v] = make_float2(sqrtf(lost[0]), dnorm[v]);
            norms[D.n + v] = make_float2(sqrtf(lost[1]), sqrtf(hs));
            norms[2 * D.n + v] = make_float2(sqrtf(lost[2]), sqrtf(hf));
        }
        ap_wave_sync();
    }
}

static inline size_t ap_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Lays out what the bounds of a corpus need, if that is at most 1/share of the free memory.  Without it (vocabularies too
// large for a table of columns, not enough memory) the searches run without bounds: never an error.
int ap_bound_ingest(ap_index *ix, int share, hipStream_t st) {
    const ap_corpus &c = ix->corpus;
    const int64_t all = (int64_t)c.sp_vocab + c.tx_vocab;
    if (all > AP_BOUND_VOCAB) return AP_OK;
    const bool own_dense = c.dense_dtype != AP_BF16 || c.dim % AP_BK16 != 0;   // else the corpus's rows are read where they lie
    const int32_t kd = own_dense ? (int32_t)ap_up((size_t)c.dim, AP_BK16) : 0;
    const int32_t kh = (int32_t)std::min<int64_t>(AP_BOUND_HEAD, (int64_t)ap_up((size_t)all, AP_BK16));
    const size_t nnz = (size_t)ix->tx_nnz + (size_t)ix->sp_nnz;
    const int64_t words = (c.n + 31) / 32;
    // two buckets for three entries of a tile's lists, about half of which are in the tail, as far as 2^13 buckets go (2^14 for 165 entries a document:
    // 1 to 8 % off the product and the tail, for twice the memory and 20 us at ingest), and more once a bucket would have over eight
    // entries, which every lookup reads past.  20,000 documents of 1,279 entries out of 500,000 terms, 1,000 queries of 28, 300 and 1,500 terms: 2^13 buckets
    // 0.44, 2.79 and 15.0 ms, 2^15 0.37, 2.26 and 11.7, 2^16 0.36, 2.17 and 11.4, for which ingest would have to go through the lists twice (3.3 -> 4.0 ms).
    const int64_t doc_tiles = (c.n + AP_BOUND_QT - 1) / AP_BOUND_QT;
    int bits = AP_BOUND_BITS_MIN;
    while (bits < AP_BOUND_BITS && ((int64_t)1 << bits) * 3 * doc_tiles < 2 * (int64_t)nnz) bits++;
    while (bits >= AP_BOUND_BITS && bits < AP_BOUND_BITS_LONG && ((int64_t)1 << bits) * 8 * doc_tiles < (int64_t)nnz) bits++;
    if (g_ap_debug.bound_buckets > 0) bits = (int)std::min<int64_t>(std::max<int64_t>(g_ap_debug.bound_buckets, AP_BOUND_BITS_MIN), AP_BOUND_BITS_LONG);
    // cleared: document frequencies of the learned-sparse terms, histogram, columns taken, bitmaps
    const size_t n_clear = (size_t)c.sp_vocab + 256 + 1 + (size_t)kh * (size_t)words;
    size_t at = 0;
    auto take = [&](size_t bytes) { const size_t a = at; at += ap_up(bytes, 256); return a; };
    const size_t o_clear = take(n_clear * 4), o_col = take((size_t)all * 4), o_start = take((size_t)doc_tiles * (((size_t)1 << bits) + 1) * 4), o_post = take((nnz + AP_BOUND_AHEAD) * 8),
                 o_norms = take((size_t)c.n * 24), o_rows = take((size_t)c.n * (size_t)(kd + kh) * 2);
    size_t free_b = 0, total_b = 0;
    if (hipMemGetInfo(&free_b, &total_b) != hipSuccess || at > free_b / (size_t)share) { (void)hipGetLastError(); return AP_OK; }
    if (!ix->bd_pool && !(ix->bd_pool = new (std::nothrow) ApBoundPool())) { ap_set_error("out of host memory"); return AP_ENOMEM; }
    if (hipMalloc(&ix->bd_mem, at) != hipSuccess) { (void)hipGetLastError(); ix->bd_mem = nullptr; return AP_OK; }
    char *m = static_cast<char *>(ix->bd_mem);
    int32_t *df_sp = reinterpret_cast<int32_t *>(m + o_clear);
    int32_t *hist = df_sp + c.sp_vocab;
    uint32_t *taken = reinterpret_cast<uint32_t *>(hist + 256);
    ix->bd_df = df_sp;
    ix->bd_col = reinterpret_cast<int32_t *>(m + o_col);
    ix->bd_start = reinterpret_cast<uint32_t *>(m + o_start);
    ix->bd_start_bits = bits;
    ix->bd_post = reinterpret_cast<uint2 *>(m + o_post);
    ix->bd_norms = reinterpret_cast<float2 *>(m + o_norms);
    ix->bd_rows = reinterpret_cast<uint16_t *>(m + o_rows);
    ix->bd_bits = taken + 1;
    ix->bd_kd = kd; ix->bd_kh = kh;
    AP_TRY(ap_fill_u32(df_sp, n_clear, 0u, st));
    if (ix->sp_nnz > 0)
        AP_TRY(ap_count_terms(c.sp_idx, nullptr, ix->sp_nnz, df_sp, nullptr, st));
    AP_TRY(ap_df_histogram(df_sp, c.sp_vocab, ix->df, c.tx_vocab, hist, st));
    hipLaunchKernelGGL(k_bd_pick, dim3((unsigned)((all + 1023) / 1024)), dim3(1024), 0, st, df_sp, c.sp_vocab, ix->df, c.tx_vocab, hist, kh, ix->bd_col, taken);
    const dim3 g((unsigned)(doc_tiles + std::min<int64_t>((c.n + 15) / 16, 1024)));
    const size_t lds = std::max((size_t)4 << bits, (size_t)16 * AP_BOUND_HEAD * 2);
    if (lds > 48 * 1024) {
        const void *f = ix->dtype == AP_F32 ? reinterpret_cast<const void *>(&k_bd_rows<AP_F32>) : reinterpret_cast<const void *>(&k_bd_rows<AP_BF16>);
        AP_CHECK_HIP(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    }
    if (ix->dtype == AP_F32)
        hipLaunchKernelGGL(k_bd_rows<AP_F32>, g, dim3(1024), lds, st, ix->docs, c.sp_vocab, ix->bd_col, kd, kh, ix->bd_rows, ix->dense_norm, ix->bd_norms, ix->bd_bits, words, (uint32_t)doc_tiles, bits, ix->bd_start, ix->bd_post);
    else
        hipLaunchKernelGGL(k_bd_rows<AP_BF16>, g, dim3(1024), lds, st, ix->docs, c.sp_vocab, ix->bd_col, kd, kh, ix->bd_rows, ix->dense_norm, ix->bd_norms, ix->bd_bits, words, (uint32_t)doc_tiles, bits, ix->bd_start, ix->bd_post);
    AP_CHECK_HIP(hipGetLastError());
    return AP_OK;
}

// ------------------------------------------------------------------ the table
__device__ __forceinline__ float ap_bound_value(float entry) { return __uint_as_float(__float_as_uint(entry) & ~AP_BOUND_COUNT); }
// Entries carry a count in their low bits (keyword searches: how many of the query's required terms the document holds);
// what clearing them takes off a value (2^-18 of it) is added first, and what the additions of the tail may have: rel is at
// least 1e-5 and 2^-22 for each of them.
__device__ __forceinline__ float ap_bound_round(float v, float rel) {
    return __uint_as_float(__float_as_uint(fmaf(fabsf(v), rel, v)) & ~AP_BOUND_COUNT);
}
__device__ __forceinline__ void ap_lds_add(float *at, float v) { (void)unsafeAtomicAdd(at, v); }   // ds_add_f32

// What the product's kernel adds the tail from: the queries' lists and weights, the tiles' postings, and for keyword
// searches the required terms (the head's are asked of the bitmaps).
struct ApBoundTail {
    const float *w;
    int32_t w_stride, nsp, ntx, bits, kw_stride;
    int64_t q0;
    const int64_t *q_sp_indptr, *q_tx_indptr;
    const int32_t *q_sp_idx, *q_tx_idx;
    const float *q_sp_val, *q_tx_val;
    const int64_t *sp_indptr, *tx_indptr;   // of the documents
    const uint2 *lists;                     // per row of the table AP_BOUND_LIST entries
    const uint32_t *start;
    const uint2 *post;
    const int32_t *kw_terms;
};
static_assert(128 * AP_BOUND_QT * 4 <= AP_BIG_LDS_BYTES, "half a tile takes the place of the product's stages");

static inline int32_t bound_kdense(const ap_index *ix) { return ix->bd_kd ? ix->bd_kd : ix->docs.dim; }

// One block per row of the query matrix: the query's dense part times its weight and its head terms times theirs, rounded to
// bf16, and what the slack of the row is made of.  With x^ for x rounded, part by part (dense, learned-sparse head, lexical
// head),  q d - q^ d^ = (q - q^) d + q^ (d - d^),  so by Cauchy-Schwarz the product is off by at most
//   |q - q^| |d| + |q^| |d - d^|,
// with the norms as they are: rounding to bf16 (8 significant bits) may take 2^-8 off a value, and on a short list or a row of
// like values it does, but over many values it takes about 0.0017 of the norm.  qc[8 r ..]: per part |q^| and the factor of
// |d|, then (6) the relative slack of an addition of the tail.  The factor of |d| is |q - q^| and, times |q|, what everything
// else takes: the product's accumulation (k 2^-23), the rounding of the scoring kernels' own sums and of the tail's additions
// (1e-5 and 2^-22 a term); 1e-18 of the norms for squares and products of values so small that they underflow.  Values so
// large that a partial sum of the scoring kernels may overflow where the product's does not (a query's beyond AP_BOUND_QMAX, a
// part of a document beyond AP_BOUND_DMAX) give a bound of infinity.
__global__ __launch_bounds__(256) void k_bound_queries(ApVecs Q, const float *__restrict__ w, int32_t w_stride, int64_t q0, int64_t nq, int32_t kdense,
                                                       int32_t kh, int32_t nsp, int32_t ntx, const int32_t *__restrict__ col,
                                                       uint16_t *__restrict__ qm, float *__restrict__ qc, uint2 *__restrict__ tails) {
    __shared__ __attribute__((aligned(16))) uint16_t head[AP_BOUND_HEAD];
    __shared__ float red[9][4];
    const int64_t r = blockIdx.x, q = q0 + r;
    uint16_t *row = qm + r * (kdense + kh);
    uint2 *list = tails + r * AP_BOUND_LIST;
    if (r >= nq) {
        if (threadIdx.x <= 8 * AP_BOUND_TERMS) list[threadIdx.x] = threadIdx.x ? make_uint2(AP_BOUND_NONE, 0u) : make_uint2(0u, AP_BOUND_NONE);
        for (int32_t c = threadIdx.x * 8; c < kdense + kh; c += 2048) *reinterpret_cast<uint4 *>(row + c) = make_uint4(0, 0, 0, 0);
        if (threadIdx.x < 8) qc[r * 8 + threadIdx.x] = 0.f;
        return;
    }
    const float wd = w[q * w_stride], ws = w[q * w_stride + 1], wf = w[q * w_stride + 2];
    for (int32_t c = threadIdx.x; c < kh; c += 256) head[c] = 0;
    float sum[9] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};   // per part: squares of the values, of the rounded values, of the differences
    auto add = [&](int part, float x) -> uint32_t {
        const uint32_t y16 = ap_bf16_bits(x);
        const float y = ap_bf16_value(y16), off = x - y;
        sum[3 * part] = fmaf(x, x, sum[3 * part]); sum[3 * part + 1] = fmaf(y, y, sum[3 * part + 1]); sum[3 * part + 2] = fmaf(off, off, sum[3 * part + 2]);
        return y16;
    };
    bool large = false;
    for (int32_t c = threadIdx.x * 4; c < kdense; c += 1024) {
        float x[4] = {0.f, 0.f, 0.f, 0.f};
        if (c < Q.dim) {
            const float4 y = *reinterpret_cast<const float4 *>(static_cast<const float *>(Q.dense) + q * Q.dim + c);
            x[0] = wd * y.x; x[1] = wd * y.y; x[2] = wd * y.z; x[3] = wd * y.w;
            large = large || !(fmaxf(fmaxf(fabsf(y.x), fabsf(y.y)), fmaxf(fabsf(y.z), fabsf(y.w))) <= AP_BOUND_QMAX);
        }
        uint32_t y16[4];
#pragma unroll
        for (int e = 0; e < 4; e++) y16[e] = add(0, x[e]);
        *reinterpret_cast<uint2 *>(row + c) = make_uint2(y16[0] | (y16[1] << 16), y16[2] | (y16[3] << 16));
    }
    __syncthreads();
    int64_t terms = 0;
    uint32_t n_tail = 0, rest = AP_BOUND_NONE;
    for (int part = 0; part < 2; part++) {
        const int64_t b = part ? Q.tx_indptr[q] : Q.sp_indptr[q], e = part ? Q.tx_indptr[q + 1] : Q.sp_indptr[q + 1];
        if (threadIdx.x >= 192) {   // the last wave lists the tail
            const int lane = threadIdx.x & 63;
            for (int64_t p0 = b; p0 < e && rest == AP_BOUND_NONE; p0 += 64) {
                const int32_t t = p0 + lane < e ? (part ? Q.tx_idx : Q.sp_idx)[p0 + lane] : -1;
                const bool in = t >= 0 && t < (part ? ntx : nsp) && col[part ? nsp + t : t] < 0;
                const uint64_t m = __ballot(in);
                const uint32_t at = n_tail + (uint32_t)__popcll(m & ((1ull << lane) - 1ull)), upto = n_tail + (uint32_t)__popcll(m);
                if (upto >= AP_BOUND_LIST) { rest = (uint32_t)(terms + (p0 - b)); break; }   // uniform
                if (in) list[1 + at] = make_uint2((uint32_t)(part ? nsp + t : t), __float_as_uint((part ? wf * Q.tx_val[p0 + lane] : ws * Q.sp_val[p0 + lane])));
                n_tail = upto;
            }
        }
        terms += e - b;
        for (int64_t p = b + threadIdx.x; p < e; p += 256) {
            const int32_t t = part ? Q.tx_idx[p] : Q.sp_idx[p];
            if (t < 0 || t >= (part ? ntx : nsp)) continue;
            const float v = part ? Q.tx_val[p] : Q.sp_val[p];
            large = large || !(fabsf(v) <= AP_BOUND_QMAX);
            const int32_t c = col[part ? nsp + t : t];
            if (c < 0) continue;
            const float x = (part ? wf : ws) * v;
            head[c] = (uint16_t)(part ? add(2, x) : add(1, x));
        }
    }
#pragma unroll
    for (int i = 0; i < 9; i++) {
        sum[i] = ap_wave_sum(sum[i]);
        if ((threadIdx.x & 63) == 0) red[i][threadIdx.x >> 6] = sum[i];
    }
    if (threadIdx.x >= 192) {   // whole batches
        for (uint32_t i = n_tail + (threadIdx.x & 63); i < AP_BOUND_LIST - 1 && (i < 8 * AP_BOUND_TERMS || i < (n_tail + 8 * AP_BOUND_TERMS - 1) / (8 * AP_BOUND_TERMS) * (8 * AP_BOUND_TERMS)); i += 64)
            list[1 + i] = make_uint2(AP_BOUND_NONE, 0u);
        if (threadIdx.x == 192) list[0] = make_uint2(n_tail, rest);
    }
    large = __syncthreads_or(large) != 0;
    for (int32_t c = threadIdx.x * 8; c < kh; c += 2048) *reinterpret_cast<uint4 *>(row + kdense + c) = *reinterpret_cast<const uint4 *>(head + c);
    if (threadIdx.x == 0) {
        float norm[9];
        for (int i = 0; i < 9; i++) norm[i] = sqrtf(red[i][0] + red[i][1] + red[i][2] + red[i][3]) * 1.0001f;
        const float rel = 1e-5f + 2.4e-7f * (float)terms, other = rel + 1.2e-7f * (float)(kdense + kh);
        for (int p = 0; p < 3; p++) {
            qc[r * 8 + 2 * p] = large ? INFINITY : norm[3 * p + 1] + 1e-18f;
            qc[r * 8 + 2 * p + 1] = norm[3 * p + 2] + norm[3 * p] * other + 1e-18f;
        }
        qc[r * 8 + 6] = rel;
        qc[r * 8 + 7] = 0.f;
    }
}

// The tail of one query and one tile's documents, by eight lanes (sub: which of them): what its additions wait for is asked for early, its terms and then
// where their buckets lie, the first entries of all buckets at once.  row: its AP_BOUND_QT entries in LDS, which no other wave touches.
// Long lists make long buckets, of terms that most documents hold above all: the eight lanes read those together, and what the query's list has no place for
// is taken by 32 terms as what it has.  20,000 documents of 1,279 entries, 1,000 queries of 28, 300 and 1,500 terms: 0.56, 4.47 and 33.6 ms by a lane a bucket and a term
// at a time (2^13 buckets), 0.37, 2.25 and 11.7 so (2^15); one block a query through postings by terms, in a kernel of its own, 0.38, 2.54 and 12.0.  With lists of
// several thousand entries, most of them of terms that hardly any document holds, such a kernel would be the faster one (6,000 documents of 6,284
// entries, 1,000 queries of 28 terms 0.24 and 0.44 ms; 4,000 of them 0.96 and 0.93).
struct ApTailJoin {
    const uint32_t *start;
    const uint2 *post;
    int bits, sub;
    uint2 term[AP_BOUND_TERMS], first;
    uint32_t at[AP_BOUND_TERMS], to[AP_BOUND_TERMS];
    __device__ __forceinline__ ApTailJoin(const ApBoundTail &tail, int64_t dt, int sub_)
        : start(tail.start + dt * ((1 << tail.bits) + 1)), post(tail.post + tail.sp_indptr[dt * AP_BOUND_QT] + tail.tx_indptr[dt * AP_BOUND_QT]), bits(tail.bits), sub(sub_) {}
    __device__ __forceinline__ void ask_terms(const uint2 *list, uint32_t from) {
#pragma unroll
        for (int u = 0; u < AP_BOUND_TERMS; u++) term[u] = list[1 + from + sub + 8 * u];
    }
    __device__ __forceinline__ void ask(const uint2 *list) { first = list[0]; ask_terms(list, 0); }
    __device__ __forceinline__ void ask_buckets() {
#pragma unroll
        for (int u = 0; u < AP_BOUND_TERMS; u++) {
            const uint32_t b = ap_bound_bucket(term[u].x, bits);
            at[u] = start[b];
            to[u] = start[b + 1];
            if (term[u].x == AP_BOUND_NONE) to[u] = at[u];
        }
    }
    static __device__ __forceinline__ void add(const uint2 &dv, bool in, uint32_t term, float x, float *row, float rel) {
        if (in && (dv.x >> 8) == term) {
            const float y = __uint_as_float(dv.y), c = x * y;
            ap_lds_add(&row[dv.x & 255u], fabsf(y) <= AP_BOUND_DMAX ? fmaf(fabsf(c), rel, c) : INFINITY);
        }
    }
    // counts a required term's documents among AP_BOUND_AHEAD entries of its bucket
    __device__ __forceinline__ void count(uint32_t k, uint32_t step, uint32_t end, uint32_t want, float *row) {
        uint32_t d[AP_BOUND_AHEAD];
#pragma unroll
        for (int u = 0; u < AP_BOUND_AHEAD; u++)
            if (k + step * u < end) d[u] = post[k + step * u].x;
#pragma unroll
        for (int u = 0; u < AP_BOUND_AHEAD; u++)
            if (k + step * u < end && (d[u] >> 8) == want) atomicAdd(reinterpret_cast<uint32_t *>(row + (d[u] & 255u)), 1u);   // at most 16 required terms: the count stays inside its bits
    }
    __device__ __forceinline__ void add_batch(float *row, float rel) {
        uint2 dv[AP_BOUND_TERMS][AP_BOUND_AHEAD];
#pragma unroll
        for (int u = 0; u < AP_BOUND_TERMS; u++)
#pragma unroll
            for (int j = 0; j < AP_BOUND_AHEAD; j++)
                if (at[u] + j < to[u]) dv[u][j] = post[at[u] + j];
#pragma unroll
        for (int u = 0; u < AP_BOUND_TERMS; u++)
#pragma unroll
            for (int j = 0; j < AP_BOUND_AHEAD; j++) add(dv[u][j], at[u] + j < to[u], term[u].x, __uint_as_float(term[u].y), row, rel);
#pragma unroll
        for (int u = 0; u < AP_BOUND_TERMS; u++) {   // what is left of them one bucket after the other, much by all eight lanes
            uint32_t i = at[u] + AP_BOUND_AHEAD, e = to[u];
            for (uint32_t much = (uint32_t)(__ballot(e > i + AP_BOUND_MUCH) >> (threadIdx.x & 56)) & 255u; much; much &= much - 1) {
                const int l = __ffs(much) - 1;
                const uint32_t b = __shfl(i, l, 8), end = __shfl(e, l, 8), t = __shfl(term[u].x, l, 8);
                const float x = __uint_as_float(__shfl(term[u].y, l, 8));
                for (uint32_t k = b + sub; k < end; k += 8 * AP_BOUND_AHEAD) {
                    uint2 more[AP_BOUND_AHEAD];
#pragma unroll
                    for (int j = 0; j < AP_BOUND_AHEAD; j++) more[j] = post[k + 8 * j < end ? k + 8 * j : k];
#pragma unroll
                    for (int j = 0; j < AP_BOUND_AHEAD; j++) add(more[j], k + 8 * j < end, t, x, row, rel);
                }
                if (sub == l) e = 0;
            }
            for (; i < e; i += AP_BOUND_AHEAD) {
                uint2 more[AP_BOUND_AHEAD];
#pragma unroll
                for (int j = 0; j < AP_BOUND_AHEAD; j++) more[j] = post[i + j];
#pragma unroll
                for (int j = 0; j < AP_BOUND_AHEAD; j++) add(more[j], i + j < e, term[u].x, __uint_as_float(term[u].y), row, rel);
            }
        }
    }
    // everything behind ask_buckets(); then the next row's terms (NULL: there is none) travel with what is left to do
    __device__ __forceinline__ void add_all(const ApBoundTail &tail, const uint2 *list, const uint2 *next, int64_t r, int64_t nq, float *row, float rel) {
        const int64_t q = tail.q0 + r;
        uint32_t from = 8 * AP_BOUND_TERMS;
        int64_t p0 = first.y != AP_BOUND_NONE ? (int64_t)first.y : INT64_MAX;   // the first of the terms that the list had no place for
        for (;;) {   // the eight lanes together
            add_batch(row, rel);
            if (from < first.x) {
                ask_terms(list, from);
                from += 8 * AP_BOUND_TERMS;
            } else if (p0 != INT64_MAX) {
                const int64_t sp0 = tail.q_sp_indptr[q], tx0 = tail.q_tx_indptr[q], sp_n = tail.q_sp_indptr[q + 1] - sp0, all = sp_n + (tail.q_tx_indptr[q + 1] - tx0);
                if (p0 >= all) break;
                const float ws = tail.w[q * tail.w_stride + 1], wf = tail.w[q * tail.w_stride + 2];
#pragma unroll
                for (int u = 0; u < AP_BOUND_TERMS; u++) {
                    const int64_t at = p0 + sub + 8 * u, p = at < all ? at : p0;
                    const bool sp = p < sp_n;
                    const int32_t t = sp ? tail.q_sp_idx[sp0 + p] : tail.q_tx_idx[tx0 + p - sp_n];
                    const float x = sp ? ws * tail.q_sp_val[sp0 + p] : wf * tail.q_tx_val[tx0 + p - sp_n];
                    term[u] = make_uint2(at < all && t >= 0 && t < (sp ? tail.nsp : tail.ntx) ? (uint32_t)(sp ? t : tail.nsp + t) : AP_BOUND_NONE, __float_as_uint(x));
                }
                p0 += 8 * AP_BOUND_TERMS;
            } else break;
            ask_buckets();
        }
        if (next) ask(next);
        ap_wave_sync();
        if (!tail.kw_terms) return;   // uniform
        if (r < nq) for (int j = sub; j < AP_BOUND_QT; j += 8) row[j] = ap_bound_round(row[j], rel);
        ap_wave_sync();
        if (r < nq)
            for (int j0 = 0; j0 < tail.kw_stride; j0 += 8) {   // a lane looks a term up, all eight read a long bucket
                const int32_t t = j0 + sub < tail.kw_stride ? tail.kw_terms[q * tail.kw_stride + j0 + sub] : -1;
                const uint32_t own = (uint32_t)(tail.nsp + t), bucket = ap_bound_bucket(own, bits);
                const bool in = t >= 0 && t < tail.ntx;
                const uint32_t b = in ? start[bucket] : 0u, e = in ? start[bucket + 1] : 0u;
                count(b, 1, e, own, row);
                for (uint32_t more = (uint32_t)(__ballot(e > b + AP_BOUND_AHEAD) >> (threadIdx.x & 56)) & 255u; more; more &= more - 1) {
                    const int l = __ffs(more) - 1;
                    const uint32_t want = __shfl(own, l, 8), end = __shfl(e, l, 8);
                    for (uint32_t k = __shfl(b, l, 8) + AP_BOUND_AHEAD + sub; k < end; k += 8 * AP_BOUND_AHEAD) count(k, 8, end, want, row);
                }
            }
        ap_wave_sync();
    }
    // four entries of a row, as the table holds them
    static __device__ __forceinline__ float4 entries(const float *in, float rel, const ApBoundTail &tail) {
        const float4 v = *reinterpret_cast<const float4 *>(in);
        if (tail.kw_terms) return v;   // rounded before they were counted in
        return make_float4(ap_bound_round(v.x, rel), ap_bound_round(v.y, rel), ap_bound_round(v.z, rel), ap_bound_round(v.w, rel));
    }
};
__device__ __forceinline__ float ap_bound_slack(float2 c0, float2 c1, float2 c2, const float2 (&dn)[3]) {
    float slack = fmaf(c0.x, dn[0].x, 1e-36f);
    slack = fmaf(c0.y, dn[0].y, slack);
    slack = fmaf(c1.x, dn[1].x, slack);
    slack = fmaf(c1.y, dn[1].y, slack);
    slack = fmaf(c2.x, dn[2].x, slack);
    return fmaf(c2.y, dn[2].y, slack);
}
// a document's norms as the slack takes them: |d - d^| and |d|, rounded up
__device__ __forceinline__ float2 ap_bound_dnorm(float2 dn) {
    return make_float2(fmaf(dn.x, 1.0001f, 1e-15f), dn.y <= AP_BOUND_DMAX ? fmaf(dn.y, 1.0001f, 1e-15f) : INFINITY);
}

// The product and the slack: a tile of 256 queries x 256 documents, 16 waves of 64 x 64, chunks of 64 columns through two
// LDS stages as in the seed sweep.  10,000 queries x 100,000 documents x 1,280 columns take 3.1 ms = 0.84 PFLOP/s without the
// tail; the matrix cores and the LDS reads that feed them bound it, as they bound the sweep.  The documents' columns come from two places: the dense part (dense, dense_ld) and
// the head (rows + head_at, rows_ld).
// The tail is added while the tile is in LDS (4.1 ms in all; about one entry in twenty is touched): a kernel of its own that went
// through the queries' postings, one block a query, took 3.3 ms for the read-modify-writes of four fifths of the table's lines.
// What is left of it is the wait for three reads that depend on each other (a query's terms, where their buckets lie, their
// entries), 8 us for half a tile when each was asked for in its turn, 4 as it is.  A lane per document entry would look up five times as
// many terms.  1,000 queries: 707 -> 480 us; 4,000 of some 150 terms, 80,000 documents of 1,024 bf16 columns: 5.5 -> 3.0 ms.
// Tile order: an XCD takes the document tiles in groups of two and walks each group's query tiles, so that a group's
// documents and the queries stay in its L2 while they are used.  Groups of four leave some XCDs a group more than others: 4,000 queries of 20,000 documents
// (79 tiles) 425 us, 367 by two, 359 by one; 10,000 of 100,000 4.1 ms, 3.9 and 4.2.  By how many tiles the longest XCD's share grows: by four at most three more than by one,
// by two at most one, a tenth of the share at 79 tiles and a fiftieth at 391, where the reuse of the queries' columns is worth eight hundredths.
#define AP_BOUND_GROUP 2
__global__ __launch_bounds__(1024) void k_bound_table(const uint16_t *__restrict__ qm, const float *__restrict__ qc, int32_t nq, int32_t q_tiles,
                                                      const uint16_t *__restrict__ dense, int32_t dense_ld, int32_t n_dense,
                                                      const uint16_t *__restrict__ head, int32_t head_ld, int32_t n_chunks,
                                                      const float2 *__restrict__ norms, int64_t n, int64_t doc_tiles, ApBoundTail tail,
                                                      float *__restrict__ table, int64_t ld) {
    extern __shared__ __attribute__((aligned(16))) uint16_t bound_lds[];
    __shared__ float2 s_qc[3][AP_BOUND_QT], s_dn[3][AP_BOUND_QT];   // per part: |q^| and the factor of |d|; |d - d^| and |d|
    using T = ApBig<4, 4>;
    constexpr int NP = T::NP, RPP = T::RPP;
    const int64_t xcd = blockIdx.x % 8, idx = blockIdx.x / 8;
    const int64_t group = idx / (AP_BOUND_GROUP * q_tiles), in = idx % (AP_BOUND_GROUP * q_tiles);
    const int64_t dt = (group * 8 + xcd) * AP_BOUND_GROUP + in % AP_BOUND_GROUP, qt = in / AP_BOUND_GROUP;
    if (dt >= doc_tiles) return;   // uniform
    const int64_t d0 = dt * AP_BOUND_QT, r0 = qt * AP_BOUND_QT;
    const int t = threadIdx.x, lane = t & 63, wave = ap_wave_id(), wm = wave >> 2, wn = wave & 3;
    if (t < 3 * AP_BOUND_QT) {
        const int p = t / AP_BOUND_QT, j = t % AP_BOUND_QT;
        const float2 dn = norms[p * n + (d0 + j < n ? d0 + j : n - 1)];
        s_qc[p][j] = *reinterpret_cast<const float2 *>(qc + (r0 + j) * 8 + 2 * p);
        s_dn[p][j] = ap_bound_dnorm(dn);
    }
    const int32_t kq = n_chunks * AP_BK16;
    const char *qa = reinterpret_cast<const char *>(qm + r0 * kq);
    const char *da = reinterpret_cast<const char *>(dense + d0 * dense_ld), *ha = reinterpret_cast<const char *>(head + d0 * head_ld);
    uint32_t qo[NP], dd[NP], ho[NP];
#pragma unroll
    for (int p = 0; p < NP; p++) {
        const int32_t row = t / AP_TPR16 + RPP * p;
        const int32_t drow = d0 + row < n ? row : (int32_t)(n - 1 - d0);   // past the end: the last document again, not stored
        const uint32_t c = (uint32_t)(t % AP_TPR16) * 16u;
        qo[p] = (uint32_t)row * (uint32_t)kq * 2u + c;
        dd[p] = (uint32_t)drow * (uint32_t)dense_ld * 2u + c;
        ho[p] = (uint32_t)drow * (uint32_t)head_ld * 2u + c;
    }
    auto load = [&](int32_t k, ap_u32x4 (&va)[NP], ap_u32x4 (&vb)[NP]) {
#pragma unroll
        for (int p = 0; p < NP; p++) va[p] = *reinterpret_cast<const ap_u32x4 *>(qa + (qo[p] + (uint32_t)k * 128u));
        if (k < n_dense) {
#pragma unroll
            for (int p = 0; p < NP; p++) vb[p] = *reinterpret_cast<const ap_u32x4 *>(da + (dd[p] + (uint32_t)k * 128u));
        } else {
#pragma unroll
            for (int p = 0; p < NP; p++) vb[p] = *reinterpret_cast<const ap_u32x4 *>(ha + (ho[p] + (uint32_t)(k - n_dense) * 128u));
        }
    };
    auto store = [&](const ap_u32x4 (&va)[NP], const ap_u32x4 (&vb)[NP], uint16_t *to) {
        ap_big_store_run<NP, RPP>(va, to);
        ap_big_store_run<NP, RPP>(vb, to + AP_BIG * AP_LDS_STRIDE16);
    };
    ap_f32x16 acc[2][2];
#pragma unroll
    for (int a = 0; a < 2; a++)
#pragma unroll
        for (int b = 0; b < 2; b++)
#pragma unroll
            for (int r = 0; r < 16; r++) acc[a][b][r] = 0.f;
    ap_u32x4 va0[NP], vb0[NP], va1[NP], vb1[NP];
    load(0, va0, vb0);
    store(va0, vb0, bound_lds);
    if (n_chunks > 1) load(1, va0, vb0);
    if (n_chunks > 2) load(2, va1, vb1);
    __syncthreads();
    const int li = lane & 31, lk = (lane >> 5) * 8;
    // round k: chunk k is multiplied out of stage k & 1; set k & 1 holds chunk k + 1, which goes to the other stage, and is
    // filled with chunk k + 3
    auto round = [&](int32_t k, ap_u32x4 (&sa)[NP], ap_u32x4 (&sb)[NP]) {
        uint16_t *cur = bound_lds + (k & 1) * AP_BIG_STAGE, *nxt = bound_lds + ((k + 1) & 1) * AP_BIG_STAGE;
        if (k + 1 < n_chunks) store(sa, sb, nxt);
        if (k + 3 < n_chunks) load(k + 3, sa, sb);
        const uint16_t *pa = cur + (wm * 64 + li) * AP_LDS_STRIDE16 + lk, *pb = cur + AP_BIG * AP_LDS_STRIDE16 + (wn * 64 + li) * AP_LDS_STRIDE16 + lk;
#pragma unroll
        for (int kk = 0; kk < AP_BK16; kk += 16) {
            ap_bf16x8 fa[2], fb[2];
#pragma unroll
            for (int a = 0; a < 2; a++) {
                fa[a] = __builtin_bit_cast(ap_bf16x8, *reinterpret_cast<const ap_u32x4 *>(pa + a * 32 * AP_LDS_STRIDE16 + kk));
                fb[a] = __builtin_bit_cast(ap_bf16x8, *reinterpret_cast<const ap_u32x4 *>(pb + a * 32 * AP_LDS_STRIDE16 + kk));
            }
#pragma unroll
            for (int a = 0; a < 2; a++)
#pragma unroll
                for (int b = 0; b < 2; b++) acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[a], fb[b], acc[a][b], 0, 0, 0);
        }
        __syncthreads();
    };
    for (int32_t k = 0; k < n_chunks; k += 2) {
        round(k, va0, vb0);
        if (k + 1 < n_chunks) round(k + 1, va1, vb1);
    }
    // The tile goes to LDS by halves, where the tail is added, and from there to memory.  Half a holds the queries of every
    // wave's accumulators a: place p of its 128 is query (p >> 5) * 64 + a * 32 + (p & 31).  Eight lanes take a query, a wave
    // the same eight queries from the first addition to the last store: only the way into LDS needs barriers.
    __builtin_amdgcn_sched_barrier(0);   // what follows, begun earlier, takes registers that the loop has not got: it would spill them in every round
    float *tile = reinterpret_cast<float *>(bound_lds);
    const int own = wave * 8 + (lane >> 3);
    const int64_t r_own = r0 + (own >> 5) * 64 + (own & 31);   // and 32 more in the second half
    const uint2 *lists = tail.lists + r_own * AP_BOUND_LIST;
    ApTailJoin join(tail, dt, lane & 7);
    join.ask(lists);
#pragma unroll
    for (int a = 0; a < 2; a++) {
        if (a) __syncthreads();
        float2 dn[2][3];
#pragma unroll
        for (int b = 0; b < 2; b++)
#pragma unroll
            for (int p = 0; p < 3; p++) dn[b][p] = s_dn[p][wn * 64 + b * 32 + li];
#pragma unroll
        for (int r = 0; r < 16; r++) {
            const int in = 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3), i = wm * 64 + a * 32 + in;
            const float2 c0 = s_qc[0][i], c1 = s_qc[1][i], c2 = s_qc[2][i];
#pragma unroll
            for (int b = 0; b < 2; b++) tile[(wm * 32 + in) * AP_BOUND_QT + wn * 64 + b * 32 + li] = acc[a][b][r] + ap_bound_slack(c0, c1, c2, dn[b]);
        }
        join.ask_buckets();
        __syncthreads();
        const int64_t r = r_own + 32 * a;
        const float rel = qc[r * 8 + 6];
        join.add_all(tail, lists + 32 * a * AP_BOUND_LIST, a == 0 ? lists + 32 * AP_BOUND_LIST : nullptr, r, nq, tile + own * AP_BOUND_QT, rel);
        const int64_t j = d0 + lane * 4;
#pragma unroll
        for (int i = 0; i < 8; i++) {
            const int at = wave * 8 + i;
            const int64_t to = r0 + (at >> 5) * 64 + a * 32 + (at & 31);
            const float f = __shfl(rel, i * 8, 64);
            if (to < nq && j < ld) *reinterpret_cast<float4 *>(table + to * ld + j) = ApTailJoin::entries(tile + at * AP_BOUND_QT + lane * 4, f, tail);
        }
    }
}

// The same for few queries, which the reading of the documents' columns bounds: A x 32 of them, every one's columns in turn out of LDS (two chunks of
// 64 a stage), a wave 32 documents, whose columns go straight to the matrix unit: a lane reads 64 consecutive bytes of a chunk, half a line, so
// that the instruction's eight columns are other ones than in the tile above, the same on both sides.  Two chunks are on their way while two are multiplied.
// 8 waves share 256 documents and their postings.  One query of 100,000 documents of 1,280 columns: 156 us by the tile of 256 queries, 54 so
// (4.7 TB/s); 37 of 120,011 of 1,536: 175 and 104.  64 queries, the whole of an exact top-k: 219 and 183 us of 100,000 documents of 1,280 columns, 235 and 196 of 120,011
// of 1,536, 129 and 110 of 20,000 of 1,280, 91 and 84 of 5,000 of 640; from 65 on the tile takes less than two passes.
#define AP_BOUND_FEW_STRIDE (256 + 16)   // bytes of a query's two chunks in LDS
template <int A>
__global__ __launch_bounds__(512, 4) void k_bound_few(const uint16_t *__restrict__ qm, const float *__restrict__ qc, int32_t nq, const uint16_t *__restrict__ dense,
                                                      int32_t dense_ld, int32_t n_dense, const uint16_t *__restrict__ head, int32_t head_ld, int32_t n_chunks,
                                                      const float2 *__restrict__ norms, int64_t n, ApBoundTail tail, float *__restrict__ table, int64_t ld) {
    constexpr int ROWS = 32 * A, STAGE = ROWS * AP_BOUND_FEW_STRIDE;
    static_assert(2 * STAGE <= ROWS * AP_BOUND_QT * 4, "the tile takes the place of the stages");
    __shared__ __attribute__((aligned(16))) unsigned char few_lds[ROWS * AP_BOUND_QT * 4];
    __shared__ float2 s_qc[3][ROWS];
    const int t = threadIdx.x, lane = t & 63, wave = ap_wave_id(), li = lane & 31, half = lane >> 5;
    const int64_t dt = blockIdx.x, d0 = dt * AP_BOUND_QT, d = d0 + wave * 32 + li < n ? d0 + wave * 32 + li : n - 1;
    if (t < 3 * ROWS) s_qc[t / ROWS][t % ROWS] = *reinterpret_cast<const float2 *>(qc + (t % ROWS) * 8 + 2 * (t / ROWS));
    float2 dn[3];
#pragma unroll
    for (int p = 0; p < 3; p++) dn[p] = ap_bound_dnorm(norms[p * n + d]);
    const char *drow = reinterpret_cast<const char *>(dense + d * dense_ld) + 64 * half, *hrow = reinterpret_cast<const char *>(head + d * head_ld) + 64 * half;
    const int32_t kq = n_chunks * AP_BK16;
    ap_u32x4 b0[2][4], b1[2][4], va[A];
    auto load_docs = [&](int32_t k, ap_u32x4 (&to)[2][4]) {
#pragma unroll
        for (int c = 0; c < 2; c++) {
            const int32_t kc = k + c < n_chunks ? k + c : k;   // uniform
            const char *from = kc < n_dense ? drow + (int64_t)kc * 128 : hrow + (int64_t)(kc - n_dense) * 128;
#pragma unroll
            for (int s = 0; s < 4; s++) to[c][s] = *reinterpret_cast<const ap_u32x4 *>(from + 16 * s);
        }
    };
    // the queries' two chunks: 16 threads a row, 32 rows at a time
    auto load_queries = [&](int32_t k) {
        const int32_t at = (t & 15) * 8, col = k * AP_BK16 + at;
#pragma unroll
        for (int p = 0; p < A; p++) va[p] = *reinterpret_cast<const ap_u32x4 *>(qm + (int64_t)(32 * p + (t >> 4)) * kq + (col < kq ? col : at));
    };
    auto store_queries = [&](unsigned char *to) {
#pragma unroll
        for (int p = 0; p < A; p++) *reinterpret_cast<ap_u32x4 *>(to + (32 * p + (t >> 4)) * AP_BOUND_FEW_STRIDE + (t & 15) * 16) = va[p];
    };
    ap_f32x16 acc[A];
#pragma unroll
    for (int a = 0; a < A; a++)
#pragma unroll
        for (int r = 0; r < 16; r++) acc[a][r] = 0.f;
    load_queries(0);
    load_docs(0, b0);
    store_queries(few_lds);
    if (n_chunks > 2) load_queries(2);
    __syncthreads();
    // round k: chunks k and k + 1 are multiplied out of stage (k / 2) & 1 while k + 2 and k + 3 travel; the queries' are there already
    auto round = [&](int32_t k, const ap_u32x4 (&b)[2][4], ap_u32x4 (&next)[2][4]) {
        const unsigned char *cur = few_lds + ((k >> 1) & 1) * STAGE;
        if (k + 2 < n_chunks) {
            load_docs(k + 2, next);
            store_queries(few_lds + (((k >> 1) + 1) & 1) * STAGE);
            if (k + 4 < n_chunks) load_queries(k + 4);
        }
#pragma unroll
        for (int c = 0; c < 2; c++) {
            if (k + c >= n_chunks) break;   // uniform
#pragma unroll
            for (int s = 0; s < 4; s++)
#pragma unroll
                for (int a = 0; a < A; a++) {
                    const ap_u32x4 q = *reinterpret_cast<const ap_u32x4 *>(cur + (32 * a + li) * AP_BOUND_FEW_STRIDE + c * 128 + 64 * half + 16 * s);
                    acc[a] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(ap_bf16x8, q), __builtin_bit_cast(ap_bf16x8, b[c][s]), acc[a], 0, 0, 0);
                }
        }
        __syncthreads();
    };
    for (int32_t k = 0; k < n_chunks; k += 4) {
        round(k, b0, b1);
        if (k + 2 < n_chunks) round(k + 2, b1, b0);
    }
    // the first 4 A waves take eight queries each, as above
    float *tile = reinterpret_cast<float *>(few_lds);
    const int own = wave * 8 + (lane >> 3);
    ApTailJoin join(tail, dt, lane & 7);
    const uint2 *list = tail.lists + (int64_t)own * AP_BOUND_LIST;
    if (wave < 4 * A) join.ask(list);
#pragma unroll
    for (int a = 0; a < A; a++)
#pragma unroll
        for (int r = 0; r < 16; r++) {
            const int i = 32 * a + 8 * (r >> 2) + 4 * half + (r & 3);
            tile[i * AP_BOUND_QT + wave * 32 + li] = acc[a][r] + ap_bound_slack(s_qc[0][i], s_qc[1][i], s_qc[2][i], dn);
        }
    if (wave < 4 * A) join.ask_buckets();
    __syncthreads();
    if (wave >= 4 * A) return;
    const float rel = qc[own * 8 + 6];
    join.add_all(tail, list, nullptr, own, nq, tile + own * AP_BOUND_QT, rel);
    const int64_t j = d0 + lane * 4;
#pragma unroll
    for (int i = 0; i < 8; i++) {
        const int at = wave * 8 + i;
        const float f = __shfl(rel, i * 8, 64);
        if (at < nq && j < ld) *reinterpret_cast<float4 *>(table + at * ld + j) = ApTailJoin::entries(tile + at * AP_BOUND_QT + lane * 4, f, tail);
    }
}

// One block per query: the bounds that shares of the documents reach, from a sample of at most 4,096 (64 runs spread over the
// corpus, 256 bytes each), and a word of two bitmaps per 32 documents: which of them a search has met (none yet), and, in the upper half, which have a
// bound that reaches the first of those floors.  The floors are the lower edges of the bins that the sample's values at the given ranks lie in
// (22 bits of their codes).  Bound by the reading of the table: 4,000 queries of 100,000 documents take 0.56 ms, of which a sort of the
// sample for one floor alone took 0.47; the search reads a bit where it read an entry, a line of memory each.
#define AP_FLOOR_SAMPLE 4096
__global__ __launch_bounds__(1024) void k_bound_floor(const float *__restrict__ table, int64_t ld, int64_t n, float4 share, float4 *__restrict__ out,
                                                      uint64_t *__restrict__ marks, int64_t words) {
    __shared__ uint32_t hist[3][2048];
    __shared__ uint32_t s_bin[3], s_left[3];
    const int lane = threadIdx.x & 63, wave = ap_wave_id();
    const float *row = table + (int64_t)blockIdx.x * ld;
    const int32_t m = n < AP_FLOOR_SAMPLE ? (int32_t)n : AP_FLOOR_SAMPLE;
    const float shares[3] = {share.x, share.y, share.z};
    uint32_t code[AP_FLOOR_SAMPLE / 1024];
#pragma unroll
    for (int j = 0; j < AP_FLOOR_SAMPLE / 1024; j++) {
        const int32_t i = (int32_t)threadIdx.x + 1024 * j;
        const int64_t d = n <= AP_FLOOR_SAMPLE ? i : (i >> 6) * ((n - 64) / 63) + (i & 63);
        float x = i < m ? row[d] : -INFINITY;
        if (!(x < INFINITY)) x = -INFINITY;   // says nothing about the scores
        code[j] = i < m ? ap_f2ord(x) : 0xffffffffu;
    }
    // wave w < 3: the bin of the entry that `rank` others of hist[w] lie above, and how many of the bin's own do
    auto find = [&](const uint32_t *h, uint32_t rank) {
        uint32_t sum = 0;
        for (int j = 0; j < 32; j++) sum += h[2016 - 32 * lane + ((j + lane) & 31)];   // from the top: lane 0 has the last 32 bins
        uint32_t upto = sum;
        for (int o = 1; o < 64; o <<= 1) { const uint32_t up = (uint32_t)__shfl_up((int)upto, o, 64); if (lane >= o) upto += up; }
        if (upto > rank && upto - sum <= rank) {   // at most one lane
            uint32_t above = upto - sum;
            int b = 2047 - 32 * lane;
            while (above + h[b] <= rank) above += h[b--];
            s_bin[wave] = (uint32_t)b; s_left[wave] = rank - above;
        }
    };
    for (int i = threadIdx.x; i < 3 * 2048; i += 1024) (&hist[0][0])[i] = 0;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < AP_FLOOR_SAMPLE / 1024; j++)
        if (code[j] != 0xffffffffu) atomicAdd(&hist[0][code[j] >> 21], 1u);
    __syncthreads();
    const int32_t rank = (int32_t)(shares[wave < 3 ? wave : 0] * (float)m);
    const bool asked = wave < 3 && rank < m;   // uniform
    if (asked) find(hist[0], (uint32_t)rank);
    __syncthreads();
    uint32_t top[3];
#pragma unroll
    for (int p = 0; p < 3; p++) top[p] = s_bin[p];
    for (int i = threadIdx.x; i < 3 * 2048; i += 1024) (&hist[0][0])[i] = 0;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < AP_FLOOR_SAMPLE / 1024; j++)
#pragma unroll
        for (int p = 0; p < 3; p++)
            if (code[j] != 0xffffffffu && (code[j] >> 21) == top[p]) atomicAdd(&hist[p][(code[j] >> 10) & 2047u], 1u);
    __syncthreads();
    if (asked) find(hist[wave], s_left[wave]);
    __syncthreads();
    float floors[3];
#pragma unroll
    for (int p = 0; p < 3; p++) floors[p] = (int32_t)(shares[p] * (float)m) < m ? fmaxf(ap_ord2f((top[p] << 21) | (s_bin[p] << 10)), -INFINITY) : -INFINITY;   // below the code of -inf lie those of NaNs
    if (threadIdx.x == 0) out[blockIdx.x] = make_float4(floors[0], floors[1], floors[2], 0.f);
    uint64_t *mark = marks + (int64_t)blockIdx.x * words;
    for (int64_t d0 = (int64_t)wave * 512; d0 < n; d0 += 16 * 512) {
        float x[8];
#pragma unroll
        for (int j = 0; j < 8; j++) x[j] = d0 + 64 * j + lane < n ? row[d0 + 64 * j + lane] : -INFINITY;
        uint32_t mine = 0;
#pragma unroll
        for (int j = 0; j < 8; j++) {
            const uint64_t b = __ballot(!(ap_bound_value(x[j]) < floors[0]));   // a NaN reaches any floor
            if ((lane >> 1) == j) mine = (uint32_t)(b >> (32 * (lane & 1)));
        }
        if (lane < 16 && (d0 >> 5) + lane < words) mark[(d0 >> 5) + lane] = (uint64_t)mine << 32;
    }
}

// The floors of the slab's queries for a pool of `beam` entries: as if the documents a search meets were drawn at random,
// with a quarter of the pool on top; they are better than that, so the pool's last score usually ends above it.  The lower ones, which four and sixteen
// times as many documents reach, serve the first iterations.
double ap_bound_floor_share(const ap_index *ix, int32_t beam) {
    const double n = (double)ix->docs.n, met = n * (1.0 - exp(-(double)beam * ix->params.degree / n));
    return g_ap_debug.search_floor == 2 ? 0.002 : std::min(1.0, 1.25 * beam / met);
}
int ap_bound_floors(const ap_index *ix, const ApBound &b, int64_t nq, int32_t beam, hipStream_t st) {
    const float share = (float)ap_bound_floor_share(ix, beam);
    hipLaunchKernelGGL(k_bound_floor, dim3((unsigned)nq), dim3(1024), 0, st, b.table, b.ld, ix->docs.n, make_float4(share, 4.f * share, 16.f * share, 0.f),
                       reinterpret_cast<float4 *>(b.floor), b.marks, (ix->docs.n + 31) / 32);
    AP_CHECK_HIP(hipGetLastError());
    return AP_OK;
}

// Bytes of the workspace a slab of nq queries takes, with one table of n entries a query or two (AP_BOUND_MARKS: one, and the words of
// the two bitmaps beside it).
size_t ap_bound_bytes(const ap_index *ix, int64_t nq, int tables) {
    const size_t rows = ap_up((size_t)nq, AP_BOUND_QT), k = (size_t)(bound_kdense(ix) + ix->bd_kh), n = (size_t)ix->docs.n;
    return rows * k * 2 + rows * 32 + rows * 20 + ap_up(rows * AP_BOUND_LIST * 8, 256) + (size_t)nq * (tables == AP_BOUND_MARKS ? ap_up(n, 64) * 4 + (n + 31) / 32 * 8 : (size_t)tables * ap_up(n, 64) * 4);
}

void ap_bound_place(const ap_index *ix, void *base, int64_t nq, int tables, ApBound *b) {
    const size_t rows = ap_up((size_t)nq, AP_BOUND_QT), k = (size_t)(bound_kdense(ix) + ix->bd_kh);
    char *m = static_cast<char *>(base);
    b->qm = reinterpret_cast<uint16_t *>(m); m += rows * k * 2;
    b->qc = reinterpret_cast<float *>(m); m += rows * 32;
    b->floor = reinterpret_cast<float *>(m); m += rows * 20;
    b->tails = reinterpret_cast<uint2 *>(m); m += ap_up(rows * AP_BOUND_LIST * 8, 256);
    b->table = reinterpret_cast<float *>(m);
    b->ld = (int64_t)ap_up((size_t)ix->docs.n, 64);
    float *behind = b->table + (size_t)nq * (size_t)b->ld;
    b->second = tables == 2 ? behind : nullptr;
    b->marks = tables == AP_BOUND_MARKS ? reinterpret_cast<uint64_t *>(behind) : nullptr;
    b->slab = (int32_t)nq;
}

void ap_bound_release(ap_index *ix) {
    if (!ix->bd_pool) return;
    for (int i = 0; i < ix->bd_pool->used; i++) {
        if (ix->bd_pool->ws[i].mem) (void)hipFree(ix->bd_pool->ws[i].mem);
        (void)hipEventDestroy(ix->bd_pool->ws[i].done);
    }
    delete ix->bd_pool;
    ix->bd_pool = nullptr;
}

// Queries per slab when a slab may take `cap` bytes (0: not even one).
static int64_t bound_slab(const ap_index *ix, int64_t nq, size_t cap, int tables) {
    int64_t slabs = 1;
    while (slabs < nq && ap_bound_bytes(ix, (nq + slabs - 1) / slabs, tables) > cap) slabs++;
    const int64_t slab = (nq + slabs - 1) / slabs;
    return ap_bound_bytes(ix, slab, tables) <= cap ? slab : 0;
}

// Sizes the workspace of stream st for slabs of as many of nq queries as `cap` bytes hold, and holds it for the caller
// (two threads may search on one stream).  A workspace that has to grow takes a quarter of the free memory at most, and
// smaller slabs then, but of `least` queries at least (fewer than a launch keeps in flight cost more than the bounds save).
// `cap` may ask for slabs smaller than that, unless `least` is AP_BOUND_WHOLE: then it is all nq queries in one slab or no bounds.
// b->table stays NULL where no such workspace is to be had: the caller goes without bounds.  That is also what a captured
// search does: a graph's replays must not depend on a workspace that a later call may replace.
int ap_bound_reserve(const ap_index *ix, int64_t nq, int64_t least, size_t cap, int tables, hipStream_t st, ApBound *b) {
    if (!ix->bd_mem || nq < 1 || st == hipStreamPerThread) return AP_OK;
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &cs) != hipSuccess) { (void)hipGetLastError(); return AP_OK; }
    if (cs != hipStreamCaptureStatusNone) return AP_OK;
    if (g_ap_debug.search_bounds_bytes > 0) cap = std::min(cap, (size_t)g_ap_debug.search_bounds_bytes);
    int64_t slab = bound_slab(ix, nq, cap, tables);
    if (slab == 0 || (least == AP_BOUND_WHOLE && slab < nq)) return AP_OK;
    least = std::min(least, slab);
    ApBoundPool *pool = ix->bd_pool;
    std::unique_lock<std::mutex> hold(pool->lock);
    int i = 0;
    while (i < pool->used && pool->ws[i].stream != st) i++;
    if (i == pool->used && i < AP_BOUND_STREAMS) {
        hipEvent_t done = nullptr;
        if (hipEventCreateWithFlags(&done, hipEventDisableTiming) != hipSuccess) { (void)hipGetLastError(); return AP_OK; }
        pool->ws[i] = {st, nullptr, 0, done, 0};
        pool->used++;
    } else if (i == pool->used) {   // a stream beyond the workspaces
        for (int j = 0; j < pool->used; j++)
            if ((i == pool->used || pool->ws[j].last < pool->ws[i].last) && hipEventQuery(pool->ws[j].done) == hipSuccess) i = j;
        (void)hipGetLastError();   // "not ready" is no error
        if (i == pool->used) return AP_OK;
        pool->ws[i].stream = st;
    } else {
        // work of the same stream comes behind its last use anyway, but the handle of a stream that is gone may name another now
        AP_CHECK_HIP(hipStreamWaitEvent(st, pool->ws[i].done, 0));
    }
    auto &w = pool->ws[i];
    w.last = ++pool->uses;
    if (ap_bound_bytes(ix, slab, tables) > w.bytes) {
        size_t free_b = 0, total_b = 0;
        if (hipMemGetInfo(&free_b, &total_b) != hipSuccess) { (void)hipGetLastError(); free_b = 0; }
        slab = bound_slab(ix, nq, std::min(cap, std::max(w.bytes, (free_b + w.bytes) / 4)), tables);
    }
    if (slab < least) return AP_OK;
    if (const size_t need = ap_bound_bytes(ix, slab, tables); need > w.bytes) {
        void *mem = nullptr;
        if (hipMalloc(&mem, need) == hipSuccess) {
            const hipError_t e = w.mem ? hipStreamSynchronize(st) : hipSuccess;
            if (w.mem) (void)hipFree(w.mem);
            w.mem = mem;
            w.bytes = need;
            AP_CHECK_HIP(e);
        } else {   // what is there goes on serving
            (void)hipGetLastError();
            slab = bound_slab(ix, nq, std::min(cap, w.bytes), tables);
            if (slab < least) return AP_OK;
        }
    }
    ap_bound_place(ix, w.mem, slab, tables, b);
    b->hold = std::move(hold);
    b->stream = st;
    b->done = w.done;
    return AP_OK;
}

// Bytes of the workspace that stream st has, and its return to the device once a call that is not made again and again is
// over (the stream has been waited for).
size_t ap_bound_held(const ap_index *ix, hipStream_t st) {
    if (!ix->bd_pool) return 0;
    std::lock_guard<std::mutex> hold(ix->bd_pool->lock);
    for (int i = 0; i < ix->bd_pool->used; i++)
        if (ix->bd_pool->ws[i].stream == st) return ix->bd_pool->ws[i].bytes;
    return 0;
}
// The same memory as scratch for what comes behind the search on its stream, where nothing else searches the index (an insertion's new one).
ApWork ap_bound_borrow(const ap_index *ix, hipStream_t st) {
    ApWork w;
    if (!ix->bd_pool) return w;
    std::lock_guard<std::mutex> hold(ix->bd_pool->lock);
    for (int i = 0; i < ix->bd_pool->used; i++)
        if (ix->bd_pool->ws[i].stream == st && ix->bd_pool->ws[i].mem) { w.mem = ix->bd_pool->ws[i].mem; w.bytes = ix->bd_pool->ws[i].bytes; }
    return w;
}
void ap_bound_give_back(const ap_index *ix, hipStream_t st) {
    if (!ix->bd_pool) return;
    std::lock_guard<std::mutex> hold(ix->bd_pool->lock);
    for (int i = 0; i < ix->bd_pool->used; i++) {
        auto &w = ix->bd_pool->ws[i];
        if (w.stream != st || !w.mem) continue;
        (void)hipFree(w.mem);
        w.mem = nullptr;
        w.bytes = 0;
    }
}

// Fills rows 0 .. nq of the table for queries q0 .. q0 + nq of Q (nq <= b.slab).
int ap_bound_fill(const ap_index *ix, const ApBound &b, const ApVecs &Q, const float *w, int32_t w_stride, int64_t q0, int64_t nq,
                  const int32_t *kw_terms, int32_t kw_stride, hipStream_t st) {
    const int32_t kdense = bound_kdense(ix), kh = ix->bd_kh, nsp = ix->corpus.sp_vocab, ntx = ix->corpus.tx_vocab;
    const int64_t n = ix->docs.n, q_tiles = (nq + AP_BOUND_QT - 1) / AP_BOUND_QT, doc_tiles = (n + AP_BOUND_QT - 1) / AP_BOUND_QT;
    const int64_t groups = (doc_tiles + 8 * AP_BOUND_GROUP - 1) / (8 * AP_BOUND_GROUP);
    const bool own = ix->bd_kd != 0;
    hipLaunchKernelGGL(k_bound_queries, dim3((unsigned)(q_tiles * AP_BOUND_QT)), dim3(256), 0, st, Q, w, w_stride, q0, nq, kdense, kh, nsp, ntx, ix->bd_col, b.qm,
                       b.qc, b.tails);
    const int32_t ld = ix->bd_kd + kh;
    const ApBoundTail tail{w, w_stride, nsp, ntx, ix->bd_start_bits, kw_terms ? kw_stride : 0, q0, Q.sp_indptr, Q.tx_indptr, Q.sp_idx, Q.tx_idx, Q.sp_val, Q.tx_val,
                           ix->docs.sp_indptr, ix->docs.tx_indptr, b.tails, ix->bd_start, ix->bd_post, kw_terms};
    const uint16_t *rows = own ? ix->bd_rows : static_cast<const uint16_t *>(ix->docs.dense), *heads = ix->bd_rows + ix->bd_kd;
    const int32_t rows_ld = own ? ld : ix->docs.dim, n_dense = kdense / AP_BK16, n_chunks = (kdense + kh) / AP_BK16;
    if (nq <= AP_BOUND_FEW) {   // one pass over the documents' columns either way
        if (nq <= 32)
            hipLaunchKernelGGL(k_bound_few<1>, dim3((unsigned)doc_tiles), dim3(512), 0, st, b.qm, b.qc, (int32_t)nq, rows, rows_ld, n_dense, heads, ld, n_chunks, ix->bd_norms, n, tail,
                               b.table, b.ld);
        else
            hipLaunchKernelGGL(k_bound_few<2>, dim3((unsigned)doc_tiles), dim3(512), 0, st, b.qm, b.qc, (int32_t)nq, rows, rows_ld, n_dense, heads, ld, n_chunks, ix->bd_norms, n, tail,
                               b.table, b.ld);
        AP_CHECK_HIP(hipGetLastError());
        return AP_OK;
    }
    AP_CHECK_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(&k_bound_table), hipFuncAttributeMaxDynamicSharedMemorySize, AP_BIG_LDS_BYTES));
    hipLaunchKernelGGL(k_bound_table, dim3((unsigned)(groups * 8 * AP_BOUND_GROUP * q_tiles)), dim3(1024), AP_BIG_LDS_BYTES, st, b.qm, b.qc, (int32_t)nq,
                       (int32_t)q_tiles, rows, rows_ld, n_dense, heads, ld, n_chunks, ix->bd_norms, n, doc_tiles, tail, b.table, b.ld);
    AP_CHECK_HIP(hipGetLastError());
    return AP_OK;
}

// The table itself, for tests: rows of the nq queries' bounds, n entries each.
extern "C" int ap_stage_score_bounds(ap_index *ix, const ap_queries *q, const float *per_query_w, const int32_t *kw_terms, int32_t kw_stride,
                                     float *out, void *stream) {
    AP_REQUIRE(ix && out, "NULL argument");
    AP_TRY(ap_validate_queries(q));
    AP_REQUIRE(!kw_terms || (kw_stride >= 1 && kw_stride <= 16), "kw_stride = %d must be in [1, 16]", kw_stride);
    if (q->nq == 0) return AP_OK;
    hipStream_t st = (hipStream_t)stream;
    const ApVecs Q{q->nq, ix->docs.dim, q->dense, q->sp_indptr, q->sp_idx, q->sp_val, q->tx_indptr, q->tx_idx, q->tx_cnt};
    ApBound b;
    AP_TRY(ap_bound_reserve(ix, q->nq, AP_BOUND_WHOLE, AP_BOUND_WS_BYTES, 1, st, &b));
    if (!b.table) { ap_set_error("no bounds for this index and batch"); return AP_ESTATE; }
    AP_TRY(ap_bound_fill(ix, b, Q, per_query_w ? per_query_w : ix->w_dev, per_query_w ? 3 : 0, 0, q->nq, kw_terms, kw_stride, st));
    AP_CHECK_HIP(hipMemcpy2DAsync(out, (size_t)ix->docs.n * 4, b.table, (size_t)b.ld * 4, (size_t)ix->docs.n * 4, (size_t)q->nq, hipMemcpyDeviceToDevice, st));
    return AP_OK;
}
