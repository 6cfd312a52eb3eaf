// Index construction (Algorithm 1, Steps 1-3 of Section 4.1): seed lists by an
// MFMA dense product with exact top-K selection, synchronous refinement rounds
// under the hybrid metric, detourable-route sort, inner-product pruning with
// keyword recycling, and assembly of the fixed-degree edge lists.
// Every stage is a pure function of the previous stage's arrays; nothing that
// decides an id depends on the order in which atomics arrive.
#include <stdlib.h>
#include <string.h>
#include <algorithm>
#include <type_traits>
#include "ap_tiles.hpp"
#include "ap_packed.hpp"

int ap_fill_u32(void *p, size_t n, uint32_t v, hipStream_t st);
int ap_alloc_graph(ap_index *ix);

#define AP_A_CAP 512   // a-side list entries staged in LDS

// =================================================================== S2: seed
// scores[r][j] = <dense[node r], dense[j]> for a slab of rows and all columns.
// Tile order of the seed products.  Workgroups are handed to the 8 XCDs round-robin by their linear id, and every XCD
// has an L2 of its own: workgroup b runs on XCD b % 8 and is the (b / 8)-th of that XCD.  Each XCD gets a contiguous
// band of row tiles and walks it column tile by column tile, so the band's rows stay in that XCD's L2 and a column
// tile is fetched once per XCD instead of once per row tile.  Returns false for the padding workgroups of a band that
// is shorter than the others.
#define AP_XCDS 8
__device__ __forceinline__ bool ap_seed_tile(int64_t row_tiles, int64_t &rt, int64_t &ct) {
    const int64_t band = (row_tiles + AP_XCDS - 1) / AP_XCDS;
    const int64_t xcd = blockIdx.x % AP_XCDS, idx = blockIdx.x / AP_XCDS;
    rt = xcd * band + idx % band;
    ct = idx / band;
    return rt < row_tiles;
}
static inline unsigned ap_seed_grid(int64_t row_tiles, int64_t col_tiles) {
    return (unsigned)(AP_XCDS * ((row_tiles + AP_XCDS - 1) / AP_XCDS) * col_tiles);
}

// The j-th of `ncols` documents that stand for a corpus of n: one of every n / ncols consecutive ones, by chance, so that a corpus in the order of its
// topics is represented by all of them: by its first documents the rows of the first topics got thresholds that left them short of K, and all others
// such that let too many through.  1,024 bf16 columns, K = 128: 33,000 documents in topics of 300 6.9 ms by the first documents, 5.3 by these, 100,000 in topics of 1,000 62 and
// 22, of 5,000 178 and 16; in no order 4.0 and 3.8, 16.6 and 16.7.
__device__ __forceinline__ int64_t ap_seed_sampled(int64_t j, int64_t ncols, int64_t n) {
    const int64_t at = j * n / ncols;
    return at + (int64_t)(((uint32_t)j * 0x9E3779B1u) >> 8) % ((j + 1) * n / ncols - at);
}

// sampled: the columns are not all documents but those (a row's own document gets a score that no other has to beat).
template <int DT>
__global__ __launch_bounds__(256) void k_seed_scores(const void *dense, int32_t dim, int64_t n, const int32_t *node_ids,
                                                     int64_t row0, int64_t nrows, int64_t ncols, bool sampled,
                                                     float *__restrict__ scores /* nrows x ncols */) {
    __shared__ __attribute__((aligned(16))) unsigned char lds[ApTileLds<DT>::BYTES];
    __shared__ int32_t a_rows[AP_TILE], b_rows[AP_TILE];
    int64_t rt, ct;
    if (!ap_seed_tile((nrows + AP_TILE - 1) / AP_TILE, rt, ct)) return;
    const int64_t i0 = rt * AP_TILE, j0 = ct * AP_TILE;
    if (threadIdx.x < AP_TILE) {
        const int64_t r = i0 + threadIdx.x;
        a_rows[threadIdx.x] = r < nrows ? (node_ids ? node_ids[row0 + r] : (int32_t)(row0 + r)) : -1;
        const int64_t j = j0 + threadIdx.x;
        b_rows[threadIdx.x] = j < ncols ? (int32_t)(sampled ? ap_seed_sampled(j, ncols, n) : j) : -1;
    }
    ap_f32x16 acc[2][2];
    ap_tile_product<DT>(dense, dim, a_rows, b_rows, lds, acc);
    ap_tile_foreach(acc, [&](int i, int j, float v) {
        if (i0 + i < nrows && j0 + j < ncols) scores[(i0 + i) * ncols + (j0 + j)] = sampled && a_rows[i] == b_rows[j] ? -INFINITY : v;
    });
}

// Appending a tile's candidates to their rows' buffers.  A candidate is not appended on the spot (an atomic on the
// row's counter whose answer the store has to wait for, at some forty of a lane's sixty-four elements): the wave notes
// it in its own part of the LDS the product has left (place = a running count + the lane's rank among the lanes that
// passed: no atomic, no wait); afterwards the candidates are counted per buffer in LDS, every buffer that has some takes its
// places with ONE atomic for the whole tile, and the candidates are written out.
// An entry: score bits | column in the tile << 32 | row in the tile << 40 | (later) place in the row's buffer << 48 | in the column's << 56.  One
// entry serves both sides of the symmetric sweep: the buffer of its row's document, with the id of its column's, and that of its
// column's document, with the id of its row's.  Which of them it is for is told when it is counted and when it is written, so that an
// element costs one comparison, with the lower of its two thresholds.
// direct(i, j, v): the append on the spot, for what the wave's part (wcap entries) cannot hold.
template <typename DIRECT>
__device__ __forceinline__ void ap_seed_stage(bool pass, int i, int j, float v, uint64_t *stage, int32_t wcap, int32_t &nw, DIRECT direct) {
    const uint64_t m = __ballot(pass);
    if (m) {
        if (pass) {
            const int32_t slot = nw + (int32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
            if (slot < wcap) stage[slot] = ((uint64_t)(uint32_t)((i << 8) | j) << 32) | __float_as_uint(v);
            else direct(i, j, v);
        }
        nw += __popcll(m);
    }
}
// Called by every thread of the workgroup once its wave has staged nw candidates.  to_row(i, j, v), to_col(i, j, v): whether a score is for the
// buffer of its row's document, of its column's.  s_cnt must be zero on entry: counters of the E rows, then (both) of the E columns; a buffer gets at
// most E <= 256 of a tile's candidates.  Buffers and counters are indexed by row0 + row and by col0 + column; the ids stored are id0 + column and id1 + row.
template <int E, typename TO_ROW, typename TO_COL>
__device__ __forceinline__ void ap_seed_flush(uint64_t *stage, int32_t wcap, int32_t nw, bool both, int32_t *s_cnt, int32_t *s_base, int32_t *__restrict__ cnt,
                                              unsigned long long *__restrict__ buf, int32_t cap, int64_t row0, int32_t id0, int64_t col0, int32_t id1,
                                              TO_ROW to_row, TO_COL to_col) {
    static_assert(E <= 256, "places of eight bits");
    const int lane = threadIdx.x & 63;
    const int32_t ns = nw < wcap ? nw : wcap;
    for (int32_t p = lane; p < ns; p += 64) {
        const uint64_t e = stage[p];
        const int32_t j = (int32_t)(e >> 32) & 255, i = (int32_t)(e >> 40) & 255;
        const float v = __uint_as_float((uint32_t)e);
        const uint32_t r = to_row(i, j, v) ? (uint32_t)atomicAdd(&s_cnt[i], 1) : 0u, c = both && to_col(i, j, v) ? (uint32_t)atomicAdd(&s_cnt[E + j], 1) : 0u;
        stage[p] = e | ((uint64_t)(r | (c << 8)) << 48);
    }
    __syncthreads();
    for (int32_t x = threadIdx.x; x < (both ? 2 * E : E); x += blockDim.x) {
        const int32_t c = s_cnt[x];
        s_base[x] = c ? atomicAdd(&cnt[x < E ? row0 + x : col0 + (x - E)], c) : 0;
    }
    __syncthreads();
    for (int32_t p = lane; p < ns; p += 64) {
        const uint64_t e = stage[p];
        const int32_t j = (int32_t)(e >> 32) & 255, i = (int32_t)(e >> 40) & 255;
        const float v = __uint_as_float((uint32_t)e);
        if (to_row(i, j, v)) {
            const int32_t pos = s_base[i] + ((int32_t)(e >> 48) & 255);
            if (pos < cap) buf[(row0 + i) * (int64_t)cap + pos] = ap_make_key(v, id0 + j, 1u);
        }
        if (both && to_col(i, j, v)) {
            const int32_t pos = s_base[E + j] + (int32_t)(e >> 56);
            if (pos < cap) buf[(col0 + j) * (int64_t)cap + pos] = ap_make_key(v, id1 + i, 1u);
        }
    }
}
// The append on the spot.
__device__ __forceinline__ void ap_seed_append(int64_t row, int32_t id, float v, int32_t *__restrict__ cnt, unsigned long long *__restrict__ buf, int32_t cap) {
    const int32_t pos = atomicAdd(&cnt[row], 1);
    if (pos < cap) buf[row * (int64_t)cap + pos] = ap_make_key(v, id, 1u);
}

// The same product over all columns, but instead of storing the scores, every
// score that reaches its row's threshold tau (a lower bound of the row's K-th
// best, found on a sample of the columns) is appended to the row's candidate
// buffer as a ranking key.  cnt[r] counts the appends (also those beyond cap).
// The launch covers column tiles from ct0 on.  SYM (rows = a slab of the whole corpus in order, every tile full and
// inside the corpus): tau, buf and cnt point at the slab's first row inside arrays that cover the whole corpus; tiles
// below the diagonal return at once, and a score of a tile above it is offered to its column's document as well (see
// k_seed_thresh_big).
template <int DT, bool SYM>
__global__ __launch_bounds__(256) void k_seed_thresh(const void *dense, int32_t dim, int64_t n, const int32_t *node_ids,
                                                     int64_t row0, int64_t nrows, const float *__restrict__ tau,
                                                     unsigned long long *__restrict__ buf, int32_t cap,
                                                     int32_t *__restrict__ cnt, int64_t ct0) {
    __shared__ __attribute__((aligned(16))) unsigned char lds[ApTileLds<DT>::BYTES];
    __shared__ int32_t a_rows[AP_TILE], b_rows[AP_TILE];
    __shared__ float s_tau[AP_TILE], s_tauc[SYM ? AP_TILE : 1];
    __shared__ int32_t s_cnt[(SYM ? 2 : 1) * AP_TILE], s_base[(SYM ? 2 : 1) * AP_TILE];
    int64_t rt, ct;
    if (!ap_seed_tile((nrows + AP_TILE - 1) / AP_TILE, rt, ct)) return;
    const int64_t i0 = rt * AP_TILE, j0 = (ct0 + ct) * AP_TILE;
    if (SYM && j0 < row0 + i0) return;   // below the diagonal: its mirror image does the work
    const bool mirror = SYM && j0 > row0 + i0;   // uniform
    if (threadIdx.x < AP_TILE) {
        const int64_t r = i0 + threadIdx.x;
        s_cnt[threadIdx.x] = 0;
        if (SYM) { s_cnt[AP_TILE + threadIdx.x] = 0; s_tauc[threadIdx.x] = mirror ? tau[j0 - row0 + threadIdx.x] : INFINITY; }
        a_rows[threadIdx.x] = r < nrows ? (node_ids ? node_ids[row0 + r] : (int32_t)(row0 + r)) : -1;
        s_tau[threadIdx.x] = r < nrows ? tau[r] : INFINITY;
        const int64_t j = j0 + threadIdx.x;
        b_rows[threadIdx.x] = j < n ? (int32_t)j : -1;
    }
    ap_f32x16 acc[2][2];
    ap_tile_product<DT>(dense, dim, a_rows, b_rows, lds, acc);
    __syncthreads();   // the product's LDS is free
    constexpr int W_CAP = ApTileLds<DT>::BYTES / 4 / 8;
    uint64_t *stage = reinterpret_cast<uint64_t *>(lds) + ap_wave_id() * W_CAP;
    auto in = [&](int i, int j) { return i0 + i < nrows && j0 + j < n && a_rows[i] != (int32_t)(j0 + j); };   // not the document itself, nor a row or column past the end
    auto to_row = [&](int i, int j, float v) { return v >= s_tau[i] && in(i, j); };
    auto to_col = [&](int i, int j, float v) { return mirror && v >= s_tauc[j] && in(i, j); };
    auto direct = [&](int i, int j, float v) {
        if (to_row(i, j, v)) ap_seed_append(i0 + i, (int32_t)(j0 + j), v, cnt, buf, cap);
        if (SYM && to_col(i, j, v)) ap_seed_append(j0 - row0 + j, (int32_t)(row0 + i0 + i), v, cnt, buf, cap);
    };
    int32_t nw = 0;
    ap_tile_foreach(acc, [&](int i, int j, float v) { ap_seed_stage(v >= (SYM ? fminf(s_tau[i], s_tauc[j]) : s_tau[i]), i, j, v, stage, W_CAP, nw, direct); });
    ap_seed_flush<AP_TILE>(stage, W_CAP, nw, SYM, s_cnt, s_base, cnt, buf, cap, i0, (int32_t)j0, j0 - row0, (int32_t)(row0 + i0), to_row, to_col);
}

// The thresholded sweep for bf16 rows on 256x256 tiles (the product above): the same appends as k_seed_thresh.
// 4 x 4 waves of 64 x 64 each: measured faster than 2 x 4 waves of 128 x 64 or 2 x 2 of 128 x 128 (fewer LDS reads per
// MFMA, but fewer waves to overlap them with), and 12 % faster than the 128 x 128 tiles of k_seed_thresh.
#ifndef AP_BIG_WM
#define AP_BIG_WM 4
#define AP_BIG_WN 4
#endif
// RUN: every tile of the launch is two runs of 256 consecutive documents inside the corpus (no node list, no ragged
// edge, dim a multiple of 64); the host launches the edges of a sweep with RUN = false.  The launch covers row tiles
// rt0 .. rt0 + nrt and column tiles from ct0 on.
// SYM (with RUN, rows = the whole corpus, row0 = 0): the product is symmetric, so only the tiles on and above the
// diagonal are computed (a launch's tiles below it return at once), and a score of an off-diagonal tile is offered
// twice: to its row's document against that document's threshold, and to its column's document against that one's.
// The mirrored pair would have got the same bits: the same products summed over k in the same order.
template <int DT, int WM, int WN, bool RUN, bool SYM>
__global__ __launch_bounds__(WM * WN * 64) void k_seed_thresh_big(const void *dense, int32_t dim, int64_t n, const int32_t *node_ids,
                                                                  int64_t row0, int64_t nrows, const float *__restrict__ tau,
                                                                  unsigned long long *__restrict__ buf, int32_t cap,
                                                                  int32_t *__restrict__ cnt, int64_t rt0, int64_t nrt, int64_t ct0) {
    static_assert(RUN || !SYM, "the symmetric sweep is for runs of consecutive documents");
    extern __shared__ __attribute__((aligned(16))) unsigned char big_lds[];
    __shared__ int32_t a_rows[AP_BIG], b_rows[AP_BIG];
    __shared__ __attribute__((aligned(16))) float s_tau[AP_BIG];
    __shared__ float s_tauc[SYM ? AP_BIG : 1];          // SYM: the thresholds of the tile's column documents
    __shared__ int32_t s_cnt[(SYM ? 2 : 1) * AP_BIG], s_base[(SYM ? 2 : 1) * AP_BIG];   // the tile's candidates per buffer, and where each buffer's go
    int64_t rt, ct;
    if (!ap_seed_tile(nrt, rt, ct)) return;
    const int64_t i0 = (rt0 + rt) * AP_BIG, j0 = (ct0 + ct) * AP_BIG;
    if (SYM && j0 < i0) return;   // below the diagonal: its mirror image does the work
    ap_f32x16 acc[ApBig<WM, WN>::FA][ApBig<WM, WN>::FB];
    constexpr int W_CAP = AP_BIG_LDS_BYTES / (WM * WN) / 8;   // entries of a wave's part of the LDS
    uint64_t *stage = reinterpret_cast<uint64_t *>(big_lds) + ap_wave_id() * W_CAP;
    int32_t nw = 0;   // uniform: candidates of this wave so far
    if (RUN) {
        const int32_t a_first = (int32_t)(row0 + i0), b_first = (int32_t)j0;
        // Only a tile whose row and column runs overlap can pair a document with itself.
        const bool diagonal = a_first < b_first + AP_BIG && b_first < a_first + AP_BIG;
        const bool mirror = SYM && !diagonal;   // uniform: the scores also go to the column documents
        // the thresholds travel while the product runs: a thread's is one of the rows' or one of the columns'
        static_assert(WM * WN * 64 >= 2 * AP_BIG, "a threshold a thread");
        const int32_t x = threadIdx.x & (AP_BIG - 1);
        float own = INFINITY;
        if (threadIdx.x < AP_BIG) own = tau[i0 + x];
        else if (mirror && threadIdx.x < 2 * AP_BIG) own = tau[j0 + x];
        ap_big_gemm_bf16<DT, WM, WN, true>(dense, dim, a_rows, b_rows, a_first, b_first, reinterpret_cast<uint16_t *>(big_lds), acc);
        if (threadIdx.x < AP_BIG) { s_tau[x] = own; s_cnt[x] = 0; }
        else if (SYM && threadIdx.x < 2 * AP_BIG) { s_tauc[x] = own; s_cnt[AP_BIG + x] = 0; }
        __syncthreads();
        const int lane = threadIdx.x & 63, wave = ap_wave_id();
        const int wm = wave / WN, wn = wave % WN;
        auto to_row = [&](int i, int j, float v) { return v >= s_tau[i] && !(diagonal && a_first + i == b_first + j); };
        auto to_col = [&](int, int j, float v) { return mirror && v >= s_tauc[j]; };
        auto direct = [&](int i, int j, float v) {
            if (to_row(i, j, v)) ap_seed_append(i0 + i, b_first + j, v, cnt, buf, cap);
            if (SYM && to_col(i, j, v)) ap_seed_append(j0 + j, a_first + i, v, cnt, buf, cap);
        };
        // A lane holds 4 consecutive rows x (FB x 32 columns apart) per 8-row group: the rows' thresholds come as one
        // 16-byte LDS read, and an element costs a minimum, a compare and a branch, taken at some three of ten.
        float tc[ApBig<WM, WN>::FB];   // the thresholds of this lane's columns
#pragma unroll
        for (int b = 0; b < ApBig<WM, WN>::FB; b++) tc[b] = SYM ? s_tauc[wn * (AP_BIG / WN) + b * 32 + (lane & 31)] : INFINITY;
#pragma unroll
        for (int a = 0; a < ApBig<WM, WN>::FA; a++)
#pragma unroll
            for (int q = 0; q < 4; q++) {
                const int ib = wm * (AP_BIG / WM) + a * 32 + 8 * q + 4 * (lane >> 5);
                const float4 t4 = *reinterpret_cast<const float4 *>(&s_tau[ib]);
                const float tt[4] = {t4.x, t4.y, t4.z, t4.w};
#pragma unroll
                for (int b = 0; b < ApBig<WM, WN>::FB; b++)
#pragma unroll
                    for (int rr = 0; rr < 4; rr++) {
                        const float v = acc[a][b][4 * q + rr];
                        ap_seed_stage(v >= (SYM ? fminf(tt[rr], tc[b]) : tt[rr]), ib + rr, wn * (AP_BIG / WN) + b * 32 + (lane & 31), v, stage, W_CAP, nw, direct);
                    }
            }
        ap_seed_flush<AP_BIG>(stage, W_CAP, nw, SYM, s_cnt, s_base, cnt, buf, cap, i0, b_first, j0, a_first, to_row, to_col);
    } else {
        for (int32_t x = threadIdx.x; x < AP_BIG; x += blockDim.x) {
            const int64_t r = i0 + x, j = j0 + x;
            a_rows[x] = r < nrows ? (node_ids ? node_ids[row0 + r] : (int32_t)(row0 + r)) : -1;
            s_tau[x] = r < nrows ? tau[r] : INFINITY;
            s_cnt[x] = 0;
            b_rows[x] = j < n ? (int32_t)j : -1;
        }
        ap_big_gemm_bf16<DT, WM, WN, false>(dense, dim, a_rows, b_rows, 0, 0, reinterpret_cast<uint16_t *>(big_lds), acc);
        auto to_row = [&](int i, int j, float v) { return v >= s_tau[i] && i0 + i < nrows && j0 + j < n && a_rows[i] != (int32_t)(j0 + j); };
        auto direct = [&](int i, int j, float v) { if (to_row(i, j, v)) ap_seed_append(i0 + i, (int32_t)(j0 + j), v, cnt, buf, cap); };
        ap_big_foreach<WM, WN>(acc, [&](int i, int j, float v) { ap_seed_stage(v >= s_tau[i], i, j, v, stage, W_CAP, nw, direct); });
        ap_seed_flush<AP_BIG>(stage, W_CAP, nw, false, s_cnt, s_base, cnt, buf, cap, i0, (int32_t)j0, (int64_t)0, 0, to_row, [](int, int, float) { return false; });
    }
}

// One block per row: exact top-K of the row (excluding the node itself), sorted.
// Row r of `scores` has ncols entries; its result goes to row out_row0 + r.
__global__ __launch_bounds__(256) void k_select_rows(const float *__restrict__ scores, int64_t ncols, int32_t K,
                                                     const int32_t *node_ids, int64_t row0, int32_t exclude_self, int64_t out_row0,
                                                     int32_t *__restrict__ out_ids, float *__restrict__ out_sc) {
    __shared__ uint32_t hist[256];
    __shared__ uint64_t sel[256];
    __shared__ int32_t misc[4];
    __shared__ uint64_t pre;
    const int64_t r = blockIdx.x;
    const int32_t self = exclude_self ? (node_ids ? node_ids[row0 + r] : (int32_t)(row0 + r)) : -1;
    for (int i = threadIdx.x; i < 256; i += blockDim.x) sel[i] = 0;
    __syncthreads();
    const int32_t got = ap_radix_select(scores + r * ncols, ncols, self, K, hist, sel, misc, &pre);
    ap_bitonic_desc(sel, 256);
    for (int32_t i = threadIdx.x; i < K; i += blockDim.x) {
        if (out_ids) out_ids[(out_row0 + r) * K + i] = i < got ? ap_key_id(sel[i]) : -1;
        out_sc[(out_row0 + r) * K + i] = i < got ? ap_key_score(sel[i]) : -INFINITY;
    }
}

// tau[r] = K-th best score of row r of a [nrows x K] sorted score table.
// ulps (a debug setting, normally 0) raises the threshold by that many representable values.
__global__ void k_take_tau(const float *__restrict__ sc, int64_t nrows, int32_t K, uint32_t ulps, float *__restrict__ tau) {
    const int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (r < nrows) {
        const float t = sc[r * K + K - 1];
        tau[r] = (ulps && t - t == 0.f) ? ap_ord2f(ap_f2ord(t) + ulps) : t;
    }
}

// One block per row: exact top-K among the row's buffered candidate keys.
// Rows whose buffer overflowed are reported in overflow_rows and left to the caller, and so are rows that hold fewer
// than `need` = min(K, n - 1) keys: the threshold came from another kernel's product of the same rows, and a score
// that kernel rounded one ulp higher would silently shorten the list.
__global__ __launch_bounds__(256) void k_select_buf(const unsigned long long *__restrict__ buf, int32_t cap,
                                                    const int32_t *__restrict__ cnt, int32_t K, int32_t need, int64_t out_row0,
                                                    int32_t *__restrict__ out_ids, float *__restrict__ out_sc,
                                                    int32_t *__restrict__ n_overflow, int32_t *__restrict__ overflow_rows) {
    __shared__ uint32_t hist[256];
    __shared__ uint64_t sel[256];
    __shared__ int32_t misc[4];
    __shared__ uint64_t pre;
    const int64_t r = blockIdx.x;
    const int32_t c = cnt[r];
    if (c > cap || c < need) {   // uniform for the block
        if (threadIdx.x == 0) overflow_rows[atomicAdd(n_overflow, 1)] = (int32_t)r;
        return;
    }
    for (int i = threadIdx.x; i < 256; i += blockDim.x) sel[i] = 0;
    __syncthreads();
    const unsigned long long *row = buf + r * (int64_t)cap;
    const int32_t got = ap_radix_select_keys([&](int64_t j) -> uint64_t { return row[j]; }, c, c, K, hist, sel, misc, &pre);
    ap_bitonic_desc(sel, 256);
    for (int32_t i = threadIdx.x; i < K; i += blockDim.x) {
        out_ids[(out_row0 + r) * K + i] = i < got ? ap_key_id(sel[i]) : -1;
        out_sc[(out_row0 + r) * K + i] = i < got ? ap_key_score(sel[i]) : -INFINITY;
    }
}

// The largest |value| of a table, as bits (of a NaN: larger than those of any number), zero at the start.  count is a multiple of 4.
__global__ __launch_bounds__(256) void k_seed_most(const float *__restrict__ v, int64_t count, uint32_t *__restrict__ most) {
    uint32_t m = 0;
    for (int64_t i = (blockIdx.x * (int64_t)256 + threadIdx.x) * 4; i < count; i += (int64_t)gridDim.x * 1024) {
        const uint4 y = *reinterpret_cast<const uint4 *>(v + i);
        m = max(m, max(max(y.x & 0x7fffffffu, y.y & 0x7fffffffu), max(y.z & 0x7fffffffu, y.w & 0x7fffffffu)));
    }
    for (int o = 32; o > 0; o >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, o, 64));
    if ((threadIdx.x & 63) == 0) atomicMax(most, m);
}
// The power of two that takes values of at most that size below 2^15 (f16 ends at 2^16), from its bits.
__host__ __device__ static inline int ap_seed_shift(uint32_t most) { return 141 - (int)(most >> 23); }
// Rows of f32 values times a power of two, rounded to f16 (columns dim .. kd are zeros; what f16 holds with fewer bits than 11 becomes zero) for a sweep on the 16-bit
// matrix cores whose candidates k_rescore_buf scores again.  lost[r] = {|a - a^|, |a|} of row r, in these units (a^: a rounded; the differences are exact), each with
// room for its own rounding.  stats: {largest |a|, largest |a - a^|, sum of |a|, largest |value| of the rows as they were}, as float bits, the first
// three zero at the start (a NaN or an infinity among the values ends up in the first).  A wave a row.
__global__ __launch_bounds__(256) void k_seed_round(const float *__restrict__ dense, int32_t dim, int64_t n, int32_t kd, uint16_t *__restrict__ rows,
                                                    float2 *__restrict__ lost, uint32_t *__restrict__ stats) {
    __shared__ uint32_t part[2][4];
    __shared__ float total[4];
    const int lane = threadIdx.x & 63, wave = ap_wave_id(), shift = ap_seed_shift(stats[3]);
    uint32_t most = 0, most_off = 0;
    float sum = 0.f;
    for (int64_t r = blockIdx.x * (int64_t)4 + wave; r < n; r += (int64_t)gridDim.x * 4) {
        float s = 0.f, o = 0.f;
        for (int32_t c = lane * 4; c < kd; c += 256) {
            const float4 y = c < dim ? *reinterpret_cast<const float4 *>(dense + r * dim + c) : make_float4(0.f, 0.f, 0.f, 0.f);   // dim is a multiple of 4
            const float x[4] = {ldexpf(y.x, shift), ldexpf(y.y, shift), ldexpf(y.z, shift), ldexpf(y.w, shift)};
            uint32_t h[4];
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const _Float16 f = fabsf(x[e]) < 0x1p-14f ? (_Float16)0.f : (_Float16)x[e];
                h[e] = (uint32_t)__builtin_bit_cast(uint16_t, f);
                const float off = x[e] - (float)f;
                s = fmaf(x[e], x[e], s);
                o = fmaf(off, off, o);
            }
            *reinterpret_cast<uint2 *>(rows + r * kd + c) = make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
        }
        const float norm = fmaf(sqrtf(ap_wave_sum(s)), 1.0001f, 1e-17f), off = fmaf(sqrtf(ap_wave_sum(o)), 1.0001f, 1e-17f);
        if (lane == 0) lost[r] = make_float2(off, norm);
        most = max(most, __float_as_uint(norm));
        most_off = max(most_off, __float_as_uint(off));
        sum += norm;
    }
    if (lane == 0) { part[0][wave] = most; part[1][wave] = most_off; total[wave] = sum; }
    __syncthreads();
    if (threadIdx.x < 2) {
        const uint32_t *p = part[threadIdx.x];
        atomicMax(&stats[threadIdx.x], max(max(p[0], p[1]), max(p[2], p[3])));
    }
    if (threadIdx.x == 2) atomicAdd(reinterpret_cast<float *>(&stats[2]), total[0] + total[1] + total[2] + total[3]);
}

// The exact top-K out of candidates whose scores are those of rounded rows.  With a^ for a rounded,  a b - a^ b^ = (a - a^) b + a^ (b - b^),
// so a row's scores are off by at most  slack = |a - a^| max|b| + |a^| max|b - b^|  and what the sums of both products round (dim 2^-22 |a| max|b|
// for the two).  With t the K-th best score of the rounded rows, a document of the exact top-K has one of at least t - 2 slack: those
// candidates (the band; some 1.1 K of them) are scored again in f32, one a lane, as a chain of fused multiply-adds in ascending order of the
// columns: what v_mfma_f32_32x32x2_f32 computes, so these are the bits of k_seed_scores and k_seed_thresh.  A row goes to the
// exact path if the band reaches below tau (where candidates are missing), or holds more than AP_BAND.
// What bounds it: the band's rows, gathered from all over the corpus.  A wave's candidates come in chunks of 32 columns, eight lanes a row (128 consecutive
// bytes), through its own part of the LDS, the next chunk's loads in flight while one is summed; of few candidates (no more than 8 or 16 a wave) eight or four
// chunks come at a time, as many bytes on their way as of many: 9.8 ms for 100,000 rows of 768 columns
// and K = 128 (some 45 GB at 4.6 TB/s); with rows rounded to bf16, whose slack is eight times as wide and whose band 1.7 K, 15.2.
// slack != NULL: what a construction needs of the lists, which is less: their members, which of them are the first `top`, the K-th score, and the
// others' scores within slack[r] of what is given.  With t the K-th best score of the rounded rows a candidate beyond t + 2 slack is one of
// the K best, whatever the rounding took, and with t' the top-th best one beyond t' + 2 slack is among the first `top`, one below t' - 2 slack is not: scored
// again are only the candidates within 2 slack of t or of t' (some twenty of 128), the others keep the rounded score.  Sorted together the
// two kinds fall on the right sides of both lines: an exact score above a line's true place lies at most slack above t, or at least slack below.
// 9.8 -> 4.4 ms of the 100,000 x 768 below (5.8 with one chunk of a row at a time).
#define AP_BAND 1024
__device__ __forceinline__ float ap_seed_slack(float2 a, const uint32_t *stats, int32_t dim) {
    const float nmax = __uint_as_float(stats[0]), emax = __uint_as_float(stats[1]);
    return 1.001f * (a.x * nmax + (a.y + a.x) * emax + (2.4e-7f * (float)(dim + 64)) * a.y * nmax);
}
__global__ __launch_bounds__(256) void k_rescore_buf(const float *__restrict__ dense, int32_t dim, const unsigned long long *__restrict__ buf, int32_t cap,
                                                     const int32_t *__restrict__ cnt, const float *__restrict__ tau, const float2 *__restrict__ lost,
                                                     const uint32_t *__restrict__ stats, int32_t K, int32_t top, float *__restrict__ slack, int32_t *__restrict__ out_ids,
                                                     float *__restrict__ out_sc, int32_t *__restrict__ n_overflow, int32_t *__restrict__ overflow_rows) {
    __shared__ uint64_t keys[AP_BAND];
    __shared__ __attribute__((aligned(16))) float s_a[1024];        // f32 rows have at most 1,024 columns
    __shared__ __attribute__((aligned(16))) float stage[4][64 * AP_LDS_STRIDE];
    __shared__ int32_t misc[4];
    __shared__ uint64_t pre;
    __shared__ uint32_t s_least, s_top;
    __shared__ int32_t s_band, s_sure;
    // while the band is looked for: the candidates (as many as fit, which is all of them but for a forced capacity), the K best, a histogram
    uint64_t *all = reinterpret_cast<uint64_t *>(stage[0]);
    constexpr int32_t ALL = 4 * 64 * AP_LDS_STRIDE / 2;
    uint64_t *sel = keys;                                           // [256]
    uint32_t *hist = reinterpret_cast<uint32_t *>(keys + 256);      // [256]
    const int64_t r = blockIdx.x;
    const int lane = threadIdx.x & 63, wave = ap_wave_id();
    const int32_t c = cnt[r];
    if (slack && threadIdx.x == 0) slack[r] = 0.f;   // rows left to the caller get exact scores
    if (c > cap || c < K) {   // uniform for the block
        if (threadIdx.x == 0) overflow_rows[atomicAdd(n_overflow, 1)] = (int32_t)r;
        return;
    }
    if (threadIdx.x == 0) { s_least = 0xffffffffu; s_top = 0xffffffffu; s_band = 0; s_sure = 0; }
    const unsigned long long *row = buf + r * (int64_t)cap;
    for (int32_t j = threadIdx.x; j < c && j < ALL; j += 256) all[j] = row[j];
    auto key_of = [&](int64_t j) -> uint64_t { return j < ALL ? all[j] : row[j]; };
    __syncthreads();
    const int32_t got = ap_radix_select_keys(key_of, c, c, K, hist, sel, misc, &pre);
    if ((int32_t)threadIdx.x < got) {
        const uint64_t own = sel[threadIdx.x];
        atomicMin(&s_least, (uint32_t)(own >> 32));
        if (slack && top < K) {   // uniform
            int32_t rank = 0;
            for (int32_t j = 0; j < got; j++) rank += sel[j] > own ? 1 : 0;
            if (rank == top - 1) s_top = (uint32_t)(own >> 32);
        }
    }
    for (int32_t x = threadIdx.x * 4; x < 1024; x += 1024)
        *reinterpret_cast<float4 *>(&s_a[x]) = x < dim ? *reinterpret_cast<const float4 *>(dense + r * dim + x) : make_float4(0.f, 0.f, 0.f, 0.f);
    __syncthreads();
    const float off = ap_seed_slack(lost[r], stats, dim), least = ap_ord2f(s_least) - 2.f * off, most = slack ? ap_ord2f(s_least) + 2.f * off : INFINITY;
    const float t_top = slack && s_top != 0xffffffffu ? ap_ord2f(s_top) : -INFINITY;
    if (least >= tau[r])
        for (int32_t j = threadIdx.x; j < c; j += 256) {
            const uint64_t key = key_of(j);
            const float x = ap_key_score(key);
            if (x >= least) {
                const bool open = !(x > most) || (x >= t_top - 2.f * off && x <= t_top + 2.f * off);
                const int32_t at = open ? atomicAdd(&s_band, 1) : AP_BAND - 1 - atomicAdd(&s_sure, 1);
                if (at >= 0 && at < AP_BAND) keys[at] = key;
            }
        }
    __syncthreads();
    const int32_t nb = s_band, sure = s_sure, all_n = nb + sure;   // all_n: at least K, or 0; sure: fewer than K
    if (nb == 0 || all_n > AP_BAND) {   // uniform
        if (threadIdx.x == 0) overflow_rows[atomicAdd(n_overflow, 1)] = (int32_t)r;
        return;
    }
    int32_t full = 256;
    while (full < all_n) full <<= 1;
    if (slack) {   // uniform: what keeps its score lies behind the others from here on
        const uint64_t key = (int32_t)threadIdx.x < sure ? keys[AP_BAND - 1 - threadIdx.x] : 0ull;
        const int scale = -2 * ap_seed_shift(stats[3]);
        __syncthreads();
        if ((int32_t)threadIdx.x < sure) keys[nb + threadIdx.x] = ap_make_key(ldexpf(ap_key_score(key), scale), ap_key_id(key), 1u);
        if (threadIdx.x == 0) slack[r] = 1.0001f * ldexpf(off, scale);
        __syncthreads();
    }
    for (int32_t x = all_n + (int32_t)threadIdx.x; x < full; x += 256) keys[x] = 0;
    const int32_t share = (nb + 3) >> 2, w1 = min(nb, (wave + 1) * share);
    float *st = stage[wave];
    // m <= 64 / SUB candidates from p0 on, SUB chunks of their rows at a time
    auto score = [&](int32_t p0, int32_t m, auto sub) {
        constexpr int SUB = decltype(sub)::value, G = 8 / SUB;   // groups of eight rows
        const int col = (lane & 7) * 4;
        const float *src[G];
        float4 v[8];
#pragma unroll
        for (int g = 0; g < G; g++) src[g] = dense + (int64_t)ap_key_id(keys[p0 + min((lane >> 3) + 8 * g, m - 1)]) * dim;
        const int32_t id = ap_key_id(keys[p0 + min(lane, m - 1)]);
        auto load = [&](int32_t k0) {
#pragma unroll
            for (int p = 0; p < 8; p++)
                if (8 * (p % G) < m) v[p] = *reinterpret_cast<const float4 *>(src[p % G] + min(k0 + 32 * (p / G) + col, dim - 4));
        };
        load(0);
        float acc = 0.f;
        for (int32_t k0 = 0; k0 < dim; k0 += 32 * SUB) {
            ap_wave_sync();
#pragma unroll
            for (int p = 0; p < 8; p++)
                if (8 * (p % G) < m) {
                    const bool inside = k0 + 32 * (p / G) + col < dim;   // s_a is zero where the columns end: any finite value does
                    float *d = st + ((lane >> 3) + 8 * p) * AP_LDS_STRIDE + col;
                    d[0] = inside ? v[p].x : 0.f; d[1] = inside ? v[p].y : 0.f; d[2] = inside ? v[p].z : 0.f; d[3] = inside ? v[p].w : 0.f;
                }
            if (k0 + 32 * SUB < dim) load(k0 + 32 * SUB);
            ap_wave_sync();
#pragma unroll
            for (int q = 0; q < SUB; q++) {
                const float *mine = st + (8 * G * q + min(lane, m - 1)) * AP_LDS_STRIDE;
#pragma unroll
                for (int e = 0; e < 32; e++) acc = fmaf(s_a[k0 + 32 * q + e], mine[e], acc);
            }
        }
        if (lane < m) keys[p0 + lane] = ap_make_key(acc, id, 1u);
    };
    if (share <= 8) {   // uniform for the block
        if (wave * share < w1) score(wave * share, w1 - wave * share, std::integral_constant<int, 8>());
    } else if (share <= 16) {
        if (wave * share < w1) score(wave * share, w1 - wave * share, std::integral_constant<int, 4>());
    } else {
        for (int32_t p0 = wave * share; p0 < w1; p0 += 64) score(p0, min(64, w1 - p0), std::integral_constant<int, 1>());
    }
    ap_bitonic_desc(keys, full);
    for (int32_t i = threadIdx.x; i < K; i += 256) {
        out_ids[r * K + i] = ap_key_id(keys[i]);
        out_sc[r * K + i] = ap_key_score(keys[i]);
    }
}

// Before the sweep: how many of a sample of rows it would leave open.  sc holds the m best scores of each with the sampled columns, `place`
// is where the K-th best of all columns is to be expected among them, `last` where the band ends at the latest: at tau, or at AP_BAND candidates.
__global__ __launch_bounds__(256) void k_seed_open(const float *__restrict__ sc, int32_t nrows, int32_t m, int32_t place, int32_t last,
                                                   const int32_t *__restrict__ rows, const float2 *__restrict__ lost, const uint32_t *__restrict__ stats,
                                                   int32_t dim, int32_t *__restrict__ n_open) {
    const int32_t i = blockIdx.x * 256 + threadIdx.x;
    if (i < nrows && sc[(int64_t)i * m + last] > sc[(int64_t)i * m + place] - 2.f * ap_seed_slack(lost[rows[i]], stats, dim)) atomicAdd(n_open, 1);
}
__global__ __launch_bounds__(256) void k_seed_spread(int32_t *__restrict__ rows, int32_t nrows, int64_t n) {
    const int32_t i = blockIdx.x * 256 + threadIdx.x;
    if (i < nrows) rows[i] = (int32_t)(i * n / nrows);
}

// Exact path: full score rows of a slab, then selection.  Rows [row0, row0+nrows) of the node list.
static hipError_t seed_exact_rows(const ap_index *ix, const int32_t *node_ids, int64_t row0, int64_t nrows, int32_t K,
                                  float *scratch, int64_t scratch_rows, int32_t *out_ids, float *out_sc, hipStream_t st) {
    const int64_t n = ix->docs.n;
    hipError_t e = hipSuccess;
    for (int64_t r0 = row0; r0 < row0 + nrows && e == hipSuccess; r0 += scratch_rows) {
        const int64_t nr = std::min(scratch_rows, row0 + nrows - r0);
        dim3 grid(ap_seed_grid((nr + AP_TILE - 1) / AP_TILE, (n + AP_TILE - 1) / AP_TILE));
        ix->seed_flops += (unsigned long long)(((nr + AP_TILE - 1) / AP_TILE) * ((n + AP_TILE - 1) / AP_TILE)) * 2ull * AP_TILE * AP_TILE * (unsigned long long)ix->docs.dim;
        if (ix->dtype == AP_F32)
            hipLaunchKernelGGL(k_seed_scores<AP_F32>, grid, dim3(256), 0, st, ix->docs.dense, ix->docs.dim, n, node_ids, r0, nr, n, false, scratch);
        else
            hipLaunchKernelGGL(k_seed_scores<AP_BF16>, grid, dim3(256), 0, st, ix->docs.dense, ix->docs.dim, n, node_ids, r0, nr, n, false, scratch);
        e = hipGetLastError();
        if (e != hipSuccess) break;
        hipLaunchKernelGGL(k_select_rows, dim3((unsigned)nr), dim3(256), 0, st, scratch, n, K, node_ids, r0, 1, r0, out_ids, out_sc);
        e = hipGetLastError();
    }
    return e;
}

// rows list[r] of a [*, K] table take the values of row r of a compact one
__global__ void k_scatter_rows(const int32_t *__restrict__ list, int64_t nlist, int32_t K, const int32_t *__restrict__ ids,
                               const float *__restrict__ sc, int32_t *__restrict__ out_ids, float *__restrict__ out_sc) {
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t < nlist * K) {
        const int64_t r = t / K, i = t % K;
        out_ids[(int64_t)list[r] * K + i] = ids[t];
        out_sc[(int64_t)list[r] * K + i] = sc[t];
    }
}

// S2 for a whole corpus: the sweep with half the products.  D D^T is symmetric, so only the tiles on and
// above the diagonal are multiplied and every score is offered to both of its documents (k_seed_thresh_big<.., SYM>).
// For that every document's candidate buffer has to exist at once, so the buffers are short (cap entries, by the
// memory that is free) and the thresholds tight: tau = the m-th best of cs sampled columns with m < K, chosen so that
// a row expects some 6 K candidates (less than half the buffer).  Such a tau is not a guaranteed lower bound of the row's K-th best: a row
// that ends up with fewer than K candidates (hardly any) or more than cap is redone by the exact path,
// like an overflowing row of the one-sided sweep.  The lists are the exact ones either way.
// rounded (f32 rows): thresholds and sweep take the rows rounded to f16, at eight times the matrix rate, and the few candidates that the
// rounding leaves open are scored in f32 (k_rescore_buf).  The lists are the same bits.  100,000 rows of 768 columns, K = 128: 82.7 ms with
// f32 products (71 of them the sweep), 20.9 ms rounded (9.4 the sweep); 96 columns: 23.4 and 9.9 ms.
// *done = false (and AP_OK): not applicable here (shape, memory; rounded: norms that differ too much, or rows too much alike for the
// rounding to tell them apart, which a sample of rows says before the sweep); the caller takes the next sweep.  Rows with a mean cosine of 0.8,
// 100,000 x 768, K = 128: 84.5 ms, the f32 sweep alone 83.8, and 100 with the rounded sweep in front of it.
// Where the line lies: a row left open takes the exact path, 5 us of 100,000 columns and 768 (1 us of 60,000 and 384), so that a tenth of them is
// what the rounding saves; corpora whose next path is the exact one for all rows (below 32,768 documents) can leave a quarter open.  Once the sweep is over its
// own time no longer counts, and an eighth (a half) may be open.
static int ap_seed_knn_symmetric(const ap_index *ix, int32_t K, bool rounded, int32_t *out_ids, float *out_sc, hipStream_t st, ApSeedRelax *relax, bool *done) {
    *done = false;
    const bool big = rounded || ix->dtype == AP_BF16;  // 16-bit rows: 256x256 tiles; f32 rows: 128x128 tiles
    const int64_t E = big ? AP_BIG : AP_TILE;
    const int64_t n = ix->docs.n, T = n / E;
    const int32_t dim = rounded ? (ix->docs.dim + AP_BK16 - 1) / AP_BK16 * AP_BK16 : ix->docs.dim;
    if ((big && dim % AP_BK16 != 0) || T < 2 || n > ((int64_t)1 << 30)) return AP_OK;
    size_t free_b = 0, total_b = 0;
    if (hipMemGetInfo(&free_b, &total_b) != hipSuccess) return AP_OK;
    int64_t cap = 4096;
    while (cap > 512 && (double)n * (double)cap * 8.0 > 0.62 * (double)free_b) cap >>= 1;
    if ((double)n * (double)cap * 8.0 > 0.62 * (double)free_b) return AP_OK;
    // Every candidate costs the sweep and the selection (200,000 bf16 documents of 1,024 columns, K = 128: the sweep 45.1 ms with 1,843 a row and a
    // comparison for each side of an element, 40.0 with 781 and one), and 6 K of them
    // do, from a sample that need not be large: a rank of 12 leaves a row in a million short of K.  Where they are scored again 4.5 K are four times
    // what the band takes, and a rank of 24 leaves a row in a hundred thousand short.
    const double mean = std::min(0.45 * (double)cap, rounded ? std::max(4.5 * K, 24.0 * (double)n / 4096.0) : std::max(6.0 * K, 12.0 * (double)n / 4096.0));
    // the rounded sweep needs more candidates than K: on a small corpus a rank beyond K
    const int64_t m_max = rounded ? 256 : K;
    int64_t m = std::min<int64_t>(m_max, rounded || mean < 6.0 * K ? 24 : 12);
    int64_t cs = (int64_t)((double)m * (double)n / mean) + 1;
    const int64_t cs_min = g_ap_debug.seed_sample_cols > 0 ? std::max<int64_t>(K + 1, g_ap_debug.seed_sample_cols) : 4096;
    if (cs < cs_min || g_ap_debug.seed_sample_cols > 0) {   // a fixed sample: the rank that gives the same expectation
        cs = cs_min;
        m = std::min<int64_t>(m_max, std::max<int64_t>(m, (int64_t)(mean * (double)cs / (double)n) + 1));
    }
    cs = (cs + AP_TILE - 1) / AP_TILE * AP_TILE;
    if (n < 2 * cs) return AP_OK;
    // The band takes some 1.1 K candidates, and a row's number of candidates is off by one part in sqrt(m).
    if (rounded && ((double)m * (double)n / (double)cs < 3.0 * K || (double)n * ((double)cap * 8.0 + (double)dim * 2.0) > 0.75 * (double)free_b)) return AP_OK;
    if (g_ap_debug.seed_buffer_cap > 0) cap = g_ap_debug.seed_buffer_cap;   // forces overflows
    const int64_t RS = 8192;
    float *scratch = nullptr, *tau = nullptr, *tmp_sc = nullptr;
    unsigned long long *buf = nullptr;
    int32_t *cnt = nullptr, *ovf = nullptr;
    const void *dense = ix->docs.dense;
    uint16_t *r16 = nullptr;
    float2 *lost = nullptr;
    uint32_t *stats = nullptr;
    float *slack = nullptr;
    if (rounded) {
        float got[3] = {0.f, 0.f, 0.f};
        uint32_t bits[4] = {0u, 0u, 0u, 0u};
        int rr = ap_dev_alloc(&r16, (size_t)n * (size_t)dim);
        if (rr == AP_OK) rr = ap_dev_alloc(&lost, (size_t)n);
        if (rr == AP_OK) rr = ap_dev_alloc(&stats, 4);
        if (rr == AP_OK) rr = ap_fill_u32(stats, 4, 0u, st);
        if (rr == AP_OK) {
            hipLaunchKernelGGL(k_seed_most, dim3(1024), dim3(256), 0, st, static_cast<const float *>(dense), n * ix->docs.dim, stats + 3);
            hipLaunchKernelGGL(k_seed_round, dim3((unsigned)std::min<int64_t>((n + 3) / 4, 2048)), dim3(256), 0, st, static_cast<const float *>(dense),
                               ix->docs.dim, n, dim, r16, lost, stats);
            if (hipGetLastError() != hipSuccess || hipMemcpyAsync(bits, stats, sizeof(bits), hipMemcpyDeviceToHost, st) != hipSuccess ||
                hipStreamSynchronize(st) != hipSuccess)
                rr = AP_EHIP;
        }
        memcpy(got, bits, sizeof(got));
        for (int i = 0; i < 3; i += 2) got[i] = ldexpf(got[i], -ap_seed_shift(bits[3]));   // the norms as they were
        // one row's slack is made with the corpus's largest norms: of use while the others come near them
        if (rr != AP_OK || !(got[0] >= 1e-10f && got[0] <= 1e15f && got[0] <= 4.f * got[2] / (float)n)) {
            void *ptrs[] = {r16, lost, stats};
            for (void *q : ptrs) if (q) (void)hipFree(q);
            (void)hipGetLastError();
            ap_set_error("%s", "");
            return AP_OK;
        }
        dense = r16;
    }
    int rc = ap_dev_alloc(&scratch, (size_t)RS * (size_t)cs);
    if (rc == AP_OK) rc = ap_dev_alloc(&tmp_sc, (size_t)RS * (size_t)m);
    if (rc == AP_OK) rc = ap_dev_alloc(&ovf, (size_t)n + 1);
    hipError_t e = hipSuccess;
    bool alike = false;   // the rounding leaves too many rows open
    int32_t *re_ids = nullptr; float *re_sc = nullptr, *ex_scratch = nullptr;
    const int64_t open_part = n < 32768 ? 4 : 10;
    const bool forced = g_ap_debug.seed_buffer_cap != 0 || g_ap_debug.seed_tau_ulps != 0;
    if (rc == AP_OK && rounded && !forced) {
        const int32_t rows = (int32_t)std::min<int64_t>(1024, n / 256 * 256);   // two tiles of 256 at least; the list of rows has n + 1 entries
        const int32_t place = std::max(0, (int32_t)((double)K * (double)cs / (double)n + 0.5) - 1);
        const int32_t last = std::max(place, (int32_t)std::min<int64_t>(m, (int64_t)AP_BAND * cs / n) - 1);
        int32_t n_open = 0;
        rc = ap_fill_u32(ovf, 1, 0u, st);
        if (rc == AP_OK) {
            hipLaunchKernelGGL(k_seed_spread, dim3(rows / 256), dim3(256), 0, st, ovf + 1, rows, n);
            ix->seed_flops += (unsigned long long)((rows / AP_TILE) * (cs / AP_TILE)) * 2ull * AP_TILE * AP_TILE * (unsigned long long)dim;
            hipLaunchKernelGGL(k_seed_scores<AP_F16>, dim3(ap_seed_grid(rows / AP_TILE, cs / AP_TILE)), dim3(256), 0, st, dense, dim, n, ovf + 1, (int64_t)0,
                               (int64_t)rows, cs, true, scratch);
            hipLaunchKernelGGL(k_select_rows, dim3(rows), dim3(256), 0, st, scratch, cs, (int32_t)m, ovf + 1, (int64_t)0, 0, (int64_t)0, (int32_t *)nullptr, tmp_sc);
            hipLaunchKernelGGL(k_seed_open, dim3(rows / 256), dim3(256), 0, st, tmp_sc, rows, (int32_t)m, place, last, ovf + 1, lost, stats, ix->docs.dim, ovf);
            e = hipGetLastError();
            if (e == hipSuccess) e = hipMemcpyAsync(&n_open, ovf, sizeof(int32_t), hipMemcpyDeviceToHost, st);
            if (e == hipSuccess) e = hipStreamSynchronize(st);
            alike = e == hipSuccess && n_open > rows / open_part;
            ap_progress("seed lists: rounding leaves %d of %d sampled rows open", (int)n_open, (int)rows);
        }
    }
    if (rc == AP_OK && !alike) rc = ap_dev_alloc(&tau, (size_t)n);
    if (rc == AP_OK && !alike) rc = ap_dev_alloc(&cnt, (size_t)n);
    if (rc == AP_OK && !alike && rounded && relax) rc = ap_dev_alloc(&slack, (size_t)n);
    const bool sweep = rc == AP_OK && e == hipSuccess && !alike;
    if (sweep && ap_dev_alloc(&buf, (size_t)n * (size_t)cap) != AP_OK) {   // no room for the buffers after all: the next sweep
        void *ptrs[] = {scratch, tau, tmp_sc, cnt, ovf, r16, lost, stats, slack};
        for (void *q : ptrs) if (q) (void)hipFree(q);
        (void)hipGetLastError();
        ap_set_error("%s", "");
        return AP_OK;
    }
    if (sweep) {
        // thresholds of all rows
        for (int64_t row0 = 0; row0 < n && e == hipSuccess; row0 += RS) {
            const int64_t nrows = std::min(RS, n - row0);
            dim3 gs(ap_seed_grid((nrows + AP_TILE - 1) / AP_TILE, cs / AP_TILE));
            ix->seed_flops += (unsigned long long)(((nrows + AP_TILE - 1) / AP_TILE) * (cs / AP_TILE)) * 2ull * AP_TILE * AP_TILE * (unsigned long long)dim;
            if (rounded)
                hipLaunchKernelGGL(k_seed_scores<AP_F16>, gs, dim3(256), 0, st, dense, dim, n, (const int32_t *)nullptr, row0, nrows,
                                   cs, true, scratch);
            else if (big)
                hipLaunchKernelGGL(k_seed_scores<AP_BF16>, gs, dim3(256), 0, st, dense, dim, n, (const int32_t *)nullptr, row0, nrows,
                                   cs, true, scratch);
            else
                hipLaunchKernelGGL(k_seed_scores<AP_F32>, gs, dim3(256), 0, st, dense, dim, n, (const int32_t *)nullptr, row0, nrows,
                                   cs, true, scratch);
            hipLaunchKernelGGL(k_select_rows, dim3((unsigned)nrows), dim3(256), 0, st, scratch, cs, (int32_t)m, (const int32_t *)nullptr, row0, 0,
                               (int64_t)0, (int32_t *)nullptr, tmp_sc);
            hipLaunchKernelGGL(k_take_tau, dim3((unsigned)((nrows + 255) / 256)), dim3(256), 0, st, tmp_sc, nrows, (int32_t)m,
                               (uint32_t)g_ap_debug.seed_tau_ulps, tau + row0);
            e = hipGetLastError();
        }
        if (e == hipSuccess) rc = ap_fill_u32(cnt, (size_t)n, 0u, st);
        if (rc == AP_OK) rc = ap_fill_u32(ovf, 1, 0u, st);
    }
    if (sweep && rc == AP_OK && e == hipSuccess) {
        ap_progress("seed lists: thresholds of %lld rows (rank %lld of %lld sampled columns), buffers of %lld", (long long)n, (long long)m,
                    (long long)cs, (long long)cap);
        // tiles multiplied: those on and above the diagonal, and the ragged last row and column of tiles
        ix->seed_flops += (unsigned long long)(T * (T + 1) / 2 + (n % E != 0 ? 2 * T + 1 : 0)) * 2ull * (unsigned long long)(E * E) * (unsigned long long)dim;
        auto sweep = [&](auto type) {
            constexpr int DT = decltype(type)::value;
            const dim3 tb(AP_BIG_WM * AP_BIG_WN * 64);
            e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_seed_thresh_big<DT, AP_BIG_WM, AP_BIG_WN, true, true>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, AP_BIG_LDS_BYTES);
            if (e == hipSuccess)
                e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_seed_thresh_big<DT, AP_BIG_WM, AP_BIG_WN, false, false>),
                                        hipFuncAttributeMaxDynamicSharedMemorySize, AP_BIG_LDS_BYTES);
            // the square of full tiles, a slab of 32 row tiles a launch: each XCD keeps four row tiles and walks the column
            // tiles from the slab's own first column on
            for (int64_t s0 = 0; s0 < T && e == hipSuccess; s0 += 32) {
                const int64_t nrt = std::min<int64_t>(32, T - s0), nct = T - s0;
                hipLaunchKernelGGL((k_seed_thresh_big<DT, AP_BIG_WM, AP_BIG_WN, true, true>), dim3(ap_seed_grid(nrt, nct)), tb, AP_BIG_LDS_BYTES, st,
                                   dense, dim, n, (const int32_t *)nullptr, (int64_t)0, n, tau, buf, (int32_t)cap, cnt, s0, nrt, s0);
                e = hipGetLastError();
                if ((s0 / 32) % 64 == 63) {
                    if (e == hipSuccess) e = hipStreamSynchronize(st);
                    ap_progress("seed lists: %lld of %lld row tiles", (long long)(s0 + nrt), (long long)T);
                }
            }
            if (e == hipSuccess && n % AP_BIG != 0) {
                // the ragged last column tile for the full row tiles, and the ragged last rows against every column: one-sided
                hipLaunchKernelGGL((k_seed_thresh_big<DT, AP_BIG_WM, AP_BIG_WN, false, false>), dim3(ap_seed_grid(T, 1)), tb, AP_BIG_LDS_BYTES, st,
                                   dense, dim, n, (const int32_t *)nullptr, (int64_t)0, n, tau, buf, (int32_t)cap, cnt, (int64_t)0, T, T);
                hipLaunchKernelGGL((k_seed_thresh_big<DT, AP_BIG_WM, AP_BIG_WN, false, false>), dim3(ap_seed_grid(1, T + 1)), tb, AP_BIG_LDS_BYTES, st,
                                   dense, dim, n, (const int32_t *)nullptr, (int64_t)0, n, tau, buf, (int32_t)cap, cnt, T, (int64_t)1, (int64_t)0);
                e = hipGetLastError();
            }
        };
        if (rounded) sweep(std::integral_constant<int, AP_F16>());
        else if (big) sweep(std::integral_constant<int, AP_BF16>());
        else {
            // f32 rows: the same on 128x128 tiles, a slab of 64 row tiles (eight per XCD) a launch
            for (int64_t s0 = 0; s0 < T && e == hipSuccess; s0 += 64) {
                const int64_t nrt = std::min<int64_t>(64, T - s0), nct = T - s0, r0 = s0 * AP_TILE;
                hipLaunchKernelGGL((k_seed_thresh<AP_F32, true>), dim3(ap_seed_grid(nrt, nct)), dim3(256), 0, st, dense, dim, n,
                                   (const int32_t *)nullptr, r0, nrt * AP_TILE, tau + r0, buf + r0 * cap, (int32_t)cap, cnt + r0, s0);
                e = hipGetLastError();
            }
            if (e == hipSuccess && n % AP_TILE != 0) {
                const int64_t r0 = T * AP_TILE;
                hipLaunchKernelGGL((k_seed_thresh<AP_F32, false>), dim3(ap_seed_grid(T, 1)), dim3(256), 0, st, dense, dim, n,
                                   (const int32_t *)nullptr, (int64_t)0, r0, tau, buf, (int32_t)cap, cnt, T);
                hipLaunchKernelGGL((k_seed_thresh<AP_F32, false>), dim3(ap_seed_grid(1, T + 1)), dim3(256), 0, st, dense, dim, n,
                                   (const int32_t *)nullptr, r0, n - r0, tau + r0, buf + r0 * cap, (int32_t)cap, cnt + r0, (int64_t)0);
                e = hipGetLastError();
            }
        }
        int32_t n_ovf = 0;
        if (e == hipSuccess) {
            if (rounded)
                hipLaunchKernelGGL(k_rescore_buf, dim3((unsigned)n), dim3(256), 0, st, static_cast<const float *>(ix->docs.dense), ix->docs.dim, buf, (int32_t)cap,
                                   cnt, tau, lost, stats, K, relax ? relax->top : 0, slack, out_ids, out_sc, ovf, ovf + 1);
            else
                hipLaunchKernelGGL(k_select_buf, dim3((unsigned)n), dim3(256), 0, st, buf, (int32_t)cap, cnt, K, (int32_t)std::min<int64_t>(K, n - 1),
                                   (int64_t)0, out_ids, out_sc, ovf, ovf + 1);
            e = hipGetLastError();
        }
        if (e == hipSuccess) e = hipMemcpyAsync(&n_ovf, ovf, sizeof(int32_t), hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e == hipSuccess && rounded && n_ovf > n / (open_part - 2) && !forced) alike = true;
        else if (e == hipSuccess && n_ovf > 0) {   // rows left short or overflowing: the exact path
            ap_progress("seed lists: %d rows redone by the exact path", (int)n_ovf);
            (void)hipFree(buf); buf = nullptr;
            int64_t ex_rows = std::max<int64_t>(AP_TILE, (((int64_t)1 << 28) / n) / AP_TILE * AP_TILE);
            ex_rows = std::min<int64_t>(ex_rows, ((int64_t)n_ovf + AP_TILE - 1) / AP_TILE * AP_TILE);
            rc = ap_dev_alloc(&ex_scratch, (size_t)ex_rows * (size_t)n);
            if (rc == AP_OK) rc = ap_dev_alloc(&re_ids, (size_t)n_ovf * (size_t)K);
            if (rc == AP_OK) rc = ap_dev_alloc(&re_sc, (size_t)n_ovf * (size_t)K);
            if (rc == AP_OK) {
                e = seed_exact_rows(ix, ovf + 1, 0, n_ovf, K, ex_scratch, ex_rows, re_ids, re_sc, st);
                if (e == hipSuccess) {
                    const int64_t tot = (int64_t)n_ovf * K;
                    hipLaunchKernelGGL(k_scatter_rows, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, st, ovf + 1, (int64_t)n_ovf, K, re_ids, re_sc,
                                       out_ids, out_sc);
                    e = hipGetLastError();
                }
                if (e == hipSuccess) e = hipStreamSynchronize(st);
            }
        }
    }
    void *ptrs[] = {scratch, tau, tmp_sc, buf, cnt, ovf, ex_scratch, re_ids, re_sc, r16, lost, stats};
    for (void *q : ptrs) if (q) (void)hipFree(q);
    if (slack && rc == AP_OK && e == hipSuccess && !alike) relax->slack = slack;
    else if (slack) (void)hipFree(slack);
    if (rc == AP_ENOMEM && rounded) {   // the f32 sweep takes less: no rounded rows, and hardly any score rows
        (void)hipGetLastError();
        ap_set_error("%s", "");
        return AP_OK;
    }
    if (rc != AP_OK) return rc;
    if (e != hipSuccess) { ap_set_error("seed k-NN failed: %s", hipGetErrorString(e)); return AP_EHIP; }
    *done = !alike;
    if (*done && rounded) ix->seed_bf16 = 1;
    return AP_OK;
}

// Whole corpora of f32 rows from which the rounded sweep is the faster one, K = 128: 7.5 ms of score rows and 4.6 ms rounded at 20,000 documents of
// 768 columns, 1.6 and 2.2 ms at 8,192 (K = 64 at 12,000: 3.0 and 2.5 ms).
#define AP_ROUNDED_MIN 16384
// S2.  Small corpora: every score row is materialised and the K best are
// selected from it.  Large corpora: the N x N scores are never stored: a
// sample of the columns gives each row a lower bound tau of its K-th best
// score, then one sweep over all columns appends only the scores >= tau to a
// per-row candidate buffer, from which the exact top-K is selected.  A row
// whose buffer overflows (not observed; the buffer holds twice the expected
// number of candidates) is redone by the exact path.  Whole corpora take the
// symmetric sweeps where they apply.
int ap_seed_knn_impl(const ap_index *ix, const int32_t *node_ids, int64_t nn, int32_t K, int32_t *out_ids,
                         float *out_sc, hipStream_t st, ApSeedRelax *relax, const ApWork &work) {
    const int64_t n = ix->docs.n;
    int64_t cs = std::max<int64_t>(16384, (n + 63) / 64);
    if (g_ap_debug.seed_sample_cols > 0) cs = std::max<int64_t>(K + 1, g_ap_debug.seed_sample_cols);
    cs = (cs + AP_TILE - 1) / AP_TILE * AP_TILE;
    // rows per launch of the exact path: a score slab of ~1 GiB
    int64_t ex_rows = std::max<int64_t>(AP_TILE, (((int64_t)1 << 28) / n) / AP_TILE * AP_TILE);
    ex_rows = std::min<int64_t>(ex_rows, (nn + AP_TILE - 1) / AP_TILE * AP_TILE);
    hipError_t e = hipSuccess;
    int rc = AP_OK;
    const bool whole = !node_ids && !g_ap_debug.seed_one_sided;   // the symmetric sweeps' case
    ix->seed_bf16 = ix->dtype == AP_BF16 ? 1 : 0;
    if (whole && ix->dtype == AP_F32 && n < 2 * cs && n >= AP_ROUNDED_MIN) {
        bool done = false;
        rc = ap_seed_knn_symmetric(ix, K, true, out_ids, out_sc, st, relax, &done);
        if (rc != AP_OK || done) return rc;
    }
    if (n < 2 * cs) {
        float *own = nullptr, *scratch = work.take<float>((size_t)ex_rows * (size_t)n);
        if (!scratch) { AP_TRY(ap_dev_alloc(&own, (size_t)ex_rows * (size_t)n)); scratch = own; }
        e = seed_exact_rows(ix, node_ids, 0, nn, K, scratch, ex_rows, out_ids, out_sc, st);
        if (own) {
            if (e == hipSuccess) e = hipStreamSynchronize(st);
            (void)hipFree(own);
        }
        if (e != hipSuccess) { ap_set_error("seed k-NN failed: %s", hipGetErrorString(e)); return AP_EHIP; }
        return AP_OK;
    }
    if (whole) {   // the symmetric sweep where it applies
        bool done = false;
        for (int rounded = ix->dtype == AP_F32 ? 1 : 0; rounded >= 0; rounded--) {
            rc = ap_seed_knn_symmetric(ix, K, rounded != 0, out_ids, out_sc, st, relax, &done);
            if (rc != AP_OK || done) return rc;
        }
    }
    const int64_t RS = std::min<int64_t>(8192, (nn + AP_TILE - 1) / AP_TILE * AP_TILE);
    // expected candidates per row = K * n / cs (tau is the K-th best of cs sampled columns)
    int64_t cap = 1024;
    while (cap < 2 * ((int64_t)K * n / cs + K)) cap <<= 1;
    if (g_ap_debug.seed_buffer_cap > 0) cap = g_ap_debug.seed_buffer_cap;   // forces overflows
    float *scratch = nullptr, *tau = nullptr, *tmp_sc = nullptr, *ex_scratch = nullptr;
    unsigned long long *buf = nullptr;
    int32_t *cnt = nullptr, *ovf = nullptr;   // ovf[0] = number of overflowed rows, ovf[1..] = their indices
    rc = ap_dev_alloc(&scratch, (size_t)RS * (size_t)cs);
    if (rc == AP_OK) rc = ap_dev_alloc(&tau, (size_t)RS);
    if (rc == AP_OK) rc = ap_dev_alloc(&tmp_sc, (size_t)RS * K);
    if (rc == AP_OK) rc = ap_dev_alloc(&buf, (size_t)RS * (size_t)cap);
    if (rc == AP_OK) rc = ap_dev_alloc(&cnt, (size_t)RS);
    if (rc == AP_OK) rc = ap_dev_alloc(&ovf, (size_t)RS + 1);
    for (int64_t row0 = 0; rc == AP_OK && row0 < nn && e == hipSuccess; row0 += RS) {
        const int64_t nrows = std::min(RS, nn - row0);
        const int64_t ytiles = (nrows + AP_TILE - 1) / AP_TILE;
        dim3 gs(ap_seed_grid(ytiles, cs / AP_TILE)), gf(ap_seed_grid(ytiles, (n + AP_TILE - 1) / AP_TILE));
        {   // FLOPs of the sample product and of the sweep (tiles of 128 for f32 rows, of 256 for bf16 rows)
            const unsigned long long d2 = 2ull * (unsigned long long)ix->docs.dim;
            ix->seed_flops += (unsigned long long)(ytiles * (cs / AP_TILE)) * AP_TILE * AP_TILE * d2;
            if (ix->dtype == AP_F32) ix->seed_flops += (unsigned long long)(ytiles * ((n + AP_TILE - 1) / AP_TILE)) * AP_TILE * AP_TILE * d2;
            else ix->seed_flops += (unsigned long long)(((nrows + AP_BIG - 1) / AP_BIG) * ((n + AP_BIG - 1) / AP_BIG)) * AP_BIG * AP_BIG * d2;
        }
        if (ix->dtype == AP_F32)
            hipLaunchKernelGGL(k_seed_scores<AP_F32>, gs, dim3(256), 0, st, ix->docs.dense, ix->docs.dim, n, node_ids, row0, nrows, cs, false, scratch);
        else
            hipLaunchKernelGGL(k_seed_scores<AP_BF16>, gs, dim3(256), 0, st, ix->docs.dense, ix->docs.dim, n, node_ids, row0, nrows, cs, false, scratch);
        hipLaunchKernelGGL(k_select_rows, dim3((unsigned)nrows), dim3(256), 0, st, scratch, cs, K, node_ids, row0, 1, (int64_t)0,
                           (int32_t *)nullptr, tmp_sc);
        hipLaunchKernelGGL(k_take_tau, dim3((unsigned)((nrows + 255) / 256)), dim3(256), 0, st, tmp_sc, nrows, K,
                           (uint32_t)g_ap_debug.seed_tau_ulps, tau);
        rc = ap_fill_u32(cnt, (size_t)nrows, 0u, st);
        if (rc == AP_OK) rc = ap_fill_u32(ovf, 1, 0u, st);
        if (rc != AP_OK) break;
        if (ix->dtype == AP_F32)
            hipLaunchKernelGGL((k_seed_thresh<AP_F32, false>), gf, dim3(256), 0, st, ix->docs.dense, ix->docs.dim, n, node_ids, row0, nrows, tau, buf, (int32_t)cap, cnt, (int64_t)0);
        else {
            // the inner tiles (runs of consecutive documents, all inside the corpus) take the lean instantiation, the ragged
            // last row tile and last column tile the general one
            const int64_t row_tiles = (nrows + AP_BIG - 1) / AP_BIG, col_tiles = (n + AP_BIG - 1) / AP_BIG;
            const bool runs = node_ids == nullptr && ix->docs.dim % AP_BK16 == 0;
            const int64_t full_rt = runs ? nrows / AP_BIG : 0, full_ct = runs ? n / AP_BIG : 0;
            auto sweep = [&](bool lean, int64_t rt0, int64_t nrt, int64_t ct0, int64_t nct) {
                if (nrt <= 0 || nct <= 0 || e != hipSuccess) return;
                const dim3 gb(ap_seed_grid(nrt, nct));
                const dim3 tb(AP_BIG_WM * AP_BIG_WN * 64);
                if (lean) {
                    e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_seed_thresh_big<AP_BF16, AP_BIG_WM, AP_BIG_WN, true, false>),
                                            hipFuncAttributeMaxDynamicSharedMemorySize, AP_BIG_LDS_BYTES);
                    if (e == hipSuccess)
                        hipLaunchKernelGGL((k_seed_thresh_big<AP_BF16, AP_BIG_WM, AP_BIG_WN, true, false>), gb, tb, AP_BIG_LDS_BYTES, st, ix->docs.dense, ix->docs.dim, n,
                                           node_ids, row0, nrows, tau, buf, (int32_t)cap, cnt, rt0, nrt, ct0);
                } else {
                    e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_seed_thresh_big<AP_BF16, AP_BIG_WM, AP_BIG_WN, false, false>),
                                            hipFuncAttributeMaxDynamicSharedMemorySize, AP_BIG_LDS_BYTES);
                    if (e == hipSuccess)
                        hipLaunchKernelGGL((k_seed_thresh_big<AP_BF16, AP_BIG_WM, AP_BIG_WN, false, false>), gb, tb, AP_BIG_LDS_BYTES, st, ix->docs.dense, ix->docs.dim, n,
                                           node_ids, row0, nrows, tau, buf, (int32_t)cap, cnt, rt0, nrt, ct0);
                }
                if (e == hipSuccess) e = hipGetLastError();
            };
            sweep(true, 0, full_rt, 0, full_ct);
            sweep(false, 0, full_rt, full_ct, col_tiles - full_ct);          // ragged last column tile
            sweep(false, full_rt, row_tiles - full_rt, 0, col_tiles);        // ragged last row tile (or everything)
            if (e != hipSuccess) break;
        }
        hipLaunchKernelGGL(k_select_buf, dim3((unsigned)nrows), dim3(256), 0, st, buf, (int32_t)cap, cnt, K,
                           (int32_t)std::min<int64_t>(K, n - 1), row0, out_ids, out_sc, ovf, ovf + 1);
        e = hipGetLastError();
        if (e != hipSuccess) break;
        int32_t n_ovf = 0;
        e = hipMemcpyAsync(&n_ovf, ovf, sizeof(int32_t), hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e != hipSuccess) break;
        if ((row0 / RS) % 64 == 63) ap_progress("seed lists: %lld of %lld rows", (long long)(row0 + nrows), (long long)nn);
        if (n_ovf > 0) {   // redo the slab by the exact path
            if (!ex_scratch) rc = ap_dev_alloc(&ex_scratch, (size_t)ex_rows * (size_t)n);
            if (rc != AP_OK) break;
            e = seed_exact_rows(ix, node_ids, row0, nrows, K, ex_scratch, ex_rows, out_ids, out_sc, st);
        }
    }
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    void *ptrs[] = {scratch, tau, tmp_sc, buf, cnt, ovf, ex_scratch};
    for (void *p : ptrs) if (p) (void)hipFree(p);
    if (rc != AP_OK) return rc;
    if (e != hipSuccess) { ap_set_error("seed k-NN failed: %s", hipGetErrorString(e)); return AP_EHIP; }
    return AP_OK;
}

extern "C" int ap_stage_seed_knn(const ap_index *ix, const int32_t *node_ids, int64_t nn, int32_t K, int32_t *out_ids,
                                 float *out_scores, void *stream) {
    AP_REQUIRE(ix && out_ids && out_scores, "NULL argument");
    AP_REQUIRE(K >= 1 && K <= 256, "K = %d must be in [1, 256]", K);
    if (!node_ids) nn = ix->docs.n;
    AP_REQUIRE(nn >= 0, "nn is negative");
    if (nn == 0) return AP_OK;
    return ap_seed_knn_impl(ix, node_ids, nn, K, out_ids, out_scores, (hipStream_t)stream, nullptr, ApWork());
}

int ap_entry_points_impl(const ap_index *ix, int32_t E, int32_t *out_entry, hipStream_t st, const ApWork &work) {
    float *own = nullptr, *sc = work.take<float>((size_t)E);
    if (!sc) { AP_TRY(ap_dev_alloc(&own, (size_t)E)); sc = own; }
    hipLaunchKernelGGL(k_select_rows, dim3(1), dim3(256), 0, st, ix->self_sim, ix->docs.n, E, (const int32_t *)nullptr,
                       (int64_t)0, 0, (int64_t)0, out_entry, sc);
    hipError_t e = hipGetLastError();
    if (own) {
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        (void)hipFree(own);
    }
    if (e != hipSuccess) { ap_set_error("entry point selection failed: %s", hipGetErrorString(e)); return AP_EHIP; }
    return AP_OK;
}

extern "C" int ap_stage_entry_points(const ap_index *ix, int32_t E, int32_t *out_entry, void *stream) {
    AP_REQUIRE(ix && out_entry, "NULL argument");
    AP_REQUIRE(E >= 1 && E <= 256, "E = %d must be in [1, 256]", E);
    return ap_entry_points_impl(ix, E, out_entry, (hipStream_t)stream, ApWork());
}

// =================================================================== S3: refinement round
#define AP_HT 4096
#define AP_MAXC 1280   // K + S*S <= 256 + 32*32

__device__ __forceinline__ bool ap_ht_insert(int32_t *ht, int32_t v) {
    uint32_t h = ((uint32_t)v * 2654435761u) >> 20;  // 12 bits
    for (;;) {
        const int32_t old = atomicCAS(&ht[h], -1, v);
        if (old == -1) return true;
        if (old == v) return false;
        h = (h + 1) & (AP_HT - 1);
    }
}
__device__ __forceinline__ bool ap_ht_has(const int32_t *ht, int32_t v) {
    uint32_t h = ((uint32_t)v * 2654435761u) >> 20;
    for (;;) {
        const int32_t cur = ht[h];
        if (cur == -1) return false;
        if (cur == v) return true;
        h = (h + 1) & (AP_HT - 1);
    }
}

// What a construction knows beyond the lists of a round and ap_stage_refine's callers do not: all NULL for a round on
// arbitrary lists, in which every candidate is scored in full.
struct ApRefineHints {
    // [nn]: no document outside the node's exact dense seed list has a dense part above this (the seed stage's K-th score, in
    // that stage's arithmetic); -inf where the seed list holds every other document
    const float *tau;
    // first round only: the scores the seed stage gave the lists' members, and how far they may be off (NULL: they are exact)
    const float *seed_sc, *seed_slack;
    // later rounds: the fused scores of the lists, and per node one bit for each of the first S list entries, set if the entry
    // was among the first S of the node's list one round ago
    const float *knn_sc;
    const uint32_t *known;
    uint32_t *known_out;   // the same bits for the lists this round returns
    // the lists of all documents, packed (NULL: not there)
    const uint32_t *pk;
    const uint2 *pk_at;
};

#define AP_RT_SPB 10   // look-up tables of the node's own lists: 1024 + 512 slots, at most a quarter full
#define AP_RT_TXB 9
// Records and dense rows a wave has on their way at once (three rounds on 200,000 bf16 documents: 2 and 1: 165 ms, 4 and 1:
// 153 ms, 4 and 2: 150 ms, 4 and 4: 150 ms, 8 and 2: 151 ms).
#define AP_RF_G 4
#define AP_RF_GD 2
#define AP_RF_GP 2               // packed records a group of 16 lanes has on their way, twice
#define AP_RF_BINS 512           // bins of the histogram that says what is scored first
#define AP_RF_TOP 0x40000000     // bit of a candidate that is among the first S entries of the node's own list (ids have 30 bits)
#define AP_RF_MORE(K) ((K) / 6)   // scored first beyond K (three rounds, 100,000 f32 and 200,000 bf16 documents: K / 4: 55.1 and 105.6 ms, K / 6: 53.8 and 105.1)
#define AP_RF_FIRST ((int32_t)0x80000000)   // bit of a candidate that is scored first

// One refinement round for one node.  What bounds it: the candidates' bytes (record and dense row) and the instructions
// of their look-ups, so the work is to touch fewer of them.  With the hints of a construction four things need no
// reading, and the lists stay what scoring everything gives, bit for bit:
//  - a candidate scored for this node before.  Lists only improve: whatever a round scored and did not keep ranks after K
//    documents that the list still holds or has exchanged for better ones, so it cannot enter again, and the per-path
//    lists were offered it.  That is the node's own list (its scores are at hand), and every neighbour's neighbour
//    w = N(v)[j] whose v was already among the first S of N(u) one round ago and w among the first S of N(v): both are
//    bits of `known`.
//  - the record of a candidate whose packed lists leave it out of reach: they are two fifths of its bytes, and give upper bounds of
//    its learned-sparse and lexical parts that lie some 2 % above them.
//  - the dense row of a candidate whose sparse and lexical parts leave it out of reach.  The seed lists are the exact
//    dense neighbours, so a document outside the node's list has a dense part of at most tau (plus the rounding of two
//    differently ordered sums, eps |u||w|) -- 0.1 where the norms alone would allow 1.
//  - what cannot beat the K best of this round.  A histogram of the candidates' bounds and the list's scores gives a line that
//    K + AP_RF_MORE(K) of them (7/6 K) reach; those are scored first, and a histogram of the scores gives T, which K of them reach and so the new
//    list's last entry does.  After that only candidates are scored whose bounds reach T, or the last entry of a per-path list (in the first
//    round, where those are empty: the P-th best of what was scored first).
// Phases: packed records of all candidates (16 lanes each, the next ones on their way; without packed lists the records themselves,
// a wave each), the histograms, records and dense rows of what is scored first, a thread per candidate decides about the others, their
// records and dense rows, the lists by counting what ranks before each entry.  With two workgroups a CU the short phases between the reads are
// what is left to hide: what a node needs of itself is requested at the start, one wave builds its tables while the others read, no
// list is sorted.  Three rounds on 200,000 documents of 1,024 bf16 columns: 308 ms with every candidate scored in full, 150 with the
// first and third of the above, 105 with all four, 89 with the short phases cut; 100,000 of 768 f32 columns: 202, 81, 54 and 49 ms
// (the first round reads 1.6 MB a node, 8 TB/s).
template <int DT, int NV>
__global__ __launch_bounds__(512, 4) void k_refine(ApVecs D, const uint2 *__restrict__ rec, const uint4 *__restrict__ meta, float wd,
                                                float ws, float wf, int32_t K, int32_t S, int32_t P,
                                                const int32_t *__restrict__ knn, const int32_t *__restrict__ sp_ids,
                                                const float *__restrict__ sp_sc, const int32_t *__restrict__ node_ids,
                                                int64_t nn, int64_t x0, int32_t *__restrict__ out_ids, float *__restrict__ out_sc,
                                                int32_t *__restrict__ out_sp_ids, float *__restrict__ out_sp_sc,
                                                unsigned long long *__restrict__ n_sims, ApRefineHints hint) {
    // 32 KB that serve three times: the hash set of the candidates; the node's weights by slot, a byte each; the histogram
    // and what else the decisions need, with the fused keys (AP_MAXC padded to a power of two) behind them
    __shared__ __attribute__((aligned(16))) uint32_t pool[AP_PK_SLOTS / 4];
    static_assert(AP_HT * 4 == 16384 && AP_PK_SLOTS == 32768, "the layout below");
    int32_t *ht = reinterpret_cast<int32_t *>(pool);
    uint32_t *hist = pool;                                                              // [AP_RF_BINS]
    uint2 *where = reinterpret_cast<uint2 *>(pool + AP_RF_BINS);                        // [AP_MAXC] records of need[]
    uint64_t (*better)[64] = reinterpret_cast<uint64_t (*)[64]>(pool + AP_RF_BINS + 2 * AP_MAXC);   // [3][64] candidates that beat a full per-path list's last entry
    static_assert(AP_RF_BINS * 4 + AP_MAXC * 8 + 3 * 64 * 8 <= AP_HT * 4, "what takes the hash set's place");
    uint64_t *keys = reinterpret_cast<uint64_t *>(pool + AP_HT);                        // [2048]
    __shared__ int32_t cand[AP_MAXC];
    // per candidate: before it is scored, where its record lies, the two lengths and the dense norm; then the norm and the
    // two list parts (or their bounds); then the three component scores of those that need[] names
    __shared__ float comp[3][AP_MAXC];
    __shared__ int32_t l_sp_idx[AP_A_CAP], l_tx_idx[AP_A_CAP];
    __shared__ float l_sp_val[AP_A_CAP], l_tx_val[AP_A_CAP];
    __shared__ uint64_t oldk[3][32];
    __shared__ __attribute__((aligned(16))) uint64_t qtab[(1 << AP_RT_SPB) + (1 << AP_RT_TXB)];
    __shared__ uint16_t need[AP_MAXC];        // from the front: candidates that are scored in full; from the back: those whose list parts alone are
    __shared__ int32_t first_ids[32];
    __shared__ int32_t s_cnt, s_seed[2], s_nk, s_need, s_lists, s_next;
    __shared__ uint32_t s_lo, s_hi, s_line, s_known;
    __shared__ float s_last[3];
    const int64_t x = x0 + blockIdx.x;   // the launch covers nodes x0 .. x0 + gridDim.x of the nn
    const int64_t u = node_ids ? (int64_t)node_ids[x] : x;
    const int lane = threadIdx.x & 63, wave = ap_wave_id();
    constexpr int NW = 8;
    const bool fast = hint.tau != nullptr, later = hint.knn_sc != nullptr;   // uniform
    // what later phases need of the node itself is requested now: its packed lists (a unit a thread, four threads a unit), the first
    // neighbours of its list, its per-path lists
    uint2 own_at = make_uint2(0, 0);
    ApPkUnit own_unit = {0, 0, 0};
    float own_sp = 0.f, own_tx = 0.f;
    int32_t own_entries = 0;
    bool packed = hint.pk != nullptr;   // uniform
    if (packed) {
        own_at = hint.pk_at[u];
        const ApPkUnit *r = reinterpret_cast<const ApPkUnit *>(hint.pk + (size_t)own_at.x * (AP_PK_LINE / 4));
        own_entries = 4 * (int32_t)((own_at.y & 0xffffu) + (own_at.y >> 16));
        own_unit = r[(int)threadIdx.x < own_entries ? 1 + ((int)threadIdx.x >> 2) : 0];
        own_sp = __uint_as_float(r[0].w); own_tx = __uint_as_float(r[0].s01);
        packed = own_sp < INFINITY && own_tx < INFINITY;   // a list without a scale (a negative value) has no bounds
    }
    int32_t old_id = -1;
    float old_sc = 0.f;
    if (wave < 3 && lane < P) {
        old_id = sp_ids[((int64_t)wave * D.n + u) * P + lane];
        old_sc = sp_sc[((int64_t)wave * D.n + u) * P + lane];
    }
    const ApLists a = ap_stage_lists(D, u, l_sp_idx, l_sp_val, l_tx_idx, l_tx_val, AP_A_CAP);
    float qa[NV * ApDense<DT>::EPC];
    ap_load_aside<DT, NV, DT>(D.dense, u, D.dim, qa);
    for (int i = threadIdx.x; i < AP_HT / 4; i += blockDim.x) reinterpret_cast<int4 *>(ht)[i] = make_int4(-1, -1, -1, -1);
    if (threadIdx.x == 0) { s_cnt = 0; s_nk = 0; s_need = 0; s_lists = 0; s_next = 0; s_known = 0u; s_lo = 0xffffffffu; s_hi = 0u; s_last[0] = s_last[1] = s_last[2] = -INFINITY; }
    __syncthreads();
    // the node's own lists as bucket tables with a hash multiplier of their own (the usual case: one 16-byte read per
    // look-up, as in the search); lists that are longer, or that no multiplier fits, are searched where they lie.  One wave
    // builds them; they are there after the next barrier.
    auto build_tables = [&]() {
        const bool fits = a.sp_n <= (1 << AP_RT_SPB) / 4 && a.tx_n <= (1 << AP_RT_TXB) / 4;
        const int32_t s0 = fits ? ap_bucket_build<4>(a.sp_idx, a.sp_val, a.sp_n, qtab, AP_RT_SPB) : -1;
        const int32_t s1 = fits ? ap_bucket_build<2>(a.tx_idx, a.tx_val, a.tx_n, qtab + (1 << AP_RT_SPB), AP_RT_TXB) : -1;
        if (lane == 0) { s_seed[0] = s0; s_seed[1] = s1; }
    };
    if (!packed && wave == NW - 1) build_tables();
    // a candidate, and where its record lies and how long it is, so that the scoring loop starts its loads without a round trip of its own
    auto put_candidate = [&](int32_t t, int32_t v, int32_t mark) {
        cand[t] = v | mark;
        if (packed) {
            const uint2 m = hint.pk_at[v];
            comp[0][t] = __uint_as_float(m.x); comp[1][t] = __uint_as_float(m.y);
        } else {
            const uint4 m = meta[v];
            comp[0][t] = __uint_as_float(m.x); comp[1][t] = __uint_as_float(m.y); comp[2][t] = __uint_as_float(m.z);
        }
    };
    // candidates: the node's own list (in later rounds its scores are at hand: it only stays out of the candidates) ...
    const int32_t sl = S < K ? S : K;
    for (int32_t s = threadIdx.x; s < K; s += blockDim.x) {
        const int32_t v = knn[u * K + s];
        if (s < sl) first_ids[s] = v;
        if (v >= 0 && v != (int32_t)u && ap_ht_insert(ht, v) && !later) {
            const int32_t at = atomicAdd(&s_cnt, 1);
            put_candidate(fast ? s : at, v, s < sl ? AP_RF_TOP : 0);   // a seed list's members are distinct and lead the list: candidate s is member s
        }
    }
    __syncthreads();
    const int32_t n_own = ap_uniform_i32(s_cnt);   // candidates of the node's own list (0 in later rounds)
    __syncthreads();
    // ... and the first S neighbours of the first S neighbours
    {
        const uint32_t mine = later ? hint.known[u] : 0u;
        for (int32_t s = threadIdx.x; s < sl * sl; s += blockDim.x) {
            const int32_t i = s / sl, j = s % sl;
            const int32_t p = first_ids[i];
            if (p < 0) continue;
            const int32_t v = knn[(int64_t)p * K + j];
            if ((mine >> i) & 1u && (hint.known[p] >> j) & 1u) continue;   // scored for this node in an earlier round
            if (v >= 0 && v != (int32_t)u && ap_ht_insert(ht, v)) put_candidate(atomicAdd(&s_cnt, 1), v, 0);
        }
    }
    __syncthreads();
    const int32_t cnt = ap_uniform_i32(s_cnt);
    // the per-path lists so far, in keys (entries scored again in a round that scores everything are left out: there the
    // caller's scores need not be this kernel's)
    if (wave < 3) {
        const bool have = old_id >= 0 && (fast || !ap_ht_has(ht, old_id));
        const uint64_t hm = __ballot(have);
        if (lane < 32) oldk[wave][lane] = 0ull;
        ap_wave_sync();
        if (have) oldk[wave][__popcll(hm & ((1ull << lane) - 1ull))] = ap_make_key(old_sc, old_id, 1u);
    }
    __syncthreads();   // the hash set is done with
    bool use_tab = false;   // uniform
    uint32_t msp = 0, mtx = 0;
    auto take_tables = [&]() {
        const int32_t seed0 = ap_uniform_i32(s_seed[0]), seed1 = ap_uniform_i32(s_seed[1]);
        use_tab = seed0 >= 0 && seed1 >= 0;
        if (use_tab) { msp = ap_seed_mult(seed0); mtx = ap_seed_mult(seed1); }
    };
    if (!packed) take_tables();
    // the sparse and lexical parts of all candidates, or bounds of them
    if (packed) {
        for (int32_t i = threadIdx.x; i < AP_PK_SLOTS / 16; i += blockDim.x) reinterpret_cast<uint4 *>(pool)[i] = make_uint4(0, 0, 0, 0);
        __syncthreads();
        auto put_own = [&](const ApPkUnit &d, int32_t i) {
            const uint32_t at = ((i & 2 ? d.s23 : d.s01) >> (16 * (i & 1))) & 0xffffu, w = (d.w >> (8 * (i & 3))) & 255u;
            if (w) atomicOr(&pool[at >> 2], w << (8 * (at & 3u)));   // two terms of one slot: at least the larger of them
        };
        const ApPkUnit *own = reinterpret_cast<const ApPkUnit *>(hint.pk + (size_t)own_at.x * (AP_PK_LINE / 4));
        if ((int)threadIdx.x < own_entries) put_own(own_unit, threadIdx.x);
        for (int32_t i = threadIdx.x + 512; i < own_entries; i += 512) put_own(own[1 + (i >> 2)], i);
        __syncthreads();
        constexpr int G = AP_RF_GP, U = 3;
        const AP_LDS uint8_t *tab = (const AP_LDS uint8_t *)pool;
        const int sub = lane >> 4, l16 = lane & 15;
        // What a sum of the scoring kernels may come out above the exact one: a lane adds what the lists share one after the other, each addition
        // rounds up by at most 2^-24 of the sum so far, and the node's list is the longest that two can share; 1e-5 for the six additions over the
        // lanes and what the products here round off.  (A fixed 4e-5 for all of it held up to some 46,000 entries, 738 a lane, of the 65,535 that are taken.)
        own_sp *= fmaf(6e-8f, 4.f * (float)(own_at.y & 0xffffu), 1.00001f);
        own_tx *= fmaf(6e-8f, 4.f * (float)(own_at.y >> 16), 1.00001f);
        if (wave == NW - 1) build_tables();   // the others begin without it: 4 G candidates at a time go to the wave that asks
        auto ask = [&]() {
            int32_t i = 0;
            if (lane == 0) i = atomicAdd(&s_next, 4 * G);
            return ap_uniform_i32(i);
        };
        ApPkUnit d[2][G][U];
        uint32_t len[2][G];
        auto load = [&](int32_t i0, ApPkUnit (&d)[G][U], uint32_t (&len)[G]) {
#pragma unroll
            for (int g = 0; g < G; g++) {
                const int32_t i = i0 + 4 * g + sub;
                const uint32_t line = i < cnt ? __float_as_uint(comp[0][i]) : own_at.x;   // past the end: unit 0 of the node's own record, for nothing
                len[g] = i < cnt ? __float_as_uint(comp[1][i]) : 0u;
                const ApPkUnit *r = reinterpret_cast<const ApPkUnit *>(hint.pk + (size_t)line * (AP_PK_LINE / 4));
                const int32_t units = 1 + (int32_t)((len[g] & 0xffffu) + (len[g] >> 16));
#pragma unroll
                for (int j = 0; j < U; j++) d[g][j] = r[l16 + 16 * j < units ? l16 + 16 * j : 0];
            }
        };
        auto sum = [&](int32_t i0, const ApPkUnit (&d)[G][U], const uint32_t (&len)[G]) {
#pragma unroll
            for (int g = 0; g < G; g++) {
                const int32_t i = i0 + 4 * g + sub, nsp = (int32_t)(len[g] & 0xffffu), units = 1 + nsp + (int32_t)(len[g] >> 16);
                uint32_t ps = 0, pf = 0;
                auto add = [&](const ApPkUnit &e, int32_t at) {
                    const uint32_t p = ap_pk_dot(tab, e);
                    ps += at >= 1 && at <= nsp ? p : 0u;
                    pf += at > nsp && at < units ? p : 0u;
                };
#pragma unroll
                for (int j = 0; j < U; j++) add(d[g][j], l16 + 16 * j);
                if (__any(units > 16 * U)) {
                    const ApPkUnit *r = reinterpret_cast<const ApPkUnit *>(hint.pk + (size_t)(i < cnt ? __float_as_uint(comp[0][i]) : own_at.x) * (AP_PK_LINE / 4));
                    for (int32_t at = l16 + 16 * U; __any(at < units); at += 16) add(r[at < units ? at : 0], at);
                }
                float fs = (float)ps, ff = (float)pf;
                fs += ap_dpp<0xB1>(fs); ff += ap_dpp<0xB1>(ff);
                fs += ap_dpp<0x4E>(fs); ff += ap_dpp<0x4E>(ff);
                fs += ap_dpp<0x141>(fs); ff += ap_dpp<0x141>(ff);
                fs += ap_dpp<0x140>(fs); ff += ap_dpp<0x140>(ff);
                if (l16 == 0 && i < cnt) {   // unit 0 is the first thing lane 0 of a group loaded
                    comp[0][i] = __uint_as_float(d[g][0].s23);
                    comp[1][i] = fs * (own_sp * __uint_as_float(d[g][0].w));
                    comp[2][i] = ff * (own_tx * __uint_as_float(d[g][0].s01));
                }
            }
        };
        int32_t i0 = ask();
        load(i0, d[0], len[0]);
        while (i0 < cnt) {   // the next candidates' units travel while these are summed
            const int32_t i1 = ask();
            load(i1, d[1], len[1]);
            sum(i0, d[0], len[0]);
            if (i1 >= cnt) break;
            i0 = ask();
            load(i0, d[0], len[0]);
            sum(i1, d[1], len[1]);
        }
        __syncthreads();
        take_tables();
    } else if (use_tab) {
        constexpr int G = AP_RF_G;
        for (int32_t i0 = wave; i0 < cnt; i0 += G * NW) {
            uint2 xs[G][2], xt[G][1];
            const uint2 *r[G];
            int32_t spn[G], txn[G];
            float norm[G];
#pragma unroll
            for (int g = 0; g < G; g++) {
                const int32_t i = i0 + NW * g < cnt ? i0 + NW * g : i0;   // past the end: the first one again, for nothing
                const uint32_t my = ap_uniform_u32(__float_as_uint(comp[1][i]));
                r[g] = rec + ap_uniform_u32(__float_as_uint(comp[0][i]));
                norm[g] = comp[2][i];
                spn[g] = (int32_t)(my & 0xffffu); txn[g] = (int32_t)(my >> 16);
                ap_rec_load_raw<2, 1>(r[g], spn[g], txn[g], xs[g], xt[g]);
            }
#pragma unroll
            for (int g = 0; g < G; g++) {
                if (i0 + NW * g >= cnt) break;   // uniform
                int32_t si[2], ti[1];
                float sv[2], tv[1], ss, sf;
                ap_rec_decode<2, 1>(xs[g], xt[g], spn[g], txn[g], si, sv, ti, tv);
                ap_rec_reduce_bucket<2, 1, AP_RT_SPB, AP_RT_TXB>(r[g], (const AP_LDS uint64_t *)qtab, (const AP_LDS uint64_t *)(qtab + (1 << AP_RT_SPB)),
                                                                 msp, mtx, spn[g], txn[g], si, sv, ti, tv, ss, sf);
                const int32_t i = i0 + NW * g;
                if (lane == 0) { comp[0][i] = norm[g]; comp[1][i] = ss; comp[2][i] = sf; }
            }
        }
    } else {
        for (int32_t i = wave; i < cnt; i += NW) {
            const uint32_t my = ap_uniform_u32(__float_as_uint(comp[1][i]));
            const uint2 *r = rec + ap_uniform_u32(__float_as_uint(comp[0][i]));
            const float norm = comp[2][i];
            const int32_t spn = (int32_t)(my & 0xffffu), txn = (int32_t)(my >> 16);
            int32_t si[2], ti[1];
            float sv[2], tv[1], ss, sf;
            ap_rec_load<2, 1>(r, spn, txn, si, sv, ti, tv);
            ap_rec_reduce_lists<2, 1>(r, a, spn, txn, si, sv, ti, tv, ss, sf);
            if (lane == 0) { comp[0][i] = norm; comp[1][i] = ss; comp[2][i] = sf; }
        }
    }

    auto list_parts = [&](const uint2 *r, int32_t spn, int32_t txn, const uint2 *xs, const uint2 *xt, float &ss, float &sf) {
        int32_t si[2], ti[1];
        float sv[2], tv[1];
        ap_rec_decode<2, 1>(xs, xt, spn, txn, si, sv, ti, tv);
        if (use_tab)
            ap_rec_reduce_bucket<2, 1, AP_RT_SPB, AP_RT_TXB>(r, (const AP_LDS uint64_t *)qtab, (const AP_LDS uint64_t *)(qtab + (1 << AP_RT_SPB)), msp, mtx, spn,
                                                             txn, si, sv, ti, tv, ss, sf);
        else
            ap_rec_reduce_lists<2, 1>(r, a, spn, txn, si, sv, ti, tv, ss, sf);
    };
    // the candidates need[d0 .. d1) in full, a wave each: dense rows, and the records where only bounds of the list parts are known
    // (where[] says where they lie)
    auto score = [&](int32_t d0, int32_t d1) {
        // One candidate at a time where a lane holds 32 columns of the node: two do not fit the registers beside them (60,000 documents of 2,048 bf16
        // columns, spilling 6 registers 74.4 ms, one at a time 74.0).
        constexpr int G = DT == AP_BF16 && NV >= 4 ? 1 : AP_RF_GD;
        for (int32_t e0 = d0 + wave; e0 < d1; e0 += G * NW) {
            uint4 raw[G][NV];
            uint2 xs[G][2], xt[G][1];
            const uint2 *r[G];
            int32_t cand_i[G], cv[G], spn[G], txn[G];
#pragma unroll
            for (int g = 0; g < G; g++) {
                const int32_t d = e0 + NW * g < d1 ? e0 + NW * g : e0;
                cand_i[g] = ap_uniform_i32(need[d]);
                cv[g] = ap_uniform_i32(cand[cand_i[g]]) & ~AP_RF_FIRST;
                if (packed) {
                    const uint2 m = where[d];
                    const uint32_t my = ap_uniform_u32(m.y);
                    r[g] = rec + ap_uniform_u32(m.x);
                    spn[g] = (int32_t)(my & 0xffffu); txn[g] = (int32_t)(my >> 16);
                    ap_rec_load_raw<2, 1>(r[g], spn[g], txn[g], xs[g], xt[g]);
                }
                ap_dense_load_raw<DT, NV>(D, cv[g] & ~AP_RF_TOP, raw[g]);
            }
#pragma unroll
            for (int g = 0; g < G; g++) {
                if (e0 + NW * g >= d1) break;   // uniform
                const int32_t i = cand_i[g];
                float ss, sf;
                if (packed) {
                    list_parts(r[g], spn[g], txn[g], xs[g], xt[g], ss, sf);
                } else { ss = comp[1][i]; sf = comp[2][i]; }
                const float sd = ap_dense_dot_raw<DT, NV>(D, qa, raw[g]);
                if (lane == 0) {
                    const float f = ap_fuse(wd, ws, wf, sd, ss, sf);
                    comp[0][i] = sd;
                    if (packed) { comp[1][i] = ss; comp[2][i] = sf; }
                    keys[atomicAdd(&s_nk, 1)] = ap_make_key(f, cv[g] & ~AP_RF_TOP, cv[g] & AP_RF_TOP ? 1u : 0u);
                }
            }
        }
    };
    // the list parts alone of the n candidates at the end of need[]
    auto score_lists = [&](int32_t n) {
        for (int32_t e0 = wave; e0 < n; e0 += 2 * NW) {
            uint2 xs[2][2], xt[2][1];
            const uint2 *r[2];
            int32_t spn[2], txn[2];
#pragma unroll
            for (int g = 0; g < 2; g++) {
                const uint2 m = where[AP_MAXC - 1 - (e0 + NW * g < n ? e0 + NW * g : e0)];
                const uint32_t my = ap_uniform_u32(m.y);
                r[g] = rec + ap_uniform_u32(m.x);
                spn[g] = (int32_t)(my & 0xffffu); txn[g] = (int32_t)(my >> 16);
                ap_rec_load_raw<2, 1>(r[g], spn[g], txn[g], xs[g], xt[g]);
            }
#pragma unroll
            for (int g = 0; g < 2; g++) {
                if (e0 + NW * g >= n) break;   // uniform
                float ss, sf;
                list_parts(r[g], spn[g], txn[g], xs[g], xt[g], ss, sf);
                const int32_t i = need[AP_MAXC - 1 - (e0 + NW * g)];
                if (lane == 0) { comp[1][i] = ss; comp[2][i] = sf; }
            }
        }
    };
    // the list so far takes its place among the keys (the records' bounds were the last use of its space)
    if (later) {
        for (int32_t s = threadIdx.x; s < K; s += blockDim.x) {
            const int32_t v = knn[u * K + s];
            if (v >= 0 && v != (int32_t)u) keys[atomicAdd(&s_nk, 1)] = ap_make_key(hint.knn_sc[u * K + s], v, s < sl ? 1u : 0u);
        }
    }
    if (!fast) {
        for (int32_t t = threadIdx.x; t < cnt; t += blockDim.x) need[t] = (uint16_t)t;
        if (threadIdx.x == 0) s_need = cnt;
        __syncthreads();
        score(0, cnt);
    } else {
        if (threadIdx.x < AP_RF_BINS) hist[threadIdx.x] = 0;
        __syncthreads();
        const int32_t n_old = ap_uniform_i32(s_nk);
        // Bounds of the dense part of candidate t with norm |w|: the seed stage's score (members of the seed list, whose
        // scores the first round has) or its K-th score (documents outside it), plus eps |u||w|: each of the two differently
        // ordered fp32 sums is off by at most dim 2^-24 |u||w| from the exact product; twice that for each is allowed.
        const float un = __uint_as_float(meta[u].z), eps = 4.f * (float)D.dim * 5.9604645e-8f;
        const float tau = hint.tau[u], seed_off = hint.seed_slack ? hint.seed_slack[u] : 0.f;
        auto bound = [&](int32_t t, float &bd, float &bf) {   // upper bounds of the dense part and of the fused score
            const float nb = un * comp[0][t] * 1.0001f, ss = comp[1][t], sf = comp[2][t];
            const float most = t < n_own ? hint.seed_sc[u * K + t] + seed_off : tau;   // n_own is 0 in later rounds
            bd = most - most == 0.f ? fminf(nb, most + eps * nb) : nb;
            const float lift = wd >= 0.f ? wd * bd : -wd * nb;
            bf = fmaf(wf, sf, ws * ss) + lift + 1e-5f * (fabsf(ws * ss) + fabsf(wf * sf) + fabsf(wd) * nb);
        };
        float T = later && n_old == K ? hint.knn_sc[u * K + K - 1] : -INFINITY;
        // the last entries of the per-path lists, or lower bounds of what they will be
        float last[3] = {-INFINITY, -INFINITY, -INFINITY};
        if (later) {
#pragma unroll
            for (int p = 0; p < 3; p++)
                if (oldk[p][P - 1]) last[p] = ap_key_score(oldk[p][P - 1]);
        } else if (P <= K && n_own >= P && wave == 0) {   // the P best of the seed list by their seed scores are at least this good
            float lo = INFINITY;
            if (lane < P) {
                const int32_t v = knn[u * K + lane];
                lo = v >= 0 ? hint.seed_sc[u * K + lane] - seed_off - eps * un * __uint_as_float(meta[v].z) * 1.0001f : -INFINITY;
            }
            for (int o = 32; o > 0; o >>= 1) lo = fminf(lo, __shfl_xor(lo, o, 64));
            if (lane == 0) s_last[0] = lo;
        }
        // What is scored first: everything from a line on that at least K scores and bounds reach, and AP_RF_MORE(K) more, since a bound
        // may lie far above its score (from T on, where the list is full).
        uint32_t mine[3] = {0u, 0u, 0u}, lo = 0xffffffffu, hi = 0u;
        static_assert(AP_MAXC <= 3 * 512, "candidates of a thread");
#pragma unroll
        for (int k = 0; k < 3; k++) {
            const int32_t t = threadIdx.x + 512 * k;
            if (t >= cnt) continue;
            float bd, bf;
            bound(t, bd, bf);
            if (bf < T) continue;
            const uint32_t o = ap_f2ord(bf);
            mine[k] = o ? o : 1u;   // 0: not to be scored first (no bound of a score has the lowest code)
            lo = min(lo, mine[k]); hi = max(hi, mine[k]);
        }
        for (int32_t t = threadIdx.x; t < n_old; t += 512) {
            const uint32_t o = (uint32_t)(keys[t] >> 32);
            lo = min(lo, o); hi = max(hi, o);
        }
        for (int o = 32; o > 0; o >>= 1) {
            lo = min(lo, (uint32_t)__shfl_xor((int)lo, o, 64));
            hi = max(hi, (uint32_t)__shfl_xor((int)hi, o, 64));
        }
        if (lane == 0) { atomicMin(&s_lo, lo); atomicMax(&s_hi, hi); }
        __syncthreads();
        lo = ap_uniform_u32(s_lo); hi = ap_uniform_u32(s_hi);
        const uint32_t least = lo;
        if (hi > lo && hi - lo > (4u << 23)) lo = hi - (4u << 23);   // four octaves (one bound may lie far above all scores): what lies below is counted in the first bin
        auto width = [](uint32_t lo, uint32_t hi) { int sh = 0; while (lo < hi && ((hi - lo) >> sh) >= AP_RF_BINS) sh++; return sh; };
        const int sh = width(lo, hi);
        auto count = [&](uint32_t o, uint32_t lo, uint32_t hi, int sh) { atomicAdd(&hist[(min(max(o, lo), hi) - lo) >> sh], 1u); };
        // wave 0: the lower edge of the bin from which on at least `many` are counted (of the first bin: 0), 1 where all are fewer, but
        // `enough`; 0xffffffff: fewer than that
        auto edge = [&](uint32_t many, uint32_t enough, uint32_t lo, int sh) {
            static_assert(AP_RF_BINS == 512, "eight bins a lane");
            const uint4 h = reinterpret_cast<const uint4 *>(hist)[2 * (63 - lane) + 1], l = reinterpret_cast<const uint4 *>(hist)[2 * (63 - lane)];   // from the top: lane 0 has the last eight
            const uint32_t bin[8] = {h.w, h.z, h.y, h.x, l.w, l.z, l.y, l.x};
            uint32_t n = 0;
#pragma unroll
            for (int i = 0; i < 8; i++) n += bin[i];
            uint32_t upto = n;
            for (int o = 1; o < 64; o <<= 1) { const uint32_t up = (uint32_t)__shfl_up((int)upto, o, 64); if (lane >= o) upto += up; }
            const uint64_t m = __ballot(upto >= many);
            if (m == 0ull) { if (lane == 63) s_line = upto >= enough ? 1u : 0xffffffffu; }
            else if (lane == (int)__ffsll((unsigned long long)m) - 1) {
                uint32_t above = upto - n, b = 8u * (64 - lane);
#pragma unroll
                for (int i = 0; i < 8; i++) {
                    b -= above < many ? 1u : 0u;
                    above += bin[i];
                }
                s_line = b ? lo + (b << sh) : 0u;
            }
        };
        auto find_line = [&](uint32_t lo, uint32_t hi, int sh) {
#pragma unroll
            for (int k = 0; k < 3; k++)
                if (mine[k]) count(mine[k], lo, hi, sh);
            for (int32_t t = threadIdx.x; t < n_old; t += 512) count((uint32_t)(keys[t] >> 32), lo, hi, sh);
            __syncthreads();
            if (wave == 0) edge((uint32_t)(K + AP_RF_MORE(K)), (uint32_t)K, lo, sh);
            __syncthreads();
            if (threadIdx.x < AP_RF_BINS) hist[threadIdx.x] = 0;
            return ap_uniform_u32(s_line);
        };
        uint32_t line = find_line(lo, hi, sh);
        // Where the line lies below the four octaves (a near duplicate far above all others, or scores that a negative weight takes
        // below zero) the bins are laid over what is left, then over the one of them that it lies in.  Else all would be scored first:
        // 30,000 documents of 768 f32 columns, every one there twice, are built in 66.0 ms then, in 55.5 so; a sparse weight of -0.3: 58.5 and 48.2.
        const bool below = line == 0u && lo > least;   // uniform
        if (below) {
            uint32_t from = least, to = lo;
            for (;;) {
                const int w = width(from, to);
                __syncthreads();
                line = max(find_line(from, to, w), from);
                if (w <= 14) break;
                from = line; to = min(to, from + ((1u << w) - 1u));
            }
        }
        if (line != 0xffffffffu) {
#pragma unroll
            for (int k = 0; k < 3; k++) {
                const int32_t t = threadIdx.x + 512 * k;
                if (mine[k] && mine[k] >= line) {
                    const int32_t at = atomicAdd(&s_need, 1);
                    need[at] = (uint16_t)t;
                    cand[t] |= AP_RF_FIRST;
                    if (packed) { const uint4 m = meta[cand[t] & (AP_RF_TOP - 1)]; where[at] = make_uint2(m.x, m.y); }
                }
            }
        }
        __syncthreads();
        const int32_t n_first = ap_uniform_i32(s_need);
        score(0, n_first);
        __syncthreads();
        if (below) {   // T: the K-th best score so far
            const int32_t nk = ap_uniform_i32(s_nk);
            for (int32_t t = threadIdx.x; t < nk; t += 512) {
                const uint64_t key = keys[t];
                int32_t rank = 0;
                for (int32_t j = 0; j < nk; j++) rank += keys[j] > key ? 1 : 0;
                if (rank == K - 1) s_line = (uint32_t)(key >> 32);
            }
            __syncthreads();
            T = fmaxf(T, ap_ord2f(ap_uniform_u32(s_line)));
        } else if (line != 0xffffffffu) {   // T: the lower edge of the bin that it lies in
            const int32_t nk = ap_uniform_i32(s_nk);
            for (int32_t t = threadIdx.x; t < nk; t += 512) {
                const uint32_t o = (uint32_t)(keys[t] >> 32);
                if (o >= lo) count(o, lo, hi, sh);
            }
            __syncthreads();
            if (wave == 0) edge((uint32_t)K, 0xffffffffu, lo, sh);
            __syncthreads();
            const uint32_t at = ap_uniform_u32(s_line);
            if (at != 0xffffffffu) T = fmaxf(T, ap_ord2f(at ? at : lo));
        }
        if (!later) {
            // first round: the P-th best of the lanes' best list parts of what was scored first, so at most the P-th best of all
            if (wave == 1 || wave == 2) {
                uint32_t best = 0;
                for (int32_t e = lane; e < n_first; e += 64) best = max(best, ap_f2ord(comp[wave][need[e]]));
                int32_t rank = 0;
                for (int j = 0; j < 64; j++) {
                    const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)best, j);
                    rank += o > best || (o == best && j < lane) ? 1 : 0;
                }
                if (rank == P - 1) s_last[wave] = best ? ap_ord2f(best) : -INFINITY;
            }
            __syncthreads();
            last[0] = P <= K && n_own >= P ? s_last[0] : -INFINITY;
            last[1] = s_last[1]; last[2] = s_last[2];
        }
        for (int32_t t = threadIdx.x; t < cnt; t += blockDim.x) {
            if (cand[t] < 0) { cand[t] &= ~AP_RF_FIRST; continue; }
            float bd, bf;
            bound(t, bd, bf);
            const bool whole = !(bf < T) || !(bd < last[0]);
            if (whole || !(comp[1][t] < last[1]) || !(comp[2][t] < last[2])) {
                const int32_t at = whole ? atomicAdd(&s_need, 1) : AP_MAXC - 1 - atomicAdd(&s_lists, 1);
                need[at] = (uint16_t)t;
                if (packed) { const uint4 m = meta[cand[t] & ~AP_RF_TOP]; where[at] = make_uint2(m.x, m.y); }
            }
        }
        __syncthreads();
        score(n_first, ap_uniform_i32(s_need));
        if (packed) score_lists(ap_uniform_i32(s_lists));
    }
    __syncthreads();
    // Three waves make the per-path lists: the best P by each single similarity among what was scored and the previous list
    // (with hints, what was not ranks after a full list's last entry, or after P of what was scored first).
    const int32_t nk = ap_uniform_i32(s_nk), n_whole = ap_uniform_i32(s_need);
    if (threadIdx.x >= 510 && n_sims) atomicAdd(n_sims + (threadIdx.x - 510), (unsigned long long)(threadIdx.x == 510 ? cnt : n_whole));   // measurement: similarities of this node and round, those computed in full
    if (wave < 3) {
        const int p = wave;
        const int32_t nold = (int32_t)__popcll(__ballot(lane < 32 && oldk[p][lane & 31] != 0ull));
        auto cand_key = [&](int32_t e) {
            const int32_t t = need[e < n_whole ? e : AP_MAXC - 1 - (e - n_whole)];
            return ap_make_key(comp[p][t], cand[t] & (AP_RF_TOP - 1), 1u);
        };
        const int32_t n_scored = n_whole + (p ? ap_uniform_i32(s_lists) : 0);
        auto put = [&](int32_t r, uint64_t key) {
            out_sp_ids[((int64_t)p * nn + x) * P + r] = key ? ap_key_id(key) : -1;
            out_sp_sc[((int64_t)p * nn + x) * P + r] = key ? ap_key_score(key) : -INFINITY;
        };
        // what can enter: what beats a full list's last entry, or reaches the line that P of the candidates do; usually few enough for one key a lane
        const uint64_t full = fast && nold == P ? oldk[p][P - 1] : 0ull;
        const float line = fast && !later ? s_last[p] : -INFINITY;
        int32_t nb = 0;
        for (int32_t t0 = 0; t0 < n_scored && nb + nold <= 64; t0 += 64) {
            const uint64_t key = t0 + lane < n_scored ? cand_key(t0 + lane) : 0ull;
            const bool in = key > full && !(ap_key_score(key) < line);
            const uint64_t m = __ballot(in);
            const int32_t at = nb + (int32_t)__popcll(m & ((1ull << lane) - 1ull));
            if (in && at < 64) better[p][at] = key;
            nb += (int32_t)__popcll(m);
        }
        ap_wave_sync();
        const int32_t n = nb + nold;
        if (n <= 64) {
            uint64_t key = lane < nb ? better[p][lane] : lane < n ? oldk[p][lane - nb] : 0ull;
            for (int32_t j = 0; j < nold; j++)   // a candidate met once more may be on the list already
                if (lane < nb && key == oldk[p][j]) key = 0ull;
            const int kh = (int)(key >> 32), kl = (int)(uint32_t)key;
            int32_t rank = 0;
            for (int32_t j = 0; j < n; j++) {
                const uint64_t other = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane(kh, j) << 32) | (uint32_t)__builtin_amdgcn_readlane(kl, j);
                rank += other > key ? 1 : 0;
            }
            if (key && rank < P) put(rank, key);
            if (lane >= (int)__popcll(__ballot(key != 0ull)) && lane < P) put(lane, 0ull);
        } else {   // every lane keeps its share of the keys and the P best are drawn one after the other by wave-wide maxima
            constexpr int PER = (AP_MAXC + 32 + 63) / 64;
            uint64_t key[PER], prev = ~0ull;
#pragma unroll
            for (int j = 0; j < PER; j++) {
                const int32_t t = j * 64 + lane;
                key[j] = t < n_scored ? cand_key(t) : (t < n_scored + nold ? oldk[p][t - n_scored] : 0ull);
            }
            for (int32_t r = 0; r < P; r++) {
                uint64_t best = 0;
#pragma unroll
                for (int j = 0; j < PER; j++)
                    if (key[j] < prev && key[j] > best) best = key[j];
                for (int o = 32; o > 0; o >>= 1) {
                    const uint64_t other = __shfl_xor(best, o, 64);
                    best = other > best ? other : best;
                }
                if (lane == 0) put(r, best);
                prev = best;   // 0 once exhausted: nothing ranks after it
            }
        }
    } else {
        // The others the top-K under the fused score.  The keys are all different (a key carries its id), so a key's place is the number
        // of larger ones; what was left out above ranks after K of them.  (By a bitonic sort this phase took 7.5 of a node's 90 us.)
        for (int32_t t = threadIdx.x - 192; t < nk; t += 320) {
            const uint64_t key = keys[t];
            int32_t rank = 0;
            for (int32_t j = 0; j + 1 < nk; j += 2) {
                const ulonglong2 o = *reinterpret_cast<const ulonglong2 *>(keys + j);
                rank += (o.x > key ? 1 : 0) + (o.y > key ? 1 : 0);
            }
            if (nk & 1) rank += keys[nk - 1] > key ? 1 : 0;
            if (rank < K) {
                out_ids[x * K + rank] = ap_key_id(key);
                out_sc[x * K + rank] = ap_key_score(key);
                if (rank < sl && (key & 1ull)) atomicOr(&s_known, 1u << rank);
            }
        }
        for (int32_t t = nk + threadIdx.x - 192; t < K; t += 320) { out_ids[x * K + t] = -1; out_sc[x * K + t] = -INFINITY; }
    }
    if (hint.known_out) {
        __syncthreads();
        if (threadIdx.x == 0) hint.known_out[x] = s_known;
    }
}

// One round for the nn listed nodes; see k_refine for what the hints are.
int ap_refine_round(const ap_index *ix, int32_t K, int32_t S, int32_t P, const int32_t *knn_ids, const int32_t *sp_ids, const float *sp_sc,
                    const int32_t *node_ids, int64_t nn, int32_t *out_ids, float *out_sc, int32_t *out_sp_ids, float *out_sp_sc,
                    const ApRefineHints &hint, hipStream_t st) {
    const float *w = ix->params.build_w;
    const int64_t slice = AP_MAX_LAUNCH_THREADS / 512;   // a launch holds fewer than 2^32 threads
    for (int64_t x0 = 0; x0 < nn; x0 += slice) {
        const int64_t cn = std::min<int64_t>(slice, nn - x0);
        AP_DISPATCH_DENSE(ix->dtype, ix->docs.dim,
                          hipLaunchKernelGGL((k_refine<DT, NV>), dim3((unsigned)cn), dim3(512), 0, st, ix->docs, ix->rec, ix->meta, w[0], w[1],
                                             w[2], K, S, P, knn_ids, sp_ids, sp_sc, node_ids, nn, x0, out_ids, out_sc, out_sp_ids, out_sp_sc,
                                             ix->counters, hint));
        AP_CHECK_HIP(hipGetLastError());
    }
    return AP_OK;
}

// The refinement rounds of a construction: from the exact dense seed lists (ids[0], sc[0]; seed_slack != NULL: their scores but the K-th are within that) of all n = ix->docs.n documents
// and empty per-path lists (spi[0], sps[0]).  Returns in *cur which of the two buffers holds the result (rounds % 2), in *later what
// is to be freed once the rounds are over.
int ap_refine_rounds(const ap_index *ix, int32_t rounds, int32_t K, int32_t S, int32_t P, int32_t *const ids[2], float *const sc[2],
                     int32_t *const spi[2], float *const sps[2], int *cur, hipStream_t st, const float *seed_slack, const ApWork &work, void **later) {
    const int64_t n = ix->docs.n;
    *cur = 0;
    if (rounds <= 0) return AP_OK;
    float *own = nullptr, *tau = work.take<float>((size_t)3 * n);   // n, then the two sets of n words of known bits
    int rc = AP_OK;
    if (!tau) { rc = ap_dev_alloc(&own, (size_t)3 * n); tau = own; }
    uint32_t *known[2] = {reinterpret_cast<uint32_t *>(tau + n), reinterpret_cast<uint32_t *>(tau + 2 * n)};
    if (rc == AP_OK) {
        hipLaunchKernelGGL(k_take_tau, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, sc[0], n, K, 0u, tau);
        if (hipGetLastError() != hipSuccess) { ap_set_error("refinement failed to start"); rc = AP_EHIP; }
    }
    ApPacked pk;
    if (rc == AP_OK) rc = ap_pack_lists(ix, st, &pk);
    ix->packed_lists = pk.rec != nullptr;
    for (int32_t t = 0; t < rounds && rc == AP_OK; t++) {
        const int c = *cur;
        const ApRefineHints hint = t == 0 ? ApRefineHints{tau, sc[c], seed_slack, nullptr, nullptr, known[0], pk.rec, pk.at}
                                          : ApRefineHints{tau, nullptr, nullptr, sc[c], known[(t - 1) & 1], known[t & 1], pk.rec, pk.at};
        rc = ap_refine_round(ix, K, S, P, ids[c], spi[c], sps[c], nullptr, n, ids[1 - c], sc[1 - c], spi[1 - c], sps[1 - c], hint, st);
        *cur = 1 - c;
    }
    if (later && pk.bytes <= AP_WORK_BYTES) { *later = pk.mem; pk.mem = nullptr; }
    void *ptrs[] = {own, pk.mem};
    for (void *p : ptrs) if (p) (void)hipFree(p);   // waits for the rounds
    return rc;
}

extern "C" int ap_stage_refine(const ap_index *ix, int32_t K, int32_t S, int32_t P, const int32_t *knn_ids,
                               const int32_t *sp_ids, const float *sp_sc, const int32_t *node_ids, int64_t nn,
                               int32_t *out_ids, float *out_sc, int32_t *out_sp_ids, float *out_sp_sc, void *stream) {
    AP_REQUIRE(ix && knn_ids && sp_ids && sp_sc && out_ids && out_sc && out_sp_ids && out_sp_sc, "NULL argument");
    AP_REQUIRE(K >= 1 && K <= 256 && S >= 0 && S <= 32 && P >= 1 && P <= 32, "need 1<=K<=256, 0<=S<=32, 1<=P<=32");
    if (!node_ids) nn = ix->docs.n;
    if (nn <= 0) return AP_OK;
    return ap_refine_round(ix, K, S, P, knn_ids, sp_ids, sp_sc, node_ids, nn, out_ids, out_sc, out_sp_ids, out_sp_sc,
                           ApRefineHints{nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr}, (hipStream_t)stream);
}

// =================================================================== S4: neighbourhood similarities
// Dense part: G = X X^T for the K gathered rows of one neighbourhood (MFMA); what follows reads the lower triangle only.
// A tile on the diagonal has the same rows on both sides, which are loaded and staged once, and takes the ten of its sixteen
// 32 x 32 blocks that reach the triangle: three, two, two and three a wave, the roles going round with the node so that
// the SIMDs of a CU get the same work.  Same products in the same order as the full tile, so the same bits.  Bound by the gather of the rows (bf16
// rows: 10.7 -> 9.5 ms for 200,000 documents of 1,024 columns); for f32 rows it was the f32 matrix instructions, at a sixteenth of the bf16
// rate.  A f32 value is the sum of three bf16 values, each the rounding of what the ones before it leave.  So a tile on the diagonal is split while it goes to LDS
// and takes eight bf16 instructions for sixteen columns where f32 ones take eight at twice the cycles each: all products of two such sums but the smallest, which
// lies 2^-34 below the value.  The bf16 instruction cuts off what it adds to a sum below the sum's last place instead of rounding it, so that a sum that takes every product
// loses more than f32 instructions do where few columns are not zero (one: 5.9e-8 and 1.3e-7 of |a||b|, twelve of 768: 1.6e-7 and 4.2e-7).  Therefore the
// products of the first parts, each exact, are summed by 32 columns from zero on and added by the vector unit, which rounds, and the others have a sum of their own.
// 100,000 documents of 768 columns: 17.0 -> 11.8 ms.  Largest and root mean square error against 64 bits, of |a||b|, with f32 instructions and so:
// 1.6e-7 and 1.8e-8, 3.4e-8 and 3.6e-9 (768 Gaussian columns); 1.6e-6 and 3.5e-7, 3.1e-7 and 7.0e-8 (768 positive ones); one column that is not zero 5.9e-8 and 2.5e-8
// either way, three 1.2e-7 and 2.1e-8, 1.1e-7 and 1.5e-8, twelve 1.6e-7 and 1.9e-8, 1.0e-7 and 0.9e-8; smaller too at 4, 16, 96, 260 and 1,024 columns.
// Not where a norm says that values may overflow as bf16 (beyond 1e15) or that a rounding's rest may get lost among the smallest numbers (below
// 1e-12), nor with an infinity or a NaN: those neighbourhoods take the f32 instructions.
#define AP_GD_STRIDE (AP_BK + 8)   // bf16 elements: 80-byte rows, of which eight lanes' 16-byte reads meet every bank once
typedef __bf16 ap_bf16x2 __attribute__((ext_vector_type(2)));
// The three parts of two values, packed as they lie in LDS.
__device__ __forceinline__ void ap_split_bf16(float x, float y, uint32_t (&part)[3]) {
#pragma unroll
    for (int p = 0; p < 3; p++) {
        part[p] = __builtin_bit_cast(uint32_t, ap_bf16x2{(__bf16)x, (__bf16)y});
        x -= __uint_as_float(part[p] << 16); y -= __uint_as_float(part[p] & 0xffff0000u);   // exact
    }
}
template <int DT>
__global__ __launch_bounds__(256, DT == AP_F32 ? 2 : 1) void k_gram_dense(const void *dense, const float *__restrict__ norm, int32_t dim, int32_t K, const int32_t *__restrict__ knn,
                                                    const int32_t *__restrict__ node_ids, int64_t x0,
                                                    float *__restrict__ pm /* chunk x K x K */) {
    __shared__ __attribute__((aligned(16))) unsigned char lds[ApTileLds<DT>::BYTES];
    __shared__ int32_t a_rows[AP_TILE], b_rows[AP_TILE];
    const int64_t x = blockIdx.y;
    const int64_t u = node_ids ? (int64_t)node_ids[x0 + x] : x0 + x;
    const int32_t tiles = (K + AP_TILE - 1) / AP_TILE;
    const int32_t i0 = (blockIdx.x / tiles) * AP_TILE, j0 = (blockIdx.x % tiles) * AP_TILE;
    if (j0 > i0) return;   // uniform: above the triangle
    if (threadIdx.x < AP_TILE) {
        a_rows[threadIdx.x] = i0 + threadIdx.x < K ? knn[u * K + i0 + threadIdx.x] : -1;
        b_rows[threadIdx.x] = j0 + threadIdx.x < K ? knn[u * K + j0 + threadIdx.x] : -1;
    }
    ap_f32x16 acc[2][2];
    float *out = pm + x * (int64_t)K * K;
    if (i0 != j0) {
        ap_tile_product<DT>(dense, dim, a_rows, b_rows, lds, acc);
        ap_tile_foreach(acc, [&](int i, int j, float v) {
            if (i0 + i < K && j0 + j < K) out[(int64_t)(i0 + i) * K + (j0 + j)] = v;
        });
        return;
    }
    const int lane = threadIdx.x & 63, li = lane & 31, half = lane >> 5;
    const int role = (ap_wave_id() + (int)(x & 3)) & 3;   // uniform
    // roles 0 and 3: blocks (r, r), (r + 1, r), (r + 1, r + 1) of r = 0, 2; roles 1 and 2: (2, 0), (2, 1) and (3, 0), (3, 1)
    const bool corner = role == 0 || role == 3;
    const int r0 = corner ? (role ? 2 : 0) : role + 1, c0 = role == 3 ? 2 : 0;
    const bool any = i0 + r0 * 32 < K;
#pragma unroll
    for (int a = 0; a < 2; a++)
#pragma unroll
        for (int b = 0; b < 2; b++)
#pragma unroll
            for (int r = 0; r < 16; r++) acc[a][b][r] = 0.f;
    bool odd = false;   // uniform, f32 rows: a neighbourhood whose values three bf16 ones may not hold
    if (DT == AP_F32) {
        if (threadIdx.x < AP_TILE && a_rows[threadIdx.x] >= 0) {   // this thread's own entry
            const float x = norm[a_rows[threadIdx.x]];
            odd = !(x <= 1e15f && x >= 1e-12f);
        }
        odd = __syncthreads_or(odd) != 0;
    } else __syncthreads();   // the row list
    if constexpr (DT == AP_F32) if (!odd) {
        uint16_t *lS = reinterpret_cast<uint16_t *>(lds);   // [3][128][AP_GD_STRIDE]
        static_assert(3 * AP_TILE * AP_GD_STRIDE * 2 <= ApTileLds<AP_F32>::BYTES, "LDS");
        constexpr int PLANE = AP_TILE * AP_GD_STRIDE;
        float4 va[4];
        int32_t ra[4];
#pragma unroll
        for (int pass = 0; pass < 4; pass++) ra[pass] = a_rows[(threadIdx.x >> 3) + 32 * pass];
        ap_tile_load<DT>(dense, dim, ra, 0, va);
        const uint16_t *pa = lS + (r0 * 32 + li) * AP_GD_STRIDE + half * 8, *pb = lS + (c0 * 32 + li) * AP_GD_STRIDE + half * 8;
        const uint16_t *pc = lS + ((corner ? r0 + 1 : c0 + 1) * 32 + li) * AP_GD_STRIDE + half * 8;
        auto read = [&](const uint16_t *at, ap_bf16x8 (&f)[3]) {
#pragma unroll
            for (int p = 0; p < 3; p++) f[p] = __builtin_bit_cast(ap_bf16x8, *reinterpret_cast<const uint4 *>(at + p * PLANE));
        };
        constexpr int N = 7, TA[N] = {1, 2, 1, 2, 0, 1, 0}, TB[N] = {2, 1, 1, 0, 2, 0, 1};   // the smaller products, the smallest first
        ap_f32x16 rest[2][2];   // their sum
#pragma unroll
        for (int a = 0; a < 2; a++)
#pragma unroll
            for (int b = 0; b < 2; b++)
#pragma unroll
                for (int r = 0; r < 16; r++) rest[a][b][r] = 0.f;
        const ap_f32x16 none = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        for (int32_t k0 = 0; k0 < dim; k0 += AP_BK) {
            __syncthreads();
            const bool inside = k0 + (int)(threadIdx.x & 7) * 4 < dim;
#pragma unroll
            for (int pass = 0; pass < 4; pass++) {
                const bool keep = ra[pass] >= 0 && inside;
                uint32_t lo[3], hi[3];
                ap_split_bf16(keep ? va[pass].x : 0.f, keep ? va[pass].y : 0.f, lo);
                ap_split_bf16(keep ? va[pass].z : 0.f, keep ? va[pass].w : 0.f, hi);
                uint16_t *to = lS + ((threadIdx.x >> 3) + 32 * pass) * AP_GD_STRIDE + (threadIdx.x & 7) * 4;
#pragma unroll
                for (int p = 0; p < 3; p++) *reinterpret_cast<uint2 *>(to + p * PLANE) = make_uint2(lo[p], hi[p]);
            }
            __syncthreads();
            if (k0 + AP_BK < dim) ap_tile_load<DT>(dense, dim, ra, k0 + AP_BK, va);
            if (!any) continue;
            auto multiply = [&](const uint16_t *px, const uint16_t *py, ap_f32x16 &to, ap_f32x16 &low) {
                ap_f32x16 first = none;
#pragma unroll
                for (int kk = 0; kk < AP_BK; kk += 16) {
                    ap_bf16x8 x[3], y[3];
                    read(px + kk, x);
                    read(py + kk, y);
#pragma unroll
                    for (int t = 0; t < N; t++) low = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[TA[t]], y[TB[t]], low, 0, 0, 0);
                    first = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[0], y[0], first, 0, 0, 0);
                }
#pragma unroll
                for (int r = 0; r < 16; r++) to[r] += first[r];
                __builtin_amdgcn_sched_barrier(0);   // one block after the other: two at a time spill
            };
            if (corner) {
                multiply(pa, pa, acc[0][0], rest[0][0]);
                multiply(pc, pa, acc[1][0], rest[1][0]);
                multiply(pc, pc, acc[1][1], rest[1][1]);
            } else {
                multiply(pa, pb, acc[0][0], rest[0][0]);
                multiply(pa, pc, acc[0][1], rest[0][1]);
            }
        }
#pragma unroll
        for (int a = 0; a < 2; a++)
#pragma unroll
            for (int b = 0; b < 2; b++)
#pragma unroll
                for (int r = 0; r < 16; r++) acc[a][b][r] += rest[a][b][r];
    }
    if (DT == AP_F32 && odd) {
        float *lA = reinterpret_cast<float *>(lds);
        float4 va[4];
        int32_t ra[4];
#pragma unroll
        for (int pass = 0; pass < 4; pass++) ra[pass] = a_rows[(threadIdx.x >> 3) + 32 * pass];
        ap_tile_load<DT>(dense, dim, ra, 0, va);
        for (int32_t k0 = 0; k0 < dim; k0 += AP_BK) {
            __syncthreads();
            ap_tile_store(va, ra, dim, k0, lA);
            __syncthreads();
            if (k0 + AP_BK < dim) ap_tile_load<DT>(dense, dim, ra, k0 + AP_BK, va);
            const float *pa = lA + (r0 * 32 + li) * AP_LDS_STRIDE + half, *pb = lA + (c0 * 32 + li) * AP_LDS_STRIDE + half;
            const float *pc = lA + ((corner ? r0 + 1 : c0 + 1) * 32 + li) * AP_LDS_STRIDE + half;
            if (!any) continue;
            if (corner) {
#pragma unroll
                for (int kk = 0; kk < AP_BK; kk += 2) {
                    const float a0 = pa[kk], a1 = pc[kk];
                    acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, a0, acc[0][0], 0, 0, 0);
                    acc[1][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1, a0, acc[1][0], 0, 0, 0);
                    acc[1][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1, a1, acc[1][1], 0, 0, 0);
                }
            } else {
#pragma unroll
                for (int kk = 0; kk < AP_BK; kk += 2) {
                    const float a0 = pa[kk], b0 = pb[kk], b1 = pc[kk];
                    acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, b0, acc[0][0], 0, 0, 0);
                    acc[0][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, b1, acc[0][1], 0, 0, 0);
                }
            }
        }
    }
    if constexpr (DT == AP_BF16) {
        uint16_t *lA = reinterpret_cast<uint16_t *>(lds);
        uint4 va[AP_NP16];
        int32_t ra[AP_NP16];
#pragma unroll
        for (int pass = 0; pass < AP_NP16; pass++) ra[pass] = a_rows[threadIdx.x / AP_TPR16 + AP_RPP16 * pass];
        ap_tile_load_bf16(dense, dim, ra, 0, va);
        for (int32_t k0 = 0; k0 < dim; k0 += AP_BK16) {
            __syncthreads();
            ap_tile_store_bf16(va, ra, dim, k0, lA);
            __syncthreads();
            if (k0 + AP_BK16 < dim) ap_tile_load_bf16(dense, dim, ra, k0 + AP_BK16, va);
            const uint16_t *pa = lA + (r0 * 32 + li) * AP_LDS_STRIDE16 + half * 8, *pb = lA + (c0 * 32 + li) * AP_LDS_STRIDE16 + half * 8;
            const uint16_t *pc = lA + ((corner ? r0 + 1 : c0 + 1) * 32 + li) * AP_LDS_STRIDE16 + half * 8;
            if (!any) continue;
#pragma unroll
            for (int kk = 0; kk < AP_BK16; kk += 16) {
                const ap_bf16x8 a0 = __builtin_bit_cast(ap_bf16x8, *reinterpret_cast<const uint4 *>(pa + kk));
                const ap_bf16x8 c1 = __builtin_bit_cast(ap_bf16x8, *reinterpret_cast<const uint4 *>(pc + kk));
                if (corner) {
                    acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, a0, acc[0][0], 0, 0, 0);
                    acc[1][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(c1, a0, acc[1][0], 0, 0, 0);
                    acc[1][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(c1, c1, acc[1][1], 0, 0, 0);
                } else {
                    const ap_bf16x8 b0 = __builtin_bit_cast(ap_bf16x8, *reinterpret_cast<const uint4 *>(pb + kk));
                    acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, b0, acc[0][0], 0, 0, 0);
                    acc[0][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, c1, acc[0][1], 0, 0, 0);
                }
            }
        }
    }
#pragma unroll
    for (int a = 0; a < 2; a++)
#pragma unroll
        for (int b = 0; b < 2; b++) {
            if (corner ? (a == 0 && b == 1) : a == 1) continue;   // uniform: not this role's
#pragma unroll
            for (int r = 0; r < 16; r++) {
                const int i = i0 + (r0 + a) * 32 + 8 * (r >> 2) + 4 * half + (r & 3), j = j0 + (c0 + b) * 32 + li;
                if (i < K && j <= i) out[(int64_t)i * K + j] = acc[a][b][r];
            }
        }
}

// Sparse and lexical parts of the neighbourhood similarities, and the fusion with the dense part: sorted lists are
// merged, one lane per pair.
// A 256-thread block takes a 16 x 16 tile of one neighbourhood's matrix (tiles on or below the diagonal; the matrix is
// symmetric and mirrored on output).  The packed records of the tile's 16 row and 16 column documents (sparse
// entries then lexical entries, ascending term ids) are copied to LDS, and thread (r, c) walks the two sorted lists
// of its pair with two cursors: about |a| + |b| steps, one 8-byte LDS read per step, products added in ascending
// term order.  Every lane works on a pair of its own, so an instruction serves 64 pairs; a wave-per-pair look-up
// scheme spends most of its instructions on terms the other list does not hold.
#define AP_GT 16                 // tile edge
#define AP_GT_ENTRIES 6144       // LDS budget of a tile: 32 records of ~165 entries; a tile that needs more reads global memory

// Straight-line body: every lane of the wave runs the same instructions until the last lane's lists are used up; a
// lane that is done keeps re-reading its last entries and adds nothing.
template <typename P>
__device__ __forceinline__ float ap_merge_dot(P a, int32_t na, P b, int32_t nb) {
    float acc = 0.f;
    bool live = na > 0 && nb > 0;
    int32_t pa = 0, pb = 0;
    uint64_t ea = live ? a[0] : 0ull, eb = live ? b[0] : 1ull;
    while (__any(live)) {
        const uint32_t ta = (uint32_t)ea, tb = (uint32_t)eb;
        const float prod = __uint_as_float((uint32_t)(ea >> 32)) * __uint_as_float((uint32_t)(eb >> 32));
        acc = (live && ta == tb) ? acc + prod : acc;
        pa += (live && ta <= tb) ? 1 : 0;
        pb += (live && tb <= ta) ? 1 : 0;
        live = live && pa < na && pb < nb;
        if (live) { ea = a[pa]; eb = b[pb]; }
    }
    return acc;
}

// The same walk over two lists in LDS that each end in a sentinel entry (weight 0) and one entry of padding: nothing is
// masked and no cursor is clamped.  The a side's sentinel term is 0xffffffff and a's cursor moves on "a's term <= b's
// term" compared UNSIGNED; the b side's is 0x7fffffff and b's cursor moves on "b's term <= a's term" compared SIGNED.
// Real terms lie in [0, 0x7fffffff), where the two orders agree; a's sentinel is the largest value of the unsigned
// order and b's the largest of the signed one, so a cursor that has reached its sentinel never moves again, whatever
// the other side shows, and the two sentinels never match each other or a term.  The walk tests "is any lane's pair
// still live" once per AP_GT_UNROLL steps: a lane whose pair is done idles on its sentinels.  a_end and b_end are the LDS byte
// addresses of the sentinels; same products in the same order as ap_merge_dot.
#define AP_GT_SENT 2
#define AP_GT_UNROLL 8   // steps per liveness test (prune stage of 200,000 documents: 2: 396 ms, 4: 361 ms, 8: 350 ms, 16: 351 ms)
#define AP_GT_SENT_A 0xffffffffull
#define AP_GT_SENT_B 0x7fffffffull
__device__ __forceinline__ float ap_merge_dot_lds(uint32_t a, uint32_t a_end, uint32_t b, uint32_t b_end) {
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));   // a plain vector value: loads from LDS as it is
    typedef const AP_LDS u32x2 *LP;
    auto at = [](uint32_t p) { return *(LP)(uintptr_t)p; };
    float acc = 0.f;
    // Each list's current entry and the one after it are in registers; a step reads the entry that follows the new
    // "next" position, which the step after it may select: the LDS round trip has a step's instructions to hide behind.
    u32x2 ea = at(a), eb = at(b), ea1 = at(a + 8u), eb1 = at(b + 8u);
    while (__any(a < a_end && b < b_end)) {
#pragma unroll
        for (int u = 0; u < AP_GT_UNROLL; u++) {
            const bool adva = ea.x <= eb.x, advb = (int32_t)eb.x <= (int32_t)ea.x;
            // adds exactly 0 when the terms differ (taking "both cursors move" for the match test saves the compare and
            // is no faster: the scalar AND of the two masks sits in the dependency chain)
            acc = fmaf(ea.x == eb.x ? __uint_as_float(ea.y) : 0.f, __uint_as_float(eb.y), acc);
            a = adva ? a + 8u : a; b = advb ? b + 8u : b;
            const u32x2 la = at(a + 8u), lb = at(b + 8u);
            ea.x = adva ? ea1.x : ea.x; ea.y = adva ? ea1.y : ea.y;
            eb.x = advb ? eb1.x : eb.x; eb.y = advb ? eb1.y : eb.y;
            ea1 = la; eb1 = lb;
        }
    }
    return acc;
}

__global__ __launch_bounds__(256) void k_gram_merge(const uint2 *__restrict__ rec, const uint4 *__restrict__ meta, float wd, float ws,
                                                    float wf, int32_t K, const int32_t *__restrict__ knn,
                                                    const int32_t *__restrict__ node_ids, int64_t x0, float *__restrict__ pm) {
    __shared__ uint64_t ent[AP_GT_ENTRIES];
    __shared__ int32_t d_id[2 * AP_GT], d_off[2 * AP_GT], d_sn[2 * AP_GT], d_tn[2 * AP_GT];
    __shared__ uint32_t d_first[2 * AP_GT];
    __shared__ int32_t s_total;
    const int64_t x = blockIdx.y;
    const int64_t u = node_ids ? (int64_t)node_ids[x0 + x] : x0 + x;
    // tile number -> (row block I, column block J), J <= I
    int32_t I = 0, rem = (int32_t)blockIdx.x;
    while (rem > I) { rem -= I + 1; I++; }
    const int32_t J = rem;
    const int tid = threadIdx.x, lane = tid & 63;
    if (tid < 64) {   // slots 0..15: row documents, 16..31: column documents
        int32_t id = -1, sn = 0, tn = 0;
        uint32_t first = 0;
        if (lane < 2 * AP_GT) {
            const int32_t pos = (lane < AP_GT ? I * AP_GT + lane : J * AP_GT + lane - AP_GT);
            if (pos < K) id = knn[u * K + pos];
            if (id >= 0) { const uint4 m = meta[id]; first = m.x; sn = (int32_t)(m.y & 0xffffu); tn = (int32_t)(m.y >> 16); }
        }
        const int32_t room = lane < 2 * AP_GT ? sn + tn + 2 * AP_GT_SENT : 0;   // a record in LDS: sparse entries, sentinels, lexical entries, sentinels
        int32_t incl = room;
        for (int o = 1; o < 64; o <<= 1) {
            const int32_t up = __shfl_up(incl, o, 64);
            if (lane >= o) incl += up;
        }
        if (lane < 2 * AP_GT) { d_id[lane] = id; d_off[lane] = incl - room; d_sn[lane] = sn; d_tn[lane] = tn; d_first[lane] = first; }
        if (lane == 2 * AP_GT - 1) s_total = incl;
    }
    __syncthreads();
    const bool in_lds = s_total <= AP_GT_ENTRIES;   // uniform
    const uint64_t *grec = reinterpret_cast<const uint64_t *>(rec);
    if (in_lds) {
        for (int d = 0; d < 2 * AP_GT; d++) {
            const int32_t sn = d_sn[d], len = sn + d_tn[d], off = d_off[d];
            const uint64_t *src = grec + d_first[d];
            for (int32_t e = tid; e < len; e += 256) ent[off + e + (e >= sn ? AP_GT_SENT : 0)] = src[e];
            if (tid < AP_GT_SENT) {   // slots 0..15 are a sides of the walks, 16..31 b sides
                const uint64_t sent = d < AP_GT ? AP_GT_SENT_A : AP_GT_SENT_B;
                ent[off + sn + tid] = sent; ent[off + len + AP_GT_SENT + tid] = sent;
            }
        }
        __syncthreads();
    }
    const int r = tid / AP_GT, c = tid % AP_GT;
    const int32_t i = I * AP_GT + r, j = J * AP_GT + c;
    if (i >= K || j >= K || j > i) return;
    float *out = pm + x * (int64_t)K * K;
    const int32_t a = d_id[r], b = d_id[AP_GT + c];
    float val = -INFINITY;
    if (a >= 0 && b >= 0) {
        float qs, qt;
        if (in_lds) {
            const uint32_t base = (uint32_t)(uintptr_t)(const AP_LDS uint64_t *)ent;
            const uint32_t la = base + 8u * (uint32_t)d_off[r], lb = base + 8u * (uint32_t)d_off[AP_GT + c];
            const uint32_t sa = 8u * (uint32_t)d_sn[r], sb = 8u * (uint32_t)d_sn[AP_GT + c];
            qs = ap_merge_dot_lds(la, la + sa, lb, lb + sb);
            const uint32_t ta = la + sa + 8u * AP_GT_SENT, tb = lb + sb + 8u * AP_GT_SENT;
            qt = ap_merge_dot_lds(ta, ta + 8u * (uint32_t)d_tn[r], tb, tb + 8u * (uint32_t)d_tn[AP_GT + c]);
        } else {
            const uint64_t *ga = grec + d_first[r], *gb = grec + d_first[AP_GT + c];
            qs = ap_merge_dot(ga, d_sn[r], gb, d_sn[AP_GT + c]);
            qt = ap_merge_dot(ga + d_sn[r], d_tn[r], gb + d_sn[AP_GT + c], d_tn[AP_GT + c]);
        }
        val = fmaf(wd, out[(int64_t)i * K + j], fmaf(wf, qt, ws * qs));
    }
    out[(int64_t)i * K + j] = val;
    out[(int64_t)j * K + i] = val;
}

// The same products as matrix products.  What bounds the walks above is instruction issue: some 330 steps of 13
// instructions per pair, nearly all of them over terms the other list does not hold.  Here the K lists of a neighbourhood
// are turned into columns instead: a term that only one of the K documents holds contributes to no pair and is dropped; the
// others (some 2,000 of a neighbourhood of 128) are numbered in ascending order.  Nine of ten of them have AP_GL_FEW holders
// or fewer: their pairs are added one by one (a tenth of a percent of the products that their columns would take in a matrix).
// The K x T matrix of the others' weights is multiplied with its transpose by f32 MFMAs, 64 columns at a time.  Same f32
// products and sums (an absent term adds exactly 0); only the order of a sum's terms differs.
//
// One workgroup of 16 waves per node; per vocabulary:
//  - a wave loads the lists of its 8 documents into registers (3 entries a lane: 192 a list; what a longer list holds beyond
//    that is read again for every chunk);
//  - two bitmaps over the vocabulary in LDS mark terms met and terms met twice; the number of set bits before a term's in
//    the second is its column;
//  - the columns' holders are counted, and those of the columns with few laid out one after the other (in any order: a document holds
//    a term once).  Eight lanes take a row and add, for its entries in ascending order of the terms, the products with the holders
//    of lower rows to the row's part of a triangle in LDS: every pair has one owner and one order.  The triangle is what the
//    product's accumulators start with;
//  - a wave writes its 8 rows of a chunk (cleared, then the entries whose column falls into it), into one of two stages,
//    while the other stage is multiplied: one barrier a chunk.
// The lower triangle of the result is 36 blocks of 16 x 16 (K = 128): two a wave and four more on the first four waves, nine
// on every SIMD.  A neighbourhood with a list beyond the registers, or more columns or entries than the LDS holds, takes all of its
// columns to the matrix, and so does one with AP_GL_SPLIT(K) columns or fewer: setting them apart takes the same steps for any K, a chunk
// of the matrix the less the fewer blocks there are.  Prune stage of 6,000 documents of 128 columns with all columns in the matrix and
// with those apart, ms: K = 128, 650 columns 3.37 and 2.98, 1,800: 5.67 and 3.90; K = 64, 490: 1.89 and 1.92, 640: 2.06 and 2.01,
// 960: 2.48 and 2.28; K = 48, 500: 1.47 and 1.51, 730: 1.75 and 1.74; K = 32, 500: 1.34 and 1.44.
// Both vocabularies are written out: with one body for the two the accumulators are chosen by the vocabulary at run time, and 64 registers
// spill (K = 32, lists of 20 and 13 terms, nothing set apart: 1.21 and 0.95 ms; K = 128 above: 3.67 and 2.98, 4.72 and 3.90).  The prune
// stage's lists over 100,000 f32 documents: 160 ms with the walks, 66 ms with all columns in the matrix, 41 ms with those of few holders
// apart and spills, 28.9 ms here; 200,000 bf16: 299, 109, 76 and 53.8 ms.  What is left is mostly marking, numbering and counting the columns
// and the pairs: chains of LDS round trips that 16 waves do not hide.
#define AP_GL_WORDS 8192          // words of a bitmap: vocabularies up to 2^18 terms
#define AP_GL_C 64                // columns of a chunk
#define AP_GL_STRIDE (AP_GL_C + 4)   // rows 16-byte aligned; 16 rows x 4 groups of 4 columns fall into distinct banks
#define AP_GL_SLOTS 3             // list entries a lane holds in registers
#define AP_GL_FEW 8               // holders of a column whose pairs are added one by one
#define AP_GL_SPLIT(K) ((K) < 64 ? 32768 / (K) : 512)   // columns beyond which setting those with few holders apart pays
#define AP_GL_COLS 4096           // columns whose holders are counted (16 KB where the bitmaps were)
#define AP_GL_HOLD 6144           // entries of the columns with few holders (48 KB behind them, 48 KB behind the triangle)
#define AP_GL_U 4                 // entries of a row on their way at a time
#define AP_GL_LDS (2 * AP_GL_WORDS * 4 + 128 * 127 / 2 * 4 + AP_GL_HOLD * 8)
typedef float ap_f32x4 __attribute__((ext_vector_type(4)));
__global__ __launch_bounds__(1024) void k_gram_lists(const uint2 *__restrict__ rec, const uint4 *__restrict__ meta, float wd, float ws, float wf,
                                                     int32_t sp_words, int32_t tx_words, int32_t K, const int32_t *__restrict__ knn,
                                                     const int32_t *__restrict__ node_ids, int64_t x0, float *__restrict__ pm) {
    extern __shared__ __attribute__((aligned(16))) uint32_t gl_lds[];
    uint32_t *seen = gl_lds, *twice = gl_lds + AP_GL_WORDS;   // seen: afterwards the columns before each word's terms
    float *X = reinterpret_cast<float *>(gl_lds + 2 * AP_GL_WORDS);   // two stages of 128 x AP_GL_STRIDE
    __shared__ int32_t s_id[128], s_sn[128], s_tn[128];
    __shared__ uint32_t s_first[128], s_part[16], s_total;
    __shared__ float s_diag[2][128];
    __shared__ int32_t s_rare[128], s_rare_at[128], s_rare_end[2];   // a row's entries of columns with few holders, the first one's place among its wave's
    uint32_t *col_map = gl_lds;                                     // [AP_GL_COLS], once the columns are known
    uint2 *hold = reinterpret_cast<uint2 *>(gl_lds + AP_GL_COLS);   // [AP_GL_HOLD] (row, weight)
    float *tri = X;                                                 // [128 * 127 / 2] row i's sums with the rows below i, before the stages are written
    uint2 *rare = reinterpret_cast<uint2 *>(X + 128 * 127 / 2);     // [AP_GL_HOLD] (first holder's place | their number << 13, weight)
    static_assert(AP_GL_COLS + 2 * AP_GL_HOLD <= 2 * AP_GL_WORDS && 2 * 128 * AP_GL_STRIDE <= 128 * 127 / 2 + 2 * AP_GL_HOLD && AP_GL_FEW <= 8, "LDS");
    const int64_t x = blockIdx.x;
    const int64_t u = node_ids ? (int64_t)node_ids[x0 + x] : x0 + x;
    const int tid = threadIdx.x, lane = tid & 63, wave = ap_wave_id();
    if (tid < 128) {
        const int32_t id = tid < K ? knn[u * K + tid] : -1;
        uint4 m = make_uint4(0, 0, 0, 0);
        if (id >= 0) m = meta[id];
        s_id[tid] = id; s_first[tid] = m.x; s_sn[tid] = (int32_t)(m.y & 0xffffu); s_tn[tid] = (int32_t)(m.y >> 16);
    }
    if (tid < 2) s_rare_end[tid] = 0;
    const int32_t blocks = (K + 15) / 16, n_tasks = blocks * (blocks + 1) / 2;
    // this wave's blocks of the lower triangle: tasks wave, wave + 16, wave + 32
    int32_t bi[3], bj[3];
#pragma unroll
    for (int a = 0; a < 3; a++) {
        int32_t p = wave + 16 * a, i = 0;
        while (p > i) { p -= i + 1; i++; }
        bi[a] = i; bj[a] = p;
    }
    ap_f32x4 acc[2][3];
#pragma unroll
    for (int part = 0; part < 2; part++)
#pragma unroll
        for (int a = 0; a < 3; a++) acc[part][a] = ap_f32x4{0.f, 0.f, 0.f, 0.f};
    __syncthreads();
#pragma unroll
    for (int part = 0; part < 2; part++) {
        const int32_t words = part ? tx_words : sp_words;
        for (int32_t i = tid * 4; i < words; i += 4096) {   // words is a multiple of 4
            *reinterpret_cast<uint4 *>(seen + i) = make_uint4(0, 0, 0, 0);
            *reinterpret_cast<uint4 *>(twice + i) = make_uint4(0, 0, 0, 0);
        }
        uint2 ent[8][AP_GL_SLOTS];   // (term, then column; weight)
#pragma unroll
        for (int d = 0; d < 8; d++) {
            const int32_t row = wave * 8 + d, len = part ? s_tn[row] : s_sn[row];
            const uint2 *r = rec + s_first[row] + (part ? s_sn[row] : 0);
#pragma unroll
            for (int k = 0; k < AP_GL_SLOTS; k++) ent[d][k] = lane + 64 * k < len ? r[lane + 64 * k] : make_uint2(0xffffffffu, 0u);
        }
        __syncthreads();   // the bitmaps are clear
        auto mark = [&](uint32_t t) {
            const uint32_t bit = 1u << (t & 31);
            if (atomicOr(&seen[t >> 5], bit) & bit) atomicOr(&twice[t >> 5], bit);
        };
#pragma unroll
        for (int d = 0; d < 8; d++) {
            const int32_t row = wave * 8 + d, len = part ? s_tn[row] : s_sn[row];
            float own = 0.f;
#pragma unroll
            for (int k = 0; k < AP_GL_SLOTS; k++) {
                const float v = __uint_as_float(ent[d][k].y);
                own = fmaf(v, v, own);
                if (ent[d][k].x != 0xffffffffu) mark(ent[d][k].x);
            }
            const uint2 *r = rec + s_first[row] + (part ? s_sn[row] : 0);
            for (int32_t e = 64 * AP_GL_SLOTS + lane; e < len; e += 64) {
                const uint2 y = r[e];
                own = fmaf(__uint_as_float(y.y), __uint_as_float(y.y), own);
                mark(y.x);
            }
            own = ap_wave_sum(own);
            if (lane == 0) s_diag[part][row] = own;
        }
        __syncthreads();
        // columns before each word: eight words a thread
        {
            uint32_t cnt[8], sum = 0;
#pragma unroll
            for (int k = 0; k < 8; k += 4) {   // words is a multiple of 4
                const uint4 t4 = tid * 8 + k < words ? *reinterpret_cast<const uint4 *>(twice + tid * 8 + k) : make_uint4(0, 0, 0, 0);
                cnt[k] = (uint32_t)__popc(t4.x); cnt[k + 1] = (uint32_t)__popc(t4.y); cnt[k + 2] = (uint32_t)__popc(t4.z); cnt[k + 3] = (uint32_t)__popc(t4.w);
                sum += cnt[k] + cnt[k + 1] + cnt[k + 2] + cnt[k + 3];
            }
            uint32_t upto = sum;
            for (int o = 1; o < 64; o <<= 1) { const uint32_t up = __shfl_up(upto, o, 64); if (lane >= o) upto += up; }
            if (lane == 63) s_part[wave] = upto;
            __syncthreads();
            uint32_t base = 0;
            for (int w = 0; w < wave; w++) base += s_part[w];
            base += upto - sum;
#pragma unroll
            for (int k = 0; k < 8; k += 4) {
                const uint32_t b1 = base + cnt[k], b2 = b1 + cnt[k + 1], b3 = b2 + cnt[k + 2];
                if (tid * 8 + k < words) *reinterpret_cast<uint4 *>(seen + tid * 8 + k) = make_uint4(base, b1, b2, b3);
                base = b3 + cnt[k + 3];
            }
            if (tid == 1023) s_total = base;
        }
        __syncthreads();
        auto column = [&](uint32_t t) -> uint32_t {
            const uint32_t m = twice[t >> 5], bit = 1u << (t & 31);
            return m & bit ? seen[t >> 5] + (uint32_t)__popc(m & (bit - 1u)) : 0xffffffffu;
        };
#pragma unroll
        for (int d = 0; d < 8; d++)
#pragma unroll
            for (int k = 0; k < AP_GL_SLOTS; k++)
                if (ent[d][k].x != 0xffffffffu) ent[d][k].x = column(ent[d][k].x);
        uint32_t longs = 0;   // uniform: documents of this wave whose list goes on behind the registers
        for (int d = 0; d < 8; d++) longs |= ap_uniform_i32(part ? s_tn[wave * 8 + d] : s_sn[wave * 8 + d]) > 64 * AP_GL_SLOTS ? 1u << d : 0u;
        int32_t n_cols = (int32_t)ap_uniform_u32(s_total);   // columns of the matrix
        if (!__syncthreads_or(longs != 0) && n_cols > AP_GL_SPLIT(K) && n_cols <= AP_GL_COLS) {   // uniform; nobody asks the bitmaps any more
            *reinterpret_cast<uint4 *>(col_map + tid * 4) = make_uint4(0, 0, 0, 0);
            __syncthreads();
            // an entry: column | place among its column's holders << 16
#pragma unroll
            for (int d = 0; d < 8; d++)
#pragma unroll
                for (int k = 0; k < AP_GL_SLOTS; k++)
                    if (ent[d][k].x != 0xffffffffu) ent[d][k].x |= atomicAdd(&col_map[ent[d][k].x], 1u) << 16;
            __syncthreads();
            // four columns a thread: 1 << 31 | its column of the matrix, or the first holder's place | their number << 13.  Sums of
            // both kinds in one scan: columns of the matrix << 18 | holders of the others (at most 8 * 4,096)
            const uint4 c4 = *reinterpret_cast<const uint4 *>(col_map + tid * 4);
            const uint32_t hc[4] = {c4.x, c4.y, c4.z, c4.w};
            uint32_t own[4], sum = 0;
#pragma unroll
            for (int k = 0; k < 4; k++) { own[k] = hc[k] > AP_GL_FEW ? 1u << 18 : hc[k]; sum += own[k]; }
            uint32_t upto = sum;
            for (int o = 1; o < 64; o <<= 1) { const uint32_t up = __shfl_up(upto, o, 64); if (lane >= o) upto += up; }
            if (lane == 63) s_part[wave] = upto;
            __syncthreads();
            uint32_t base = upto - sum;
            for (int w = 0; w < wave; w++) base += s_part[w];
            uint32_t to[4];
#pragma unroll
            for (int k = 0; k < 4; k++) {
                to[k] = hc[k] > AP_GL_FEW ? 0x80000000u | (base >> 18) : (base & 0x1fffu) | (hc[k] << 13);
                base += own[k];
            }
            *reinterpret_cast<uint4 *>(col_map + tid * 4) = make_uint4(to[0], to[1], to[2], to[3]);
            if (tid == 1023) s_total = base;
            __syncthreads();
            const uint32_t total = ap_uniform_u32(s_total);
            if ((int32_t)(total & 0x3ffffu) <= AP_GL_HOLD) {   // uniform
                n_cols = (int32_t)(total >> 18);
                uint32_t most = 0, n_all = 0;   // uniform
#pragma unroll
                for (int d = 0; d < 8; d++) {
                    uint32_t n_rare = 0;
#pragma unroll
                    for (int k = 0; k < AP_GL_SLOTS; k++) {
                        const uint32_t e = ent[d][k].x;
                        bool few = false;
                        if (e != 0xffffffffu) {
                            const uint32_t m = col_map[e & 0xffffu];
                            few = m < 0x80000000u;
                            if (few) hold[(m & 0x1fffu) + (e >> 16)] = make_uint2((uint32_t)(wave * 8 + d), ent[d][k].y);
                            ent[d][k].x = few ? 0x80000000u | m : m & 0x7fffffffu;
                        }
                        n_rare += (uint32_t)__popcll(__ballot(few));
                    }
                    if (lane == 0) { s_rare[wave * 8 + d] = (int32_t)n_rare; s_rare_at[wave * 8 + d] = (int32_t)n_all; }
                    n_all += n_rare;
                    most = max(most, n_rare);
                }
                int32_t at = 0;   // the wave's place among the rows' entries; any will do
                if (lane == 0) at = atomicAdd(&s_rare_end[part], (int32_t)n_all);
                at = ap_uniform_i32(at);
                const int32_t wave_at = at;
#pragma unroll
                for (int d = 0; d < 8; d++)
#pragma unroll
                    for (int k = 0; k < AP_GL_SLOTS; k++) {
                        const uint32_t e = ent[d][k].x;
                        const bool few = e != 0xffffffffu && e >= 0x80000000u;
                        const uint64_t m = __ballot(few);
                        if (few) rare[at + (int32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] = make_uint2(e & 0x7fffffffu, ent[d][k].y);
                        at += __popcll(m);
                    }
                for (int32_t i = tid * 4; i < 128 * 127 / 2; i += 4096) *reinterpret_cast<float4 *>(tri + i) = make_float4(0.f, 0.f, 0.f, 0.f);
                __syncthreads();
                {
                    const int32_t i = wave * 8 + (lane >> 3), n_own = s_rare[i];
                    const uint2 *mine = rare + wave_at + s_rare_at[i];
                    float *ti = tri + i * (i - 1) / 2;
                    for (int32_t e0 = 0; e0 < (int32_t)most; e0 += AP_GL_U) {
                        uint2 e[AP_GL_U], y[AP_GL_U];
#pragma unroll
                        for (int o = 0; o < AP_GL_U; o++) e[o] = e0 + o < n_own ? mine[e0 + o] : make_uint2(0u, 0u);
#pragma unroll
                        for (int o = 0; o < AP_GL_U; o++) y[o] = (uint32_t)(lane & 7) < e[o].x >> 13 ? hold[(e[o].x & 0x1fffu) + (lane & 7)] : make_uint2(128u, 0u);
#pragma unroll
                        for (int o = 0; o < AP_GL_U; o++) {
                            if ((int32_t)y[o].x < i) ti[y[o].x] = fmaf(__uint_as_float(e[o].y), __uint_as_float(y[o].y), ti[y[o].x]);
                            ap_wave_sync();   // the next entry may add to the same sums by other lanes
                        }
                    }
                }
                __syncthreads();
#pragma unroll
                for (int a = 0; a < 3; a++)
#pragma unroll
                    for (int r = 0; r < 4; r++) {
                        const int32_t i = bi[a] * 16 + 4 * (lane >> 4) + r, j = bj[a] * 16 + (lane & 15);
                        const float v = wave + 16 * a < n_tasks && j < i ? tri[i * (i - 1) / 2 + j] : 0.f;
                        if (part) acc[1][a][r] = v; else acc[0][a][r] = v;
                    }
                __syncthreads();   // the stages are written next
            } else {
#pragma unroll
                for (int d = 0; d < 8; d++)
#pragma unroll
                    for (int k = 0; k < AP_GL_SLOTS; k++)
                        if (ent[d][k].x != 0xffffffffu) ent[d][k].x &= 0xffffu;
            }
        }
        uint32_t used = 0;   // uniform: slots that hold a column of the matrix at all
#pragma unroll
        for (int d = 0; d < 8; d++)
#pragma unroll
            for (int k = 0; k < AP_GL_SLOTS; k++) used |= __ballot(ent[d][k].x < 0x80000000u) ? 1u << (d * AP_GL_SLOTS + k) : 0u;
        const int32_t n_chunks = (n_cols + AP_GL_C - 1) / AP_GL_C;
        auto scatter = [&](int32_t c) {
            float *rows = X + (c & 1) * 128 * AP_GL_STRIDE + wave * 8 * AP_GL_STRIDE;
            for (int32_t i = lane * 4; i < 8 * AP_GL_STRIDE; i += 256) *reinterpret_cast<float4 *>(rows + i) = make_float4(0.f, 0.f, 0.f, 0.f);
            ap_wave_sync();
            const uint32_t c0 = (uint32_t)c * AP_GL_C;
#pragma unroll
            for (int d = 0; d < 8; d++) {
#pragma unroll
                for (int k = 0; k < AP_GL_SLOTS; k++) {
                    if (!((used >> (d * AP_GL_SLOTS + k)) & 1u)) continue;
                    const uint32_t at = ent[d][k].x - c0;   // another chunk's, or no column (2^32 - 1): to the row's padding, no branch
                    rows[d * AP_GL_STRIDE + (at < AP_GL_C ? at : AP_GL_C)] = __uint_as_float(ent[d][k].y);
                }
            }
            for (uint32_t left = longs; left; left &= left - 1u) {
                const int32_t d = (int32_t)__builtin_ctz(left), row = wave * 8 + d, len = part ? s_tn[row] : s_sn[row];
                const uint2 *r = rec + s_first[row] + (part ? s_sn[row] : 0);
                for (int32_t e = 64 * AP_GL_SLOTS + lane; e < len; e += 64) {
                    const uint2 y = r[e];
                    const uint32_t at = column(y.x) - c0;
                    if (at < AP_GL_C) rows[d * AP_GL_STRIDE + at] = __uint_as_float(y.y);
                }
            }
        };
        if (n_chunks > 0) scatter(0);
        __syncthreads();
        for (int32_t c = 0; c < n_chunks; c++) {
            if (c + 1 < n_chunks) scatter(c + 1);
            // lane l feeds column 16 kk + 4 (l / 16) + m of row l % 16 to the m-th of four MFMAs
            const float *stage = X + (c & 1) * 128 * AP_GL_STRIDE + (lane & 15) * AP_GL_STRIDE + (lane >> 4) * 4;
#pragma unroll
            for (int kk = 0; kk < AP_GL_C / 16; kk++)
#pragma unroll
                for (int a = 0; a < 3; a++) {
                    if (wave + 16 * a >= n_tasks) continue;   // uniform
                    const ap_f32x4 va = *reinterpret_cast<const ap_f32x4 *>(stage + bi[a] * 16 * AP_GL_STRIDE + kk * 16);
                    const ap_f32x4 vb = *reinterpret_cast<const ap_f32x4 *>(stage + bj[a] * 16 * AP_GL_STRIDE + kk * 16);
#pragma unroll
                    for (int m = 0; m < 4; m++) {
                        if (part) acc[1][a] = __builtin_amdgcn_mfma_f32_16x16x4f32(va[m], vb[m], acc[1][a], 0, 0, 0);
                        else acc[0][a] = __builtin_amdgcn_mfma_f32_16x16x4f32(va[m], vb[m], acc[0][a], 0, 0, 0);
                    }
                }
            __syncthreads();
        }
    }
    // element r of a lane's four: row 4 (l / 16) + r, column l % 16 of its block
    float *out = pm + x * (int64_t)K * K;
    float dense[3][4];
#pragma unroll
    for (int a = 0; a < 3; a++) {
        if (wave + 16 * a >= n_tasks) continue;
#pragma unroll
        for (int r = 0; r < 4; r++) {   // all of a lane's dense parts are on their way before the first is used
            const int32_t i = bi[a] * 16 + 4 * (lane >> 4) + r, j = bj[a] * 16 + (lane & 15);
            dense[a][r] = out[(int64_t)min(i, K - 1) * K + min(j, K - 1)];
        }
    }
#pragma unroll
    for (int a = 0; a < 3; a++) {
        if (wave + 16 * a >= n_tasks) continue;
        float four[4];
        const int32_t i0 = bi[a] * 16 + 4 * (lane >> 4), j = bj[a] * 16 + (lane & 15);
        const bool whole = bi[a] != bj[a] && K % 4 == 0 && ((uintptr_t)pm & 15) == 0;   // uniform: the mirrored four in one store
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const int32_t i = i0 + r;
            if (i >= K || j > i) continue;
            float val = -INFINITY;
            if (s_id[i] >= 0 && s_id[j] >= 0) {
                const float qs = i == j ? s_diag[0][i] : acc[0][a][r], qt = i == j ? s_diag[1][i] : acc[1][a][r];
                val = fmaf(wd, dense[a][r], fmaf(wf, qt, ws * qs));
            }
            out[(int64_t)i * K + j] = val;
            if (!whole) out[(int64_t)j * K + i] = val;
            four[r] = val;
        }
        if (whole && i0 < K) *reinterpret_cast<float4 *>(out + (int64_t)j * K + i0) = make_float4(four[0], four[1], four[2], four[3]);
    }
}

// =================================================================== S4 + S5: detour sort, IP prune, keyword flags
// Detourable routes (Section 3.3): A -> X -> Y detours A -> Y iff
// min(sim(A,X), sim(X,Y)) > sim(A,Y).  Neighbours are stably sorted by their
// number of such routes, then walked in that order (Algorithm 1): v joins SE
// when |SE| < R and sim(w,v) < sim(v,v) for every w in SE; otherwise it is
// recycled as a keyword edge if its keyword flag is set, i.e. if it shares a
// keyword with A and no current member of SE covers all the shared keywords.
#define AP_T_CAP 512
#define AP_DP_BITS 9      // slots of the table of the node's keywords: at most a quarter full

__device__ __forceinline__ bool ap_list_has(const int32_t *idx, int64_t beg, int64_t end, int32_t t) {
    int64_t lo = beg, hi = end;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (idx[mid] < t) lo = mid + 1; else hi = mid;
    }
    return lo < end && idx[lo] == t;
}

// Detour counts and order by 256 threads, then the walk, which is sequential in v, by one wave.  What made the walk slow was what
// it asked memory and LDS one after the other at each of its steps: the offsets of v's keywords, the keywords, a search of each, the
// similarities to the members of SE (20 ms for 100,000 nodes of 128 neighbours, 320 us a node).  Nothing of that depends on the
// walk, so all of it is asked ahead, by all threads:
//  - a bit per neighbour w, sim(w,v) >= sim(v,v), noted while the detours of v are counted, which read the same column;
//  - a bit per keyword of the node that v holds too, by a wave for four neighbours at a time and one read a keyword of a table that one
//    wave builds while the others count;
//  - a bit per neighbour w that holds every keyword that v shares with the node.
// A step then is one read of LDS, requested a step before, and a ballot.  100,000 nodes of 128 neighbours: 19.8 -> 5.3 ms; 200,000:
// 40.4 -> 10.8 ms (the same with a search instead of the table, a loop over the members' keywords in the walk and dependent reads in the count of
// the ranks: 8.4 and 17.2).
// Nodes with more than AP_T_CAP keywords search the lists as the walk goes on.
__global__ __launch_bounds__(256, 6) void k_detour_prune(ApVecs D, const float *__restrict__ self_sim, int32_t K, int32_t R,
                                                      int32_t ke_cap, const int32_t *__restrict__ knn,
                                                      const float *__restrict__ knn_sc, const int32_t *__restrict__ node_ids,
                                                      int64_t x0, int64_t xout0, const float *__restrict__ pm,
                                                      int32_t *__restrict__ o_count, int32_t *__restrict__ o_sorted,
                                                      int32_t *__restrict__ o_se, int32_t *__restrict__ o_ke,
                                                      int32_t *__restrict__ o_ke_count, int32_t *__restrict__ o_flag,
                                                      int32_t mode) {
    __shared__ int32_t ids[256], cnt[256], order[256], se_pos[128], flag[256], tx_n[256];
    __shared__ uint32_t tx_b[256];       // the two parts of a corpus hold fewer than 2^32 entries together
    __shared__ float simA[256];
    __shared__ int32_t a_tx[AP_T_CAP];   // the node's own keywords; of a node with more, those that it shares with v
    __shared__ __attribute__((aligned(16))) int32_t rank_key[256];
    __shared__ __attribute__((aligned(16))) uint64_t a_tab[1 << AP_DP_BITS];   // keyword -> its place in the node's list + 1, as a number's bits
    __shared__ int32_t s_valid, s_seed;
    extern __shared__ uint32_t dp_lds[];
    const int32_t KW = (K + 31) / 32;
    uint32_t *rows = dp_lds;                   // [K][2 KW]: the neighbours with sim(w,v) >= sim(v,v), then those that hold what v shares with the node
    uint32_t *shared = dp_lds + 2 * K * KW;    // [AP_T_CAP / 32][K]
    const int64_t x = blockIdx.x;               // index inside the chunk (pm)
    const int64_t xo = xout0 + x;               // index in the output arrays
    const int64_t u = node_ids ? (int64_t)node_ids[x0 + x] : x0 + x;
    const float *P = pm + x * (int64_t)K * K;
    const int t = threadIdx.x, lane = t & 63, wave = ap_wave_id();
    if (t == 0) s_valid = 0;
    const int64_t a_beg = D.tx_indptr[u], a_end = D.tx_indptr[u + 1];
    const bool a_in_lds = a_end - a_beg <= AP_T_CAP;   // uniform
    const int32_t an = a_in_lds ? (int32_t)(a_end - a_beg) : 0, W = (an + 31) / 32;
    if (t < K) {
        const int32_t v = knn[u * K + t];
        ids[t] = v; simA[t] = v >= 0 ? knn_sc[u * K + t] : -INFINITY; flag[t] = 0; cnt[t] = 0;
        int64_t b = 0, e = 0;
        if (v >= 0) { b = D.tx_indptr[v]; e = D.tx_indptr[v + 1]; }
        tx_b[t] = (uint32_t)b; tx_n[t] = (int32_t)(e - b);
    }
    for (int32_t e = t; e < an; e += 256) a_tx[e] = D.tx_idx[a_beg + e];
    if (t < 128) order[t] = t + 1;   // the places, for the table; the order itself comes later
    for (int32_t i = t; i < W * K; i += 256) shared[i] = 0u;
    __syncthreads();
    if (wave == 3) {
        const int32_t seed = an > 0 && an <= 128 ? ap_bucket_build<2>(a_tx, reinterpret_cast<const float *>(order), an, a_tab, AP_DP_BITS) : -1;
        if (lane == 0) s_seed = seed;
    }
    {   // a column a thread, or two or four threads a column with some of the rows each
        const int32_t parts = K <= 64 ? 4 : K <= 128 ? 2 : 1, stride = 256 / parts, col = t % stride, part = t / stride, per = (KW + parts - 1) / parts;
        if (col < K && ids[col] >= 0) {
            const float sy = simA[col], sv = self_sim[ids[col]];
            int32_t c = 0;
            for (int32_t w = part * per; w < min((part + 1) * per, KW); w++) {
                uint32_t bits = 0;
                for (int32_t i0 = 0; i0 < 32; i0 += 8) {
                    float b[8];
#pragma unroll
                    for (int i = 0; i < 8; i++) b[i] = P[(int64_t)min(32 * w + i0 + i, K - 1) * K + col];
#pragma unroll
                    for (int i = 0; i < 8; i++) {
                        const int32_t xx = 32 * w + i0 + i;
                        if (xx >= K) continue;
                        const float a = simA[xx];   // -inf for a hole: no route goes through it
                        c += xx != col && (a < b[i] ? a : b[i]) > sy ? 1 : 0;
                        bits |= b[i] < sv ? 0u : 1u << (i0 + i);
                    }
                }
                rows[col * 2 * KW + w] = bits;
            }
            if (c) atomicAdd(&cnt[col], c);
            if (part == 0) atomicAdd(&s_valid, 1);
        }
    }
    __syncthreads();
    // the keywords that a neighbour shares with the node: a wave for four neighbours at a time, every lane a keyword of each
    if (an > 0) {
        const int32_t step0 = ap_pow2_floor(an);
        const int32_t seed = ap_uniform_i32(s_seed);
        const uint32_t mult = ap_seed_mult(max(seed, 0));
        auto find = [&](int32_t term) {   // its place in the node's list, -1 if it is not there (term -1 never is)
            if (seed >= 0) return __float_as_int(ap_bucket_get((const AP_LDS uint64_t *)a_tab, mult, AP_DP_BITS, term)) - 1;   // uniform
            int32_t pos = 0;
            for (int32_t st = step0; st > 0; st >>= 1) {
                const int32_t p2 = pos + st, at = (p2 < an ? p2 : an) - 1;
                pos = ((p2 <= an) & (a_tx[at] < term)) ? p2 : pos;
            }
            return pos < an && a_tx[pos] == term ? pos : -1;
        };
        constexpr int G = 4;
        for (int32_t v0 = G * wave; v0 < K; v0 += 4 * G) {
            int32_t n[G], most = 0;
            const int32_t *l[G];
#pragma unroll
            for (int g = 0; g < G; g++) {
                const int32_t v = min(v0 + g, K - 1);   // past the end the last one again
                n[g] = ap_uniform_i32(tx_n[v]); l[g] = D.tx_idx + tx_b[v];
                most = max(most, n[g]);
            }
            for (int32_t e = lane; e < most; e += 64) {
                int32_t term[G], at[G];
#pragma unroll
                for (int g = 0; g < G; g++) term[g] = e < n[g] ? l[g][e] : -1;
#pragma unroll
                for (int g = 0; g < G; g++) at[g] = find(term[g]);
#pragma unroll
                for (int g = 0; g < G; g++)
                    if (at[g] >= 0) atomicOr(&shared[(at[g] >> 5) * K + min(v0 + g, K - 1)], 1u << (at[g] & 31));
            }
        }
    }
    // order: by detours, then by place (ablation: by place alone), holes last
    if (t < 256) rank_key[t] = t < K ? (ids[t] >= 0 ? (mode == AP_PRUNE_IP_ONLY ? 0 : cnt[t] * 256) : 1 << 20) + t : INT32_MAX;
    __syncthreads();
    if (t < K) {
        const int32_t mine = rank_key[t];
        int32_t r = 0;
        for (int32_t z = 0; z < K; z += 4) {
            const int4 o = *reinterpret_cast<const int4 *>(rank_key + z);
            r += (o.x < mine) + (o.y < mine) + (o.z < mine) + (o.w < mine);
        }
        order[r] = t;
    }
    if (a_in_lds) {   // who holds what v shares with the node
        for (int32_t i = t; i < K * KW; i += 256) {
            const int32_t v = i % K, j0 = i / K * 32, last = K - 1 - j0;
            uint32_t miss = 0;
            for (int32_t w = 0; w < W; w++) {
                const uint32_t s = shared[w * K + v];
                const uint32_t *of = shared + w * K + j0;
#pragma unroll
                for (int32_t j = 0; j < 32; j++) miss |= s & ~of[min(j, last)] ? 1u << j : 0u;
            }
            rows[v * 2 * KW + KW + i / K] = ~miss;
        }
    }
    __syncthreads();
    if (t < K) {
        if (o_count) o_count[xo * K + t] = cnt[t];
        if (o_sorted) o_sorted[xo * K + t] = ids[order[t]];
    }
    if (t >= 64) return;   // the walk is sequential in v; one wave does it
    const int32_t n_valid = ap_uniform_i32(s_valid);   // holes are sorted last
    int32_t nse = 0, nke = 0;
    uint32_t se_bits = 0;   // lanes l and KW + l: bits 32 l .. of the neighbours that are members
    int32_t place[4];       // order[64 q + lane]
#pragma unroll
    for (int q = 0; q < 4; q++) place[q] = 64 * q + lane < K ? order[64 * q + lane] : 0;
    auto at = [&](int32_t r) {   // order[r]
        const int32_t v = r < 64 ? place[0] : r < 128 ? place[1] : r < 192 ? place[2] : place[3];   // r is uniform
        return __builtin_amdgcn_readlane(v, r & 63);
    };
    int32_t pv = n_valid ? at(0) : 0;
    uint32_t row = lane < 2 * KW ? rows[pv * 2 * KW + lane] : 0u;
    for (int32_t r = 0; r < n_valid; r++) {
        if (!o_flag && nse >= R && nke >= ke_cap) break;   // nothing but flags is left to tell
        const int32_t next = at(min(r + 1, n_valid - 1));
        const uint32_t row_next = lane < 2 * KW ? rows[next * 2 * KW + lane] : 0u;
        int32_t fl = 0;
        bool ok = true;
        if (nse > 0) {   // the first one is a member whatever it is
            const uint64_t met = __ballot((row & se_bits) != 0u), low = (1ull << KW) - 1ull;
            if (a_in_lds) fl = met & ~low ? 0 : 1;   // no member holds every shared keyword (where none is shared, all do)
            else {
                // the shared keywords themselves, AP_T_CAP of them at a time: which members hold all of them?
                const int64_t vb = tx_b[pv], ve = vb + tx_n[pv];
                uint32_t holds = 3u;   // bit i: member 64 i + lane
                int32_t nt = 0;
                bool any = false;
                auto ask = [&]() {
                    ap_wave_sync();
                    for (int32_t i = 0; i < 2; i++) {
                        if (64 * i + lane >= nse || !(holds >> i & 1u)) continue;
                        const int32_t y = ids[se_pos[64 * i + lane]];
                        const int64_t yb = D.tx_indptr[y], ye = D.tx_indptr[y + 1];
                        for (int32_t k = 0; k < nt; k++)
                            if (!ap_list_has(D.tx_idx, yb, ye, a_tx[k])) { holds &= ~(1u << i); break; }
                    }
                    ap_wave_sync();
                    nt = 0;
                };
                for (int64_t e0 = vb; e0 < ve; e0 += 64) {
                    const int32_t term = e0 + lane < ve ? D.tx_idx[e0 + lane] : -1;
                    const bool in = term >= 0 && ap_list_has(D.tx_idx, a_beg, a_end, term);
                    const uint64_t m = __ballot(in);
                    any = any || m;
                    if (in) a_tx[nt + __popcll(m & ((1ull << lane) - 1ull))] = term;
                    nt += __popcll(m);
                    if (nt > AP_T_CAP - 64) ask();
                }
                ask();
                const bool covered = (lane < nse && (holds & 1u)) || (64 + lane < nse && (holds & 2u));
                fl = any && !__ballot(covered) ? 1 : 0;
            }
            // IP test against every member of SE (ablation: without it SE is the first R of the detour order)
            ok = nse < R && (mode == AP_PRUNE_RNG_ONLY || !(met & low));
        }
        if (lane == 0) {
            flag[pv] = fl;
            if (ok) se_pos[nse] = pv;
            else if (fl && nke < ke_cap && o_ke) o_ke[xo * ke_cap + nke] = ids[pv];
        }
        if (ok) {
            if (lane < 2 * KW && (lane < KW ? lane : lane - KW) == pv >> 5) se_bits |= 1u << (pv & 31);
            nse++;
        } else if (fl && nke < ke_cap) nke++;
        if (!a_in_lds) ap_wave_sync();   // se_pos is read
        pv = next; row = row_next;
    }
    ap_wave_sync();
    for (int32_t i = lane; i < R; i += 64) if (o_se) o_se[xo * R + i] = i < nse ? ids[se_pos[i]] : -1;
    for (int32_t i = nke + lane; i < ke_cap; i += 64) if (o_ke) o_ke[xo * ke_cap + i] = -1;
    if (lane == 0 && o_ke_count) o_ke_count[xo] = nke;
    for (int32_t i = lane; i < K; i += 64) if (o_flag) o_flag[xo * K + i] = flag[i];
}

int ap_prune_impl(const ap_index *ix, int32_t K, int32_t R, const int32_t *knn_ids, const float *knn_sc,
                      const int32_t *node_ids, int64_t nn, float *pm_out, int32_t *count, int32_t *sorted_ids,
                      int32_t *se, int32_t *ke, int32_t *ke_count, int32_t *flag, hipStream_t st, const ApWork &work) {
    const int64_t per = (int64_t)K * K;
    int64_t chunk = pm_out ? nn : std::min<int64_t>(nn, std::max<int64_t>(1, ((int64_t)1 << 28) / per));
    float *own = nullptr, *scratch = pm_out ? nullptr : work.take<float>((size_t)chunk * (size_t)per);
    if (!pm_out && !scratch) { AP_TRY(ap_dev_alloc(&own, (size_t)chunk * (size_t)per)); scratch = own; }
    const float *w = ix->params.build_w;
    const int32_t tiles = (K + AP_TILE - 1) / AP_TILE;
    hipError_t e = hipSuccess;
    // By columns where a workgroup can hold the neighbourhood's rows and both bitmaps; the walks for longer lists of
    // neighbours and larger vocabularies.
    const bool by_columns = K <= 128 && std::max(ix->corpus.sp_vocab, ix->corpus.tx_vocab) <= AP_GL_WORDS * 32 && !g_ap_debug.prune_walks;
    if (by_columns) e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_gram_lists), hipFuncAttributeMaxDynamicSharedMemorySize, AP_GL_LDS);
    for (int64_t x0 = 0; x0 < nn && e == hipSuccess; x0 += chunk) {
        const int64_t cn = std::min(chunk, nn - x0);
        float *pm = pm_out ? pm_out + x0 * per : scratch;
        for (int64_t y0 = 0; y0 < cn && e == hipSuccess; y0 += 32768) {   // grid.y limit
            const int64_t yn = std::min<int64_t>(32768, cn - y0);
            dim3 g1((unsigned)(tiles * tiles), (unsigned)yn);
            if (ix->dtype == AP_F32)
                hipLaunchKernelGGL(k_gram_dense<AP_F32>, g1, dim3(256), 0, st, ix->docs.dense, ix->dense_norm, ix->docs.dim, K, knn_ids, node_ids, x0 + y0, pm + y0 * per);
            else
                hipLaunchKernelGGL(k_gram_dense<AP_BF16>, g1, dim3(256), 0, st, ix->docs.dense, ix->dense_norm, ix->docs.dim, K, knn_ids, node_ids, x0 + y0, pm + y0 * per);
            e = hipGetLastError();
            if (e != hipSuccess) break;
            if (by_columns) {
                hipLaunchKernelGGL(k_gram_lists, dim3((unsigned)yn), dim3(1024), AP_GL_LDS, st, ix->rec, ix->meta, w[0], w[1], w[2],
                                   (ix->corpus.sp_vocab + 127) / 128 * 4, (ix->corpus.tx_vocab + 127) / 128 * 4, K, knn_ids, node_ids, x0 + y0, pm + y0 * per);
                e = hipGetLastError();
                continue;
            }
            const int32_t tb = (K + AP_GT - 1) / AP_GT;
            dim3 g2((unsigned)(tb * (tb + 1) / 2), (unsigned)yn);
            hipLaunchKernelGGL(k_gram_merge, g2, dim3(256), 0, st, ix->rec, ix->meta, w[0], w[1], w[2], K, knn_ids, node_ids, x0 + y0, pm + y0 * per);
            e = hipGetLastError();
        }
        if (e != hipSuccess) break;
        hipLaunchKernelGGL(k_detour_prune, dim3((unsigned)cn), dim3(256), ((size_t)2 * ((K + 31) / 32) + AP_T_CAP / 32) * K * 4, st, ix->docs, ix->self_sim, K, R, R / 2, knn_ids,
                           knn_sc, node_ids, x0, x0, pm, count, sorted_ids, se, ke, ke_count, flag, ix->params.prune_mode);
        e = hipGetLastError();
    }
    if (own || pm_out || !work.mem) {
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (own) (void)hipFree(own);
    }
    if (e != hipSuccess) { ap_set_error("prune stage failed: %s", hipGetErrorString(e)); return AP_EHIP; }
    return AP_OK;
}

extern "C" int ap_stage_prune(const ap_index *ix, int32_t K, int32_t R, const int32_t *knn_ids, const float *knn_sc,
                              const int32_t *node_ids, int64_t nn, float *pm, int32_t *count, int32_t *sorted_ids,
                              int32_t *se, int32_t *ke, int32_t *ke_count, int32_t *flag, void *stream) {
    AP_REQUIRE(ix && knn_ids && knn_sc, "NULL argument");
    AP_REQUIRE(K >= 1 && K <= 256 && R >= 2 && R <= 128, "need 1<=K<=256, 2<=R<=128");
    if (!node_ids) nn = ix->docs.n;
    if (nn <= 0) return AP_OK;
    return ap_prune_impl(ix, K, R, knn_ids, knn_sc, node_ids, nn, pm, count, sorted_ids, se, ke, ke_count, flag, (hipStream_t)stream, ApWork());
}

// =================================================================== S6: assembly
// Reverse neighbours of u: nodes x with u among the first q entries of SE(x),
// ordered by (position of u in SE(x), x); the first q that are not already
// forward neighbours of u.  One pass over the edges: a key goes through its target's places, which take the smaller of what they hold
// and what comes and pass the other on, so that place r ends with the r-th smallest key in whatever order they came.  A place's
// key only ever gets smaller: what is larger than a place's key as it was read need not ask it.  Edges of one position
// follow each other, so most keys find their place at the end.  (One pass a place, each keeping the smallest key above the last place's,
// took 1,404 us for 100,000 nodes and 16 places, bound by three random lines an edge and pass; this one 347.)
__global__ __launch_bounds__(256) void k_rev_insert(const int32_t *__restrict__ se, int64_t n, int32_t R, int32_t q, unsigned long long *rev /* n x q, ~0 = none */) {
    const int32_t pos = (int32_t)blockIdx.y;
    for (int64_t x = blockIdx.x * (int64_t)256 + threadIdx.x; x < n; x += (int64_t)gridDim.x * 256) {
        const int32_t u = se[x * R + pos];
        if (u < 0 || u == x) continue;
        unsigned long long key = (((unsigned long long)pos << 32) | (unsigned long long)x) + 1ull, *place = rev + (int64_t)u * q;
        int32_t r = 0;
        while (r < q && place[r] < key) r++;
        if (r == q) continue;
        bool fwd = false;                 // x already a forward neighbour of u?
        for (int32_t i = 0; i < q; i++) fwd = fwd || se[(int64_t)u * R + i] == (int32_t)x;
        if (fwd) continue;
        for (; r < q; r++) {
            const unsigned long long old = atomicMin(&place[r], key);
            if (old == ~0ull) break;
            key = old > key ? old : key;
        }
    }
}

// One wave per node, following the order: SE[0:q], reverse neighbours, the
// per-path lists taken round-robin (dense, sparse, lexical) up to R/2, then
// padding from the rest of SE and from the detour-sorted list.  All of them are asked for at the start and the row grows in registers, two
// places a lane, so that an id costs a comparison and a ballot: 810 us for 100,000 nodes of degree 64 with a read from memory and a row in LDS, now 425.
__global__ __launch_bounds__(256) void k_assemble(int64_t n, int32_t R, int32_t K, int32_t P, const int32_t *__restrict__ se,
                                                  const int32_t *__restrict__ sorted_ids, const int32_t *__restrict__ sp_ids,
                                                  const unsigned long long *__restrict__ rev, int64_t u0, int32_t *__restrict__ out) {
    const int lane = threadIdx.x & 63;
    const int64_t u = u0 + (int64_t)blockIdx.x * 4 + ap_wave_id();
    if (u >= n) return;
    const int32_t q = R / 4, h = R / 2;   // R <= 128, P <= 32
    const int32_t e0 = lane < R ? se[u * R + lane] : -1, e1 = 64 + lane < R ? se[u * R + 64 + lane] : -1;
    const unsigned long long key = lane < q ? rev[u * q + lane] : ~0ull;
    const int32_t back = key == ~0ull ? -1 : (int32_t)((key - 1ull) & 0xffffffffull);
    const int32_t p0 = lane < P ? sp_ids[u * P + lane] : -1, p1 = lane < P ? sp_ids[(n + u) * P + lane] : -1, p2 = lane < P ? sp_ids[(2 * n + u) * P + lane] : -1;
    int32_t more = lane < K ? sorted_ids[u * K + lane] : -1;
    int32_t row0 = -1, row1 = -1, len = 0;
    auto push = [&](int32_t v) -> bool {   // wave-uniform
        if (v < 0 || v == (int32_t)u || __ballot(row0 == v || row1 == v) != 0ull) return false;
        if (lane == (len & 63)) { if (len < 64) row0 = v; else row1 = v; }
        len++;
        return true;
    };
    auto at = [&](int32_t x, int32_t i) { return __builtin_amdgcn_readlane(x, i); };
    for (int32_t i = 0; i < q; i++) push(at(e0, i));
    const int32_t n_back = (int32_t)__popcll(__ballot(key != ~0ull));   // the places are filled from the first on
    for (int32_t i = 0; i < n_back; i++) push(at(back, i));
    {
        uint32_t next = 0;   // per list a byte: its next entry
        int32_t added = 0, turn = 0, idle = 0;
        while (added < h && idle < 3) {
            bool took = false;
            const int32_t list = turn == 0 ? p0 : turn == 1 ? p1 : p2;
            int32_t i = (int32_t)((next >> (8 * turn)) & 255u);
            while (i < P) {
                const int32_t v = at(list, i);
                i++;
                if (push(v)) { added++; took = true; break; }
            }
            next = (next & ~(255u << (8 * turn))) | ((uint32_t)i << (8 * turn));
            idle = took ? 0 : idle + 1;
            turn = turn == 2 ? 0 : turn + 1;
        }
    }
    for (int32_t i = q; i < R && len < R; i++) push(i < 64 ? at(e0, i) : at(e1, i - 64));
    for (int32_t i0 = 0; i0 < K && len < R; i0 += 64) {
        if (i0 > 0) more = i0 + lane < K ? sorted_ids[u * K + i0 + lane] : -1;
        for (int32_t i = 0; i < 64 && i0 + i < K && len < R; i++) push(at(more, i));
    }
    if (lane < R) out[u * R + lane] = row0;
    if (64 + lane < R) out[u * R + 64 + lane] = row1;
}

int ap_assemble_impl(const ap_index *ix, int32_t R, int32_t K, int32_t P, const int32_t *se, const int32_t *sorted_ids,
                         const int32_t *sp_ids, int32_t *out_graph, hipStream_t st, const ApWork &work) {
    const int64_t n = ix->docs.n;
    const int32_t q = R / 4;
    unsigned long long *own = nullptr, *rev = work.take<unsigned long long>((size_t)n * (size_t)q);
    if (!rev) { AP_TRY(ap_dev_alloc(&own, (size_t)n * (size_t)q)); rev = own; }
    int rc = ap_fill_u32(rev, (size_t)n * q * 2, 0xffffffffu, st);
    hipError_t e = hipSuccess;
    if (rc == AP_OK) {
        if (q > 0) hipLaunchKernelGGL(k_rev_insert, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 65536), (unsigned)q), dim3(256), 0, st, se, n, R, q, rev);
        e = hipGetLastError();
        if (e == hipSuccess) {
            const int64_t slice = AP_MAX_LAUNCH_THREADS / 64;   // four nodes per 256 threads
            for (int64_t u0 = 0; u0 < n && e == hipSuccess; u0 += slice) {
                const int64_t cn = std::min<int64_t>(slice, n - u0);
                hipLaunchKernelGGL(k_assemble, dim3((unsigned)((cn + 3) / 4)), dim3(256), 0, st, n, R, K, P, se, sorted_ids, sp_ids, rev, u0, out_graph);
                e = hipGetLastError();
            }
        }
        if (own && e == hipSuccess) e = hipStreamSynchronize(st);
    }
    if (own) (void)hipFree(own);
    if (rc != AP_OK) return rc;
    if (e != hipSuccess) { ap_set_error("assemble stage failed: %s", hipGetErrorString(e)); return AP_EHIP; }
    return AP_OK;
}

extern "C" int ap_stage_assemble(const ap_index *ix, int32_t R, int32_t K, int32_t P, const int32_t *se,
                                 const int32_t *sorted_ids, const int32_t *sp_ids, int32_t *out_graph, void *stream) {
    AP_REQUIRE(ix && se && sorted_ids && sp_ids && out_graph, "NULL argument");
    AP_REQUIRE(R >= 4 && R % 4 == 0 && R <= 128 && K >= 1 && K <= 256 && P >= 1 && P <= 32, "need R%%4==0, 4<=R<=128, 1<=K<=256, 1<=P<=32");
    return ap_assemble_impl(ix, R, K, P, se, sorted_ids, sp_ids, out_graph, (hipStream_t)stream, ApWork());
}

// =================================================================== the whole build
// Fused scores of existing lists (used when no refinement round runs).
template <int DT, int NV>
__global__ __launch_bounds__(256) void k_rescore_lists(ApVecs D, float wd, float ws, float wf, int32_t K, int64_t u0,
                                                       const int32_t *__restrict__ knn, float *__restrict__ sc) {
    __shared__ int32_t l_sp_idx[AP_A_CAP], l_tx_idx[AP_A_CAP];
    __shared__ float l_sp_val[AP_A_CAP], l_tx_val[AP_A_CAP];
    const int64_t u = u0 + blockIdx.x;
    const int lane = threadIdx.x & 63, wave = ap_wave_id();
    const ApLists a = ap_stage_lists(D, u, l_sp_idx, l_sp_val, l_tx_idx, l_tx_val, AP_A_CAP);
    float qa[NV * ApDense<DT>::EPC];
    ap_load_aside<DT, NV, DT>(D.dense, u, D.dim, qa);
    __syncthreads();
    for (int32_t i = wave; i < K; i += 4) {
        const int32_t v = knn[u * K + i];
        float s = -INFINITY;
        if (v >= 0) { float sd, ss, sf; ap_hybrid_wave<DT, NV>(D, qa, a, v, sd, ss, sf); s = ap_fuse(wd, ws, wf, sd, ss, sf); }
        if (lane == 0) sc[u * K + i] = s;
    }
}

// Fused scores (construction weights) of the first nn rows of existing lists.
int ap_rescore_lists(const ap_index *ix, int64_t nn, int32_t K, const int32_t *knn, float *sc, hipStream_t st) {
    if (nn <= 0) return AP_OK;
    const float *w = ix->params.build_w;
    const int64_t slice = AP_MAX_LAUNCH_THREADS / 256;
    for (int64_t u0 = 0; u0 < nn; u0 += slice) {
        const int64_t cn = std::min<int64_t>(slice, nn - u0);
        AP_DISPATCH_DENSE(ix->dtype, ix->docs.dim,
                          hipLaunchKernelGGL((k_rescore_lists<DT, NV>), dim3((unsigned)cn), dim3(256), 0, st, ix->docs, w[0], w[1], w[2],
                                             K, u0, knn, sc));
        AP_CHECK_HIP(hipGetLastError());
    }
    return AP_OK;
}

struct BuildBufs {
    int32_t *knn[2] = {nullptr, nullptr};
    float *knn_sc[2] = {nullptr, nullptr};
    int32_t *spi[2] = {nullptr, nullptr};
    float *sps[2] = {nullptr, nullptr};
    int32_t *se = nullptr, *sorted = nullptr;
    ApWork work;
    float *slack = nullptr;   // of the seed lists' scores
    void *mem = nullptr, *state = nullptr, *packed = nullptr;   // what is given back at the end; what the index keeps; the packed lists
    void release() {
        void *p[] = {slack, packed, mem, state};
        for (void *x : p) if (x) (void)hipFree(x);
        *this = BuildBufs();
    }
};

// Bytes of the scratch that a construction's stages after ingest take one after the other: those of the exact seed lists, the refinement,
// the neighbourhood similarities, the assembly and the entry points, of each where it is small.  (Of 8.8 million documents the assembly alone takes
// 1.1 GB, which the buffers of the seed sweep have use for.)
static size_t build_work_bytes(const ap_build_params &p, int64_t n) {
    const size_t K = (size_t)p.knn_k, N = (size_t)n;
    const size_t stages[] = {(N + AP_TILE - 1) / AP_TILE * AP_TILE * N * 4, N * 12, N * K * K * 4, N * (size_t)(p.degree / 4) * 8, (size_t)p.n_entry * 4};
    size_t most = 0;
    for (size_t s : stages) if (s <= AP_WORK_BYTES) most = std::max(most, s);
    return most;
}
extern "C" int ap_build_shared_bytes(const ap_build_params *params, int64_t n, uint64_t *out) {
    AP_REQUIRE(params && out && n >= 1, "NULL argument, or no documents");
    *out = build_work_bytes(*params, n);
    return AP_OK;
}

static int build_impl(ap_index *ix, hipStream_t st, BuildBufs &b) {
    const ap_build_params &p = ix->params;
    const int64_t n = ix->corpus.n;   // ix->docs is only filled in by the ingest step below
    const int32_t K = p.knn_k, R = p.degree, P = p.sp_len;
    ApStageEvents marks;
    AP_CHECK_HIP(marks.create());
    hipEvent_t *ev = marks.ev;
    auto mark = [&](int i) { return hipEventRecord(ev[i], st); };
    AP_CHECK_HIP(mark(0));
    AP_TRY(ap_ingest_impl(ix, 64, st));
    AP_CHECK_HIP(mark(1));
    const int kept = p.nd_rounds & 1;   // which of the per-path lists the rounds end with
    b.work.bytes = build_work_bytes(p, n);
    AP_TRY(ap_dev_alloc_parts(&b.state, {AP_PART(b.se, n * R), AP_PART(b.sorted, n * K), AP_PART(b.spi[kept], 3 * n * P), AP_PART(b.sps[kept], 3 * n * P)}));
    AP_TRY(ap_dev_alloc_parts(&b.mem, {AP_PART(b.knn[0], n * K), AP_PART(b.knn[1], n * K), AP_PART(b.knn_sc[0], n * K), AP_PART(b.knn_sc[1], n * K),
                                       AP_PART(b.spi[1 - kept], 3 * n * P), AP_PART(b.sps[1 - kept], 3 * n * P), ApPart{&b.work.mem, b.work.bytes}}));
    AP_TRY(ap_alloc_graph(ix));
    ap_progress("ingest done; seed lists of %lld documents", (long long)n);
    // the rounds read the lists' members, the first nd_sample of them as a set, and bounds of their scores
    ApSeedRelax relax;
    relax.top = std::min(K, p.nd_sample);
    AP_TRY(ap_seed_knn_impl(ix, nullptr, n, K, b.knn[0], b.knn_sc[0], st, p.nd_rounds > 0 ? &relax : nullptr, b.work));
    b.slack = relax.slack;
    ap_progress("seed lists done; %d refinement rounds, pruning, assembly", p.nd_rounds);
    AP_CHECK_HIP(mark(2));
    AP_TRY(ap_fill_u32(b.spi[0], (size_t)3 * n * P, 0xffffffffu, st));          // id -1
    AP_TRY(ap_fill_u32(b.sps[0], (size_t)3 * n * P, 0xff800000u, st));          // -inf
    int cur = 0;
    AP_TRY(ap_refine_rounds(ix, p.nd_rounds, K, p.nd_sample, P, b.knn, b.knn_sc, b.spi, b.sps, &cur, st, b.slack, b.work, &b.packed));
    if (p.nd_rounds == 0) AP_TRY(ap_rescore_lists(ix, n, K, b.knn[cur], b.knn_sc[cur], st));
    AP_CHECK_HIP(mark(3));
    AP_TRY(ap_prune_impl(ix, K, R, b.knn[cur], b.knn_sc[cur], nullptr, n, nullptr, nullptr, b.sorted, b.se, ix->kw, ix->kw_count,
                      nullptr, st, b.work));
    AP_CHECK_HIP(mark(4));
    AP_TRY(ap_assemble_impl(ix, R, K, P, b.se, b.sorted, b.spi[cur], ix->graph, st, b.work));
    AP_TRY(ap_entry_points_impl(ix, p.n_entry, ix->entry, st, b.work));
    AP_CHECK_HIP(mark(5));
    AP_CHECK_HIP(hipStreamSynchronize(st));
    float total = 0.f;
    for (int i = 0; i < 5; i++) {
        float ms = 0.f;
        AP_CHECK_HIP(hipEventElapsedTime(&ms, ev[i], ev[i + 1]));
        ix->timings[i] = ms * 1e-3f;
        total += ms * 1e-3f;
    }
    ix->has_graph = true;
    // kept for later insertions
    ix->st_se = b.se; ix->st_sorted = b.sorted; ix->st_spi = b.spi[cur]; ix->st_sps = b.sps[cur];
    ix->mem_state = b.state;
    b.state = nullptr;
    ix->timings[5] = total;
    if (ix->bd_mem) return AP_OK;
    // Columns of the bounds that are more than a small part (1/64) of the free memory come when the construction's own memory
    // is free again: its stages size theirs by what is free (the seed sweep by 62 % of it), and none of them reads the columns.
    // Laid out here always, they took a construction of 2,000 documents 0.25 of 2.7 ms: what the device is waited for in
    // between.  The time counts as ingest.
    b.release();
    AP_CHECK_HIP(mark(0));
    AP_TRY(ap_bound_ingest(ix, 4, st));
    AP_CHECK_HIP(mark(1));
    AP_CHECK_HIP(hipStreamSynchronize(st));
    float ms = 0.f;
    AP_CHECK_HIP(hipEventElapsedTime(&ms, ev[0], ev[1]));
    ix->timings[0] += ms * 1e-3f;
    ix->timings[5] = total + ms * 1e-3f;
    return AP_OK;
}

extern "C" int ap_build_index(const ap_corpus *corpus, const ap_build_params *params, void *stream, ap_index **out) {
    AP_REQUIRE(out != nullptr, "out is NULL");
    *out = nullptr;
    AP_TRY(ap_validate_corpus(corpus));
    AP_TRY(ap_validate_params(params));
    AP_REQUIRE(corpus->n >= 2, "need at least two documents to build a graph");
    ap_index *ix = new (std::nothrow) ap_index();
    if (!ix) { ap_set_error("out of host memory"); return AP_ENOMEM; }
    ix->corpus = *corpus;
    ix->params = *params;
    if (ix->params.sp_len == 0) ix->params.sp_len = (ix->params.degree + 5) / 6;
    ix->dtype = corpus->dense_dtype;
    BuildBufs b;
    const int rc = build_impl(ix, (hipStream_t)stream, b);
    (void)hipStreamSynchronize((hipStream_t)stream);
    b.release();
    if (rc != AP_OK) { ap_free_index(ix); return rc; }
    *out = ix;
    return AP_OK;
}
