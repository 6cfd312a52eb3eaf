// S1 as stand-alone calls: hybrid similarities of explicit (a, candidate)
// pairs, and the exhaustive scorer + exact top-k used as ground truth.
#include <algorithm>
#include "ap_tiles.hpp"

#define AP_LIST_CAP 512  // a-side list entries staged in LDS; longer lists are read from global memory

// One block (4 waves) per a row and chunk of candidates; wave w takes
// candidates chunk_begin + w, + 4, ...
template <int DT, int NV, int SRC>
__global__ __launch_bounds__(256) void k_hybrid_pairs(ApVecs A, ApVecs B, const int32_t *__restrict__ a_ids,
                                                      const int32_t *__restrict__ cand, int32_t c, int32_t chunk,
                                                      const float *__restrict__ w, int32_t w_stride,
                                                      float *__restrict__ out4) {
    __shared__ int32_t l_sp_idx[AP_LIST_CAP];
    __shared__ float l_sp_val[AP_LIST_CAP];
    __shared__ int32_t l_tx_idx[AP_LIST_CAP];
    __shared__ float l_tx_val[AP_LIST_CAP];
    const int64_t x = blockIdx.x;
    const int64_t row = a_ids ? (int64_t)a_ids[x] : x;
    const int32_t y0 = blockIdx.y * chunk;
    const int32_t y1 = y0 + chunk < c ? y0 + chunk : c;
    if (row < 0 || row >= A.n) {   // not a row of A: the whole line of results is holes (uniform over the workgroup)
        for (int32_t y = y0 + (int32_t)threadIdx.x; y < y1; y += blockDim.x)
            *reinterpret_cast<float4 *>(out4 + (x * c + y) * 4) = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
        return;
    }
    const ApLists a = ap_stage_lists(A, row, l_sp_idx, l_sp_val, l_tx_idx, l_tx_val, AP_LIST_CAP);
    float qa[NV * ApDense<DT>::EPC];
    ap_load_aside<DT, NV, SRC>(A.dense, row, A.dim, qa);
    __syncthreads();
    const float wd = w[x * w_stride + 0], ws = w[x * w_stride + 1], wf = w[x * w_stride + 2];
    const int lane = threadIdx.x & 63, wave = ap_wave_id();
    for (int32_t y = y0 + wave; y < y1; y += 4) {
        const int32_t j = cand[x * c + y];
        float sd, ss, sf, fu;
        if (j >= 0 && j < B.n) {
            ap_hybrid_wave<DT, NV>(B, qa, a, j, sd, ss, sf);
            fu = ap_fuse(wd, ws, wf, sd, ss, sf);
        } else {
            sd = ss = sf = fu = -INFINITY;
        }
        if (lane == 0) *reinterpret_cast<float4 *>(out4 + (x * c + y) * 4) = make_float4(sd, ss, sf, fu);
    }
}

static ApVecs query_view(const ap_queries *q, int32_t dim) {
    return ApVecs{q->nq, dim, q->dense, q->sp_indptr, q->sp_idx, q->sp_val, q->tx_indptr, q->tx_idx, q->tx_cnt};
}

int ap_validate_queries(const ap_queries *q) {
    AP_REQUIRE(q != nullptr, "queries is NULL");
    AP_REQUIRE(q->nq >= 0, "queries.nq is negative");
    if (q->nq == 0) return AP_OK;
    AP_REQUIRE(q->dense && q->sp_indptr && q->sp_idx && q->sp_val && q->tx_indptr && q->tx_idx && q->tx_cnt,
               "queries has a NULL array");
    AP_REQUIRE(((uintptr_t)q->dense & 15) == 0, "queries.dense must be 16-byte aligned");
    return AP_OK;
}

extern "C" int ap_hybrid_scores(const ap_index *ix, const ap_queries *q, const int32_t *cand_ids, int32_t c,
                                const float *per_query_w, float *out4, void *stream) {
    AP_REQUIRE(ix && cand_ids && out4, "NULL argument");
    AP_TRY(ap_validate_queries(q));
    AP_REQUIRE(c >= 0, "c is negative");
    if (q->nq == 0 || c == 0) return AP_OK;
    AP_REQUIRE(((uintptr_t)out4 & 15) == 0, "out4 must be 16-byte aligned");
    const ApVecs A = query_view(q, ix->docs.dim);
    const float *w = per_query_w ? per_query_w : ix->w_dev;
    const int32_t ws = per_query_w ? 3 : 0;
    int32_t chunk = 256;
    // enough blocks to fill the chip even for few queries
    while (chunk > 16 && (int64_t)q->nq * ((c + chunk - 1) / chunk) < 2048) chunk >>= 1;
    dim3 grid((unsigned)q->nq, (unsigned)((c + chunk - 1) / chunk));
    AP_REQUIRE(grid.y <= 65535, "too many candidates per query");
    AP_DISPATCH_DENSE(ix->dtype, ix->docs.dim,
                      hipLaunchKernelGGL((k_hybrid_pairs<DT, NV, AP_F32>), grid, dim3(256), 0, (hipStream_t)stream, A,
                                         ix->docs, (const int32_t *)nullptr, cand_ids, c, chunk, w, ws, out4));
    AP_CHECK_HIP(hipGetLastError());
    return AP_OK;
}

extern "C" int ap_hybrid_scores_docs(const ap_index *ix, const int32_t *a_ids, int32_t na, const int32_t *cand_ids,
                                     int32_t c, const float w3[3], float *out4, void *stream) {
    AP_REQUIRE(ix && a_ids && cand_ids && out4 && w3, "NULL argument");
    AP_REQUIRE(na >= 0 && c >= 0, "negative count");
    if (na == 0 || c == 0) return AP_OK;
    AP_REQUIRE(((uintptr_t)out4 & 15) == 0, "out4 must be 16-byte aligned");
    hipStream_t st = (hipStream_t)stream;
    // weights travel through a small device buffer owned by this call
    float *wdev = nullptr;
    AP_TRY(ap_dev_alloc(&wdev, 4));
    hipError_t e = hipMemcpyAsync(wdev, w3, 3 * sizeof(float), hipMemcpyHostToDevice, st);
    if (e != hipSuccess) { (void)hipFree(wdev); ap_set_error("weight copy failed: %s", hipGetErrorString(e)); return AP_EHIP; }
    int32_t chunk = 256;
    while (chunk > 16 && (int64_t)na * ((c + chunk - 1) / chunk) < 2048) chunk >>= 1;
    dim3 grid((unsigned)na, (unsigned)((c + chunk - 1) / chunk));
    if (grid.y > 65535) { (void)hipFree(wdev); ap_set_error("too many candidates per row"); return AP_EINVAL; }
    AP_DISPATCH_DENSE(ix->dtype, ix->docs.dim,
                      hipLaunchKernelGGL((k_hybrid_pairs<DT, NV, DT>), grid, dim3(256), 0, st, ix->docs, ix->docs, a_ids,
                                         cand_ids, c, chunk, (const float *)wdev, 0, out4));
    e = hipGetLastError();
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    (void)hipFree(wdev);
    if (e != hipSuccess) { ap_set_error("ap_hybrid_scores_docs failed: %s", hipGetErrorString(e)); return AP_EHIP; }
    return AP_OK;
}

// ------------------------------------------------------------------ exhaustive scorer
// Ground truth for recall: fused scores of a block of queries against every
// document, then exact top-k by repeated arg-max under the total order.
// The document row sits in registers and is reused for QB queries staged in
// LDS, so the corpus is streamed nq/QB times instead of nq times.
// list: the queries to do (place s of the batch is query list[s]); NULL: query s.
#define AP_BF_QB 8
#define AP_BF_QCAP 64

template <int DT, int NV>
__global__ __launch_bounds__(256) void k_bf_scores(ApVecs Q, ApVecs D, const int32_t *__restrict__ list, int32_t q0, int32_t nqb,
                                                   const float *__restrict__ w, int32_t w_stride,
                                                   float *__restrict__ scores /* nqb x n */) {
    constexpr int EPC = ApDense<DT>::EPC;
    extern __shared__ __attribute__((aligned(16))) float smem[];
    float *qd = smem;                                                // QB x dim
    int32_t *qsi = reinterpret_cast<int32_t *>(qd + AP_BF_QB * Q.dim);  // QB x QCAP
    float *qsv = reinterpret_cast<float *>(qsi + AP_BF_QB * AP_BF_QCAP);
    int32_t *qti = reinterpret_cast<int32_t *>(qsv + AP_BF_QB * AP_BF_QCAP);
    float *qtv = reinterpret_cast<float *>(qti + AP_BF_QB * AP_BF_QCAP);
    __shared__ ApLists lists[AP_BF_QB];
    __shared__ float wq[AP_BF_QB][3];
    const int32_t qb = q0 + blockIdx.y * AP_BF_QB;
    const int32_t nq_here = (q0 + nqb - qb) < AP_BF_QB ? (q0 + nqb - qb) : AP_BF_QB;
    for (int x = ap_wave_id(); x < nq_here; x += 4) {   // a wave a row; dim is a multiple of 4
        const int64_t q = list ? list[qb + x] : qb + x;
        for (int i = (threadIdx.x & 63) * 4; i < Q.dim; i += 256)
            *reinterpret_cast<float4 *>(qd + x * Q.dim + i) = *reinterpret_cast<const float4 *>(static_cast<const float *>(Q.dense) + q * Q.dim + i);
    }
    for (int x = 0; x < nq_here; x++) {
        const int64_t q = list ? list[qb + x] : qb + x;   // uniform
        const ApLists a = ap_stage_lists(Q, q, qsi + x * AP_BF_QCAP, qsv + x * AP_BF_QCAP, qti + x * AP_BF_QCAP,
                                         qtv + x * AP_BF_QCAP, AP_BF_QCAP);
        if (threadIdx.x == 0) {
            lists[x] = a;
            wq[x][0] = w[q * w_stride + 0];
            wq[x][1] = w[q * w_stride + 1];
            wq[x][2] = w[q * w_stride + 2];
        }
    }
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int64_t wave = blockIdx.x * 4 + ap_wave_id();
    const int64_t nwaves = (int64_t)gridDim.x * 4;
    for (int64_t j = wave; j < D.n; j += nwaves) {
        float dr[NV * EPC];
        ap_load_aside<DT, NV, DT>(D.dense, j, D.dim, dr);
        const int64_t sb = D.sp_indptr[j], se = D.sp_indptr[j + 1], tb = D.tx_indptr[j], te = D.tx_indptr[j + 1];
        for (int x = 0; x < nq_here; x++) {
            float pd = 0.f;
#pragma unroll
            for (int i = 0; i < NV; i++) {
                const int col = (i * 64 + lane) * EPC;
                if (col < D.dim) {
#pragma unroll
                    for (int e = 0; e < EPC; e++) pd = fmaf(qd[x * Q.dim + col + e], dr[i * EPC + e], pd);
                }
            }
            const ApLists a = lists[x];
            const float ps = ap_sparse_partial(a.sp_idx, a.sp_val, a.sp_n, D.sp_idx, D.sp_val, sb, se, lane);
            const float pf = ap_sparse_partial(a.tx_idx, a.tx_val, a.tx_n, D.tx_idx, D.tx_val, tb, te, lane);
            const float sd = ap_wave_sum(pd), ss = ap_wave_sum(ps), sf = ap_wave_sum(pf);
            if (lane == 0) scores[(int64_t)(qb - q0 + x) * D.n + j] = ap_fuse(wq[x][0], wq[x][1], wq[x][2], sd, ss, sf);
        }
    }
}

// k rounds of block-wide arg-max: round r finds the best key that ranks after
// the winner of round r-1.
__global__ __launch_bounds__(256) void k_bf_topk(const float *__restrict__ scores, int64_t n, int32_t k, const int32_t *__restrict__ list, int32_t q0,
                                                 int32_t *__restrict__ out_ids, float *__restrict__ out_scores) {
    __shared__ uint64_t red[4];
    __shared__ uint64_t prev_s;
    const float *row = scores + (int64_t)blockIdx.x * n;
    const int64_t q = list ? list[q0 + blockIdx.x] : (int64_t)q0 + blockIdx.x;
    uint64_t prev = ~0ull;
    for (int32_t r = 0; r < k; r++) {
        uint64_t best = 0;
        for (int64_t j = threadIdx.x; j < n; j += blockDim.x) {
            const uint64_t key = ap_make_key(row[j], (int32_t)j, 1);
            if (key < prev && key > best) best = key;
        }
        for (int o = 32; o > 0; o >>= 1) {
            const uint64_t other = __shfl_xor(best, o, 64);
            best = other > best ? other : best;
        }
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = best;
        __syncthreads();
        if (threadIdx.x == 0) {
            uint64_t b = red[0];
            for (int i = 1; i < 4; i++) b = red[i] > b ? red[i] : b;
            prev_s = b;
            out_ids[q * k + r] = b ? ap_key_id(b) : -1;
            out_scores[q * k + r] = b ? ap_key_score(b) : -INFINITY;
        }
        __syncthreads();
        prev = prev_s;  // 0 when nothing is left: later rounds find nothing either
    }
}

// The exact top-k out of the table of upper bounds: one workgroup per query.  Every thread keeps the AP_BT_KEPT best bounds of its
// share of the row; k of the best of all of them are scored, and the least of their scores, T, is one that the k-th
// result reaches at least, so only documents whose bound is not below T have to be scored (some fifty for k = 10 on
// 100,000 documents).  Those are among the kept ones, unless all that a thread kept reach T: then the row is read once more.  Bound by
// reading the row and by the waits of the few scores that follow; eight waves a workgroup where there are many queries, so that four share
// a CU and 1,000 queries run at once.  A query with more than AP_BT_CAND candidates is left to
// the exhaustive scorer.  1,000 queries of 100,000 documents (768 f32 columns), k = 10: 74.9 ms with the exhaustive scorer,
// 0.96 ms with the table read twice by 1,024 threads that sort their best bounds (this kernel 0.249), 0.84 now (scalar registers of seven waves a SIMD: 0.88).
// A call lasts as long as its query with the most candidates, some thousands where the bounds tell little (lexical part alone, negative
// weights), and fewer waves a query take longer for those.  So a candidate costs one wait, for its record and its row, and not three (offsets,
// lists, row).  4,200 documents, 1,000 queries, lexical part alone, k = 10, 100, 256: 0.82, 1.43, 2.11 ms with 1,024 threads and three waits, 1.19, 1.85,
// 2.32 with 512 and three, 0.99, 1.58, 2.04 with 512 and one, 0.68, 1.15, 1.64 with 1,024 and one; 150,000 documents, weights 0.5, -0.3, -0.2, k = 100: 2.12, 2.50, 2.19, 1.84.
#define AP_BT_CAND 4096
// Queries up to which a workgroup has 1,024 threads, two of which fit a CU: with fewer queries a CU would have waves to spare.  With 512 threads
// instead, k = 100: 1 query of 150,000 documents 301 -> 347 us, 16 of 12,000 158 -> 190, 400 of 12,000 201 -> 229 (k = 10: 150 -> 151).
// More queries where k is larger than 64, for the sake of those with many candidates (k = 100, 1,000 queries of 4,200, 20,000 and 100,000 documents:
// 249, 346 and 979 us with 512 threads, 257, 348 and 962 with 1,024; 4,000 queries: 610, 1,123 and 3,510 us, 670, 1,163 and 3,530).
#define AP_BT_FEW(k) ((k) > 64 ? 1024 : 512)
#define AP_BT_KEPT 4
#define AP_BT_BINS 512
template <int DT, int NV, int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(DT == AP_BF16 && NV >= 3 ? 5 : 8, 8))) void k_bound_topk(ApVecs Q, ApVecs D, const uint2 *__restrict__ rec,
                                                     const uint4 *__restrict__ meta, int64_t q0, const float *__restrict__ w, int32_t w_stride,
                                                     const float *__restrict__ table, int64_t ld, int32_t k, int32_t *__restrict__ out_ids,
                                                     float *__restrict__ out_scores, int32_t *__restrict__ over /* [0] count, then queries */) {
    __shared__ uint64_t keys[AP_BT_CAND];   // candidates: their ids, then their keys
    __shared__ int32_t l_sp_idx[AP_BF_QCAP], l_tx_idx[AP_BF_QCAP];
    __shared__ float l_sp_val[AP_BF_QCAP], l_tx_val[AP_BF_QCAP];
    __shared__ uint32_t hist[AP_BT_BINS];
    __shared__ int32_t s_n;
    __shared__ uint32_t s_T, s_lo, s_hi, s_line;
    const int64_t q = q0 + blockIdx.x;
    const float *row = table + (int64_t)blockIdx.x * ld;
    const int lane = threadIdx.x & 63, wave = ap_wave_id();
    const ApLists a = ap_stage_lists(Q, q, l_sp_idx, l_sp_val, l_tx_idx, l_tx_val, AP_BF_QCAP);
    float qa[NV * ApDense<DT>::EPC];
    ap_load_aside<DT, NV, AP_F32>(Q.dense, q, D.dim, qa);
    const float wd = w[q * w_stride], ws = w[q * w_stride + 1], wf = w[q * w_stride + 2];
    // the documents keys[0 .. n), a wave each: a wave's lanes fetch the descriptors of its next 64 at once
    auto score = [&](int32_t n, auto &&put) {
        constexpr int NW = NT / 64;
        for (int32_t i0 = wave; i0 < n; i0 += NT) {
            const int32_t own = (int32_t)(uint32_t)keys[i0 + NW * lane < n ? i0 + NW * lane : i0];
            const uint4 m = meta[own];
            for (int32_t i = i0, j = 0; i < n && j < 64; i += NW, j++) {
                const int32_t v = __builtin_amdgcn_readlane(own, j);
                const uint2 *r = rec + (uint32_t)__builtin_amdgcn_readlane((int)m.x, j);
                const uint32_t len = (uint32_t)__builtin_amdgcn_readlane((int)m.y, j);
                const int32_t spn = (int32_t)(len & 0xffffu), txn = (int32_t)(len >> 16);
                uint2 xs[2], xt[1];
                uint4 raw[NV];
                int32_t si[2], ti[1];
                float sv[2], tv[1], ss, sf;
                ap_rec_load_raw<2, 1>(r, spn, txn, xs, xt);
                ap_dense_load_raw<DT, NV>(D, v, raw);
                ap_rec_decode<2, 1>(xs, xt, spn, txn, si, sv, ti, tv);
                ap_rec_reduce_lists<2, 1>(r, a, spn, txn, si, sv, ti, tv, ss, sf);
                const float sd = ap_dense_dot_raw<DT, NV>(D, qa, raw);
                if (lane == 0) put(i, v, ap_fuse(wd, ws, wf, sd, ss, sf));
            }
        }
    };
    const int64_t n4 = (D.n + 3) / 4;
    // bounds as codes that ascend with them, one that is no number above all; 0: none
    uint32_t best[AP_BT_KEPT];
    int32_t id[AP_BT_KEPT];
#pragma unroll
    for (int i = 0; i < AP_BT_KEPT; i++) { best[i] = 0u; id[i] = -1; }
    for (int64_t j = threadIdx.x; j < n4; j += NT) {
        const float4 x4 = reinterpret_cast<const float4 *>(row)[j];
        const float x[4] = {x4.x, x4.y, x4.z, x4.w};
#pragma unroll
        for (int e = 0; e < 4; e++) {
            uint32_t o = x[e] == x[e] ? ap_f2ord(x[e]) : 0xffffffffu;
            if (j * 4 + e >= D.n) o = 0u;
            if (o > best[AP_BT_KEPT - 1]) {
                int32_t v = (int32_t)(j * 4 + e);
#pragma unroll
                for (int i = 0; i < AP_BT_KEPT; i++) {   // into its place, what it pushes out one further
                    const bool up = o > best[i];
                    const uint32_t ob = best[i];
                    const int32_t oi = id[i];
                    best[i] = up ? o : ob; id[i] = up ? v : oi;
                    o = up ? ob : o; v = up ? oi : v;
                }
            }
        }
    }
    // k of the best: everything above the bin that the k-th lies in, and as many of the bin as are missing
    for (int32_t i = threadIdx.x; i < AP_BT_BINS; i += NT) hist[i] = 0u;
    if (threadIdx.x == 0) { s_n = 0; s_T = 0xffffffffu; s_lo = 0xffffffffu; s_hi = 0u; s_line = 0u; }
    __syncthreads();
    {
        uint32_t lo = best[0] ? best[0] : 0xffffffffu, hi = best[0];   // the k best of all are best of their shares or above the worst of those
        for (int o = 32; o > 0; o >>= 1) { lo = min(lo, (uint32_t)__shfl_xor((int)lo, o, 64)); hi = max(hi, (uint32_t)__shfl_xor((int)hi, o, 64)); }
        if (lane == 0) { atomicMin(&s_lo, lo); atomicMax(&s_hi, hi); }
    }
    __syncthreads();
    const uint32_t lo = ap_uniform_u32(s_lo), hi = ap_uniform_u32(s_hi);
    int sh = 0;
    while (lo < hi && ((hi - lo) >> sh) >= AP_BT_BINS) sh++;
#pragma unroll
    for (int i = 0; i < AP_BT_KEPT; i++)
        if (best[i] && best[i] >= lo) atomicAdd(&hist[(best[i] - lo) >> sh], 1u);
    __syncthreads();
    if (wave == 0) {   // lane l: bins 8 (63 - l) .. + 7, so that the prefix sum runs from the top
        uint32_t bin[8], n = 0;
#pragma unroll
        for (int i = 0; i < 8; i++) { bin[i] = hist[8 * (63 - lane) + 7 - i]; n += bin[i]; }
        uint32_t upto = n;
        for (int o = 1; o < 64; o <<= 1) { const uint32_t up = (uint32_t)__shfl_up((int)upto, o, 64); if (lane >= o) upto += up; }
        const uint64_t m = __ballot(upto >= (uint32_t)k);
        if (m && lane == (int)__ffsll((unsigned long long)m) - 1) {
            uint32_t above = upto - n, b = 8u * (64 - lane);
#pragma unroll
            for (int i = 0; i < 8; i++) { b -= above < (uint32_t)k ? 1u : 0u; above += bin[i]; }
            s_line = b;
        }
    }
    __syncthreads();
    const uint32_t line = ap_uniform_u32(s_line);
    auto bin_of = [&](uint32_t o) { return o && o >= lo ? (int32_t)((o - lo) >> sh) : -1; };
#pragma unroll
    for (int i = 0; i < AP_BT_KEPT; i++)
        if (bin_of(best[i]) > (int32_t)line) keys[atomicAdd(&s_n, 1)] = (uint64_t)(uint32_t)id[i];   // fewer than k of them
    __syncthreads();
#pragma unroll
    for (int i = 0; i < AP_BT_KEPT; i++)
        if (bin_of(best[i]) == (int32_t)line) { const int32_t at = atomicAdd(&s_n, 1); if (at < k) keys[at] = (uint64_t)(uint32_t)id[i]; }
    __syncthreads();
    const int32_t first = min(ap_uniform_i32(s_n), k);
    score(first, [&](int32_t, int32_t, float s) { atomicMin(&s_T, ap_f2ord(s)); });
    __syncthreads();
    const float T = first == k ? ap_ord2f(s_T) : -INFINITY;
    const bool more = !(ap_ord2f(best[AP_BT_KEPT - 1]) < T) && best[AP_BT_KEPT - 1] != 0u;
    if (threadIdx.x == 0) s_n = 0;
    const bool again = __syncthreads_or(more) != 0;   // uniform
    if (!again) {
#pragma unroll
        for (int i = 0; i < AP_BT_KEPT; i++)
            if (best[i] && !(ap_ord2f(best[i]) < T)) keys[atomicAdd(&s_n, 1)] = (uint64_t)(uint32_t)id[i];   // 4 * NT at most, which keys[] holds
    } else {
        for (int64_t j = threadIdx.x; j < n4; j += NT) {
            const float4 x4 = reinterpret_cast<const float4 *>(row)[j];
            const float x[4] = {x4.x, x4.y, x4.z, x4.w};
#pragma unroll
            for (int e = 0; e < 4; e++)
                if (j * 4 + e < D.n && !(x[e] < T)) {
                    const int32_t pos = atomicAdd(&s_n, 1);
                    if (pos < AP_BT_CAND) keys[pos] = (uint64_t)(uint32_t)(j * 4 + e);
                }
        }
    }
    __syncthreads();
    const int32_t c = ap_uniform_i32(s_n);
    if (c > AP_BT_CAND || c < k) {   // uniform (fewer than k: scores that compare with nothing)
        if (threadIdx.x == 0) over[1 + atomicAdd(over, 1)] = (int32_t)q;
        return;
    }
    score(c, [&](int32_t i, int32_t v, float s) { keys[i] = ap_make_key(s, v, 1u); });
    int32_t n2 = 64;
    while (n2 < c) n2 <<= 1;
    for (int32_t i = c + (int32_t)threadIdx.x; i < n2; i += NT) keys[i] = 0ull;
    ap_bitonic_desc(keys, n2);
    for (int32_t i = threadIdx.x; i < k; i += NT) {
        out_ids[q * k + i] = ap_key_id(keys[i]);
        out_scores[q * k + i] = ap_key_score(keys[i]);
    }
}

// Every document scored, for the `count` queries of the list (device), or the first `count` ones.
static int bf_exhaustive(const ap_index *ix, const ApVecs &Q, const float *w, int32_t ws, const int32_t *list, int32_t count, int32_t k, int32_t *out_ids,
                         float *out_scores, hipStream_t st) {
    const int64_t n = ix->docs.n;
    // queries are processed in slabs so that the score scratch stays <= 2 GiB
    int64_t slab = (int64_t)(1ull << 29) / n;
    slab = slab / AP_BF_QB * AP_BF_QB;
    if (slab < AP_BF_QB) slab = AP_BF_QB;
    if (slab > count) slab = (count + AP_BF_QB - 1) / AP_BF_QB * AP_BF_QB;
    float *scratch = nullptr;
    AP_TRY(ap_bound_make_room(ix, st, &scratch, (size_t)slab * (size_t)n));
    const size_t smem = (size_t)AP_BF_QB * ((size_t)ix->docs.dim + 4 * AP_BF_QCAP) * 4;
    int rc = AP_OK;
    hipError_t e = hipSuccess;
    for (int32_t q0 = 0; q0 < count && e == hipSuccess; q0 += (int32_t)slab) {
        const int32_t nqb = (count - q0) < slab ? (count - q0) : (int32_t)slab;
        int64_t xb = (n + 3) / 4;
        if (xb > 256) xb = 256;
        dim3 grid((unsigned)xb, (unsigned)((nqb + AP_BF_QB - 1) / AP_BF_QB));
        AP_DISPATCH_DENSE(ix->dtype, ix->docs.dim, {
            e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_bf_scores<DT, NV>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
            if (e == hipSuccess)
                hipLaunchKernelGGL((k_bf_scores<DT, NV>), grid, dim3(256), smem, st, Q, ix->docs, list, q0, nqb, w, ws, scratch);
        });
        if (e == hipSuccess) e = hipGetLastError();
        if (e != hipSuccess) break;
        hipLaunchKernelGGL(k_bf_topk, dim3((unsigned)nqb), dim3(256), 0, st, scratch, n, k, list, q0, out_ids, out_scores);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    (void)hipFree(scratch);
    if (e != hipSuccess) { ap_set_error("ap_bruteforce_topk failed: %s", hipGetErrorString(e)); rc = AP_EHIP; }
    return rc;
}

extern "C" int ap_bruteforce_topk(const ap_index *ix, const ap_queries *q, const float *per_query_w, int32_t k,
                                  int32_t *out_ids, float *out_scores, void *stream) {
    AP_REQUIRE(ix && out_ids && out_scores, "NULL argument");
    AP_TRY(ap_validate_queries(q));
    AP_REQUIRE(k >= 1, "k must be positive");
    if (q->nq == 0) return AP_OK;
    hipStream_t st = (hipStream_t)stream;
    const ApVecs Q = query_view(q, ix->docs.dim);
    const float *w = per_query_w ? per_query_w : ix->w_dev;
    const int32_t ws = per_query_w ? 3 : 0;
    // Out of the table of bounds where that leaves most documents unscored: k well below the AP_BT_KEPT * NT documents (2,048 or 4,096) that
    // the threshold comes from, and a corpus as large at least (below, the exhaustive scorer has little to do).  The histogram of the kept
    // bounds begins at the worst of the threads' best ones, so it holds as many as there are threads at least: with 4,096 documents every
    // one of 1,024 threads has four.
    constexpr int32_t most_k = 256, least_n = 4096;
    static_assert(most_k <= 512 && least_n / 4 >= 1024, "k of the kept bounds are in the histogram");
    ApBound b;
    const size_t held = ap_bound_held(ix, st);
    if (k <= most_k && ix->docs.n >= least_n) AP_TRY(ap_bound_reserve(ix, q->nq, 256, AP_BOUND_WS_BYTES, 1, st, &b));
    if (!b.table) return bf_exhaustive(ix, Q, w, ws, nullptr, q->nq, k, out_ids, out_scores, st);
    int32_t *over = nullptr;
    AP_TRY(ap_dev_alloc(&over, (size_t)q->nq + 1));
    int rc = ap_fill_u32(over, 1, 0u, st);
    for (int32_t q0 = 0; q0 < q->nq && rc == AP_OK; q0 += b.slab) {
        const int32_t nqb = std::min(b.slab, q->nq - q0);
        rc = ap_bound_fill(ix, b, Q, w, ws, q0, nqb, nullptr, 0, st);
        if (rc != AP_OK) break;
        if (nqb <= AP_BT_FEW(k))
            AP_DISPATCH_DENSE(ix->dtype, ix->docs.dim, hipLaunchKernelGGL((k_bound_topk<DT, NV, 1024>), dim3((unsigned)nqb), dim3(1024), 0, st, Q, ix->docs, ix->rec, ix->meta,
                                                                          (int64_t)q0, w, ws, b.table, b.ld, k, out_ids, out_scores, over));
        else
            AP_DISPATCH_DENSE(ix->dtype, ix->docs.dim, hipLaunchKernelGGL((k_bound_topk<DT, NV, 512>), dim3((unsigned)nqb), dim3(512), 0, st, Q, ix->docs, ix->rec, ix->meta,
                                                                          (int64_t)q0, w, ws, b.table, b.ld, k, out_ids, out_scores, over));
        if (hipGetLastError() != hipSuccess) { ap_set_error("ap_bruteforce_topk failed to launch"); rc = AP_EHIP; }
    }
    b.finish();   // the host waits below: searches of this index on other streams need not
    int32_t n_over = 0;
    hipError_t e = hipSuccess;
    if (rc == AP_OK) {
        e = hipMemcpyAsync(&n_over, over, sizeof(n_over), hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
    }
    // a workspace that this call made larger than its own scratch ever was does not stay
    if (const size_t now = ap_bound_held(ix, st); now > held && now > AP_BOUND_KEEP_BYTES) ap_bound_give_back(ix, st);
    if (rc == AP_OK && e != hipSuccess) { ap_set_error("ap_bruteforce_topk failed: %s", hipGetErrorString(e)); rc = AP_EHIP; }
    // the queries the bounds left undecided, in whatever order they were noted, as one batch (it waits for the stream)
    if (rc == AP_OK && n_over > 0) rc = bf_exhaustive(ix, Q, w, ws, over + 1, n_over, k, out_ids, out_scores, st);
    (void)hipFree(over);
    return rc;
}
