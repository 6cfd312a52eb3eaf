// The two lists of every document in a third of their bytes, for the rounds of a construction: what k_refine reads to tell
// which candidates can enter a list before it reads anything of them in full.
#include <algorithm>
#include "ap_common.hpp"
#include "ap_packed.hpp"

// The slot of every term: the terms of the top bins of document frequency that fit AP_PK_DIRECT slots together get one each, the
// others share what is left, either vocabulary a part of its own (lexical weights are larger, and a false meeting of two of
// them weighs more, so that part is the larger one).  100,000 documents of 120 and 43 entries: the bound then lies 0.4 above a
// score of 25 on average; with one slot in two shared it would be 0.7.
__global__ __launch_bounds__(1024) void k_pk_slots(const int32_t *__restrict__ df_sp, int32_t nsp, const int32_t *__restrict__ df_tx, int32_t ntx,
                                                   const int32_t *__restrict__ hist, uint16_t *__restrict__ slot, uint32_t *__restrict__ used) {
    __shared__ int32_t s_low;
    if (threadIdx.x == 0) {
        int32_t low = 256, sum = 0;
        while (low > 0 && sum + hist[low - 1] <= AP_PK_DIRECT) sum += hist[--low];
        s_low = low;
    }
    __syncthreads();
    const int64_t t = blockIdx.x * (int64_t)1024 + threadIdx.x, all = (int64_t)nsp + ntx;
    if (t >= all) return;
    const int32_t df = t < nsp ? df_sp[t] : df_tx[t - nsp];
    const uint32_t h = (uint32_t)(((uint64_t)((uint32_t)t * 2654435761u) * (uint64_t)(t < nsp ? AP_PK_SP : AP_PK_TX)) >> 32);
    slot[t] = df > 0 && ap_df_bin(df) >= s_low ? (uint16_t)(atomicAdd(used, 1u) & (AP_PK_DIRECT - 1))
                                               : (uint16_t)(AP_PK_DIRECT + (t < nsp ? h : AP_PK_SP + h));
}

// One wave per document.  A list's weights are rounded up to 8 bits of its largest one; a list with a value that is negative or no
// number gets an infinite scale, with which every bound of it is infinite or no number.  Bound by the reads of the lists
// (8 bytes an entry) and the scattered reads of the slots: 0.2 ms for 29 million entries.
__global__ __launch_bounds__(256) void k_pk_rows(ApVecs D, int32_t nsp, const uint16_t *__restrict__ slot, const float *__restrict__ dnorm, uint32_t *__restrict__ rec,
                                                 uint2 *__restrict__ at) {
    const int lane = threadIdx.x & 63;
    const int64_t off0 = D.sp_indptr[0] + D.tx_indptr[0];
    for (int64_t v = blockIdx.x * (int64_t)4 + ap_wave_id(); v < D.n; v += (int64_t)gridDim.x * 4) {
        const int64_t b[2] = {D.sp_indptr[v], D.tx_indptr[v]};
        const int32_t n[2] = {(int32_t)(D.sp_indptr[v + 1] - b[0]), (int32_t)(D.tx_indptr[v + 1] - b[1])};
        const int64_t line = ap_pk_line(b[0] + b[1] - off0, v);
        uint32_t *r = rec + line * (AP_PK_LINE / 4);
        float scale[2];
        int32_t u0 = 1;
#pragma unroll
        for (int part = 0; part < 2; part++) {
            const int32_t *idx = part ? D.tx_idx : D.sp_idx;
            const float *val = part ? D.tx_val : D.sp_val;
            float most = 0.f;
            bool odd = false;
            for (int32_t e = lane; e < n[part]; e += 64) {
                const float x = val[b[part] + e];
                odd = odd || !(x >= 0.f && x - x == 0.f);
                most = fmaxf(most, x);
            }
            for (int o = 32; o > 0; o >>= 1) most = fmaxf(most, __shfl_xor(most, o, 64));
            odd = __ballot(odd) != 0ull;
            const float sc = fmaxf(most * (1.00001f / 254.f), 1e-18f), inv = 1.000002f / sc;
            scale[part] = odd ? INFINITY : sc;
            const int32_t units = (n[part] + 3) / 4;
            for (int32_t u = lane; u < units; u += 64) {
                uint32_t w = 0, sl[4];
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    const int32_t e = 4 * u + i;
                    sl[i] = 0;
                    if (e < n[part]) {
                        const float x = val[b[part] + e];
                        w |= (odd || x == 0.f ? 0u : min((uint32_t)(x * inv) + 1u, 255u)) << (8 * i);
                        sl[i] = slot[(part ? nsp : 0) + idx[b[part] + e]];
                    }
                }
                uint32_t *d = r + (u0 + u) * 3;
                d[0] = w; d[1] = sl[0] | (sl[1] << 16); d[2] = sl[2] | (sl[3] << 16);
            }
            u0 += units;
        }
        if (lane == 0) {
            r[0] = __float_as_uint(scale[0]); r[1] = __float_as_uint(scale[1]); r[2] = __float_as_uint(dnorm[v]);
            at[v] = make_uint2((uint32_t)line, (uint32_t)((n[0] + 3) / 4) | ((uint32_t)((n[1] + 3) / 4) << 16));
        }
    }
}

// The packed lists of the documents of ix (or of a view of it).  out->mem stays NULL for a few hundred documents, whose
// rounds take no longer than the packing (constructions of 130, 500 and 1,000 documents of 128 columns, without and with: 1.01 and
// 1.06, 1.22 and 1.24, 1.99 and 1.91 ms), where there is no room for them, where the
// vocabularies are too large for a table of slots, or where a weight of the construction is negative (a bound from above
// of a list's part would then be one from below): the rounds read the lists themselves then.
int ap_pack_lists(const ap_index *ix, hipStream_t st, ApPacked *out) {
    *out = ApPacked();
    const ap_corpus &c = ix->corpus;
    const float *w = ix->params.build_w;
    const int64_t all = (int64_t)c.sp_vocab + c.tx_vocab, n = ix->docs.n;
    if (n < AP_PK_LEAST || all > AP_PK_VOCAB || !(w[1] >= 0.f) || !(w[2] >= 0.f)) return AP_OK;
    int64_t nnz = ix->sp_nnz + ix->tx_nnz;
    if (ix->docs.sp_indptr != c.sp_indptr) {   // a view that ends with the corpus (the new documents of an insertion)
        int64_t first[2] = {0, 0};
        AP_CHECK_HIP(hipMemcpyAsync(&first[0], ix->docs.sp_indptr, 8, hipMemcpyDeviceToHost, st));
        AP_CHECK_HIP(hipMemcpyAsync(&first[1], ix->docs.tx_indptr, 8, hipMemcpyDeviceToHost, st));
        AP_CHECK_HIP(hipStreamSynchronize(st));
        nnz -= first[0] + first[1];
    }
    if (nnz * ix->params.knn_k < AP_PK_WORK) return AP_OK;
    const size_t rec_bytes = (size_t)ap_pk_line(nnz, n) * AP_PK_LINE;
    auto up = [](size_t x) { return (x + 255) / 256 * 256; };
    const bool count = ix->bd_df == nullptr;   // the columns of the bounds are not there: their document frequencies are not either
    const size_t n_clear = 256 + 1 + (count ? (size_t)c.sp_vocab : 0);
    const size_t o_at = up(rec_bytes), o_slot = o_at + up((size_t)n * 8), o_clear = o_slot + up((size_t)all * 2), bytes = o_clear + n_clear * 4;
    size_t free_b = 0, total_b = 0;   // a large one takes a quarter of what is free at most; asking costs a small construction more than it is worth
    if (bytes > (size_t)64 << 20 && (hipMemGetInfo(&free_b, &total_b) != hipSuccess || bytes > free_b / 4)) { (void)hipGetLastError(); return AP_OK; }
    void *mem = nullptr;
    if (hipMalloc(&mem, bytes) != hipSuccess) { (void)hipGetLastError(); return AP_OK; }
    out->mem = mem;
    out->bytes = bytes;
    char *m = static_cast<char *>(mem);
    uint32_t *rec = reinterpret_cast<uint32_t *>(m);
    uint2 *at = reinterpret_cast<uint2 *>(m + o_at);
    uint16_t *slot = reinterpret_cast<uint16_t *>(m + o_slot);
    int32_t *hist = reinterpret_cast<int32_t *>(m + o_clear);
    uint32_t *used = reinterpret_cast<uint32_t *>(hist + 256);
    int32_t *df = count ? hist + 257 : ix->bd_df;
    AP_TRY(ap_fill_u32(hist, n_clear, 0u, st));
    if (count) AP_TRY(ap_count_terms(c.sp_idx, nullptr, ix->sp_nnz, df, nullptr, st));
    AP_TRY(ap_df_histogram(df, c.sp_vocab, ix->df, c.tx_vocab, hist, st));
    hipLaunchKernelGGL(k_pk_slots, dim3((unsigned)((all + 1023) / 1024)), dim3(1024), 0, st, df, c.sp_vocab, ix->df, c.tx_vocab, hist, slot, used);
    hipLaunchKernelGGL(k_pk_rows, dim3((unsigned)std::min<int64_t>((n + 3) / 4, 8192)), dim3(256), 0, st, ix->docs, c.sp_vocab, slot, ix->dense_norm, rec, at);
    AP_CHECK_HIP(hipGetLastError());
    out->rec = rec;
    out->at = at;
    return AP_OK;
}
