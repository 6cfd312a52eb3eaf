// What the searches share: the visited set, the pool's keys, and the scoring of a list of candidates against one query.
#pragma once
#include "ap_common.hpp"

// The visited set of a query: one bit per document, in LDS when the corpus is small enough for that not to cost a
// workgroup its place on the CU (ap_search_launch decides), else in a per-call global workspace.  Marks document v and
// tells whether it had been marked before.  Only the workgroup that searches the query ever touches its set, so the
// global atomic needs workgroup scope only.
#ifndef AP_VIS_SCOPE
#define AP_VIS_SCOPE __HIP_MEMORY_SCOPE_WORKGROUP
#endif
struct ApVisited {
    uint32_t *g;             // global bitset of this query
    AP_LDS uint32_t *l;      // LDS bitset, or null
    __device__ __forceinline__ bool test_and_set(int32_t v) const {
        const uint32_t bit = 1u << (v & 31);
        uint32_t old;
        if (l) old = __hip_atomic_fetch_or(l + (v >> 5), bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);   // uniform branch
        else old = __hip_atomic_fetch_or(g + (v >> 5), bit, __ATOMIC_RELAXED, AP_VIS_SCOPE);
        return (old & bit) != 0u;
    }
};

// Pool keys.  Plain search: ap_make_key (30-bit id, bit 0 = "not yet expanded").
// Keyword search: 29-bit id, bit 0 as before, bit 1 = "satisfies the keyword
// constraint".  Ids are unique within a pool, so the flag bits never decide an order.
#define AP_KW_MAX_TERMS 16
template <bool KW> __device__ __forceinline__ uint64_t ap_pool_key(float s, int32_t id, uint32_t flags) {
    if (KW) return ((uint64_t)ap_f2ord(s) << 32) | (uint64_t)(((0x1fffffffu - (uint32_t)id) << 2) | flags);
    return ap_make_key(s, id, flags);
}
template <bool KW> __device__ __forceinline__ int32_t ap_pool_id(uint64_t k) {
    if (KW) return (int32_t)(0x1fffffffu - (((uint32_t)k) >> 2));
    return ap_key_id(k);
}

// Scores the c candidates of this iteration; wave w of the workgroup's NW takes candidates w, w+NW, ...
// The sparse and lexical parts (the short segments) are evaluated first.  When
// the pool is full and even the largest dense part the norms allow,
// |w_d| |q_d| |d_d|, could not lift the candidate past the pool's last entry,
// the dense row is not read at all: the candidate could not have entered the
// pool, so the result of the search is unchanged (it still counts as visited).
// TAB: the query's lists are look-up tables in LDS (the usual case); otherwise
// they are searched where they lie in global memory.
// Returns the number of candidates whose dense row was skipped (wave-uniform).
// Sizes of the query's two look-up tables (at most a quarter full).  Ordinary queries: 256 + 128 slots (lists up to
// 64 / 32 entries).  Queries that are documents (insertion): 1024 + 512 slots (lists up to 256 / 128 entries).  Both are
// bucketed: two slots a bucket, a hash multiplier per table under which no bucket needs a third.
template <bool BIG> struct ApQTab {
    static constexpr int SPB = BIG ? 10 : 8;
    static constexpr int TXB = BIG ? 9 : 7;
    static constexpr int SLOTS = (1 << SPB) + (1 << TXB);
};

// KW: each candidate's lexical terms are also compared with the query's required
// terms (s_kw[0..n_kw)); the key of a candidate that satisfies the constraint
// carries the "satisfies" flag, and its dense row may only be skipped when the
// bound also rules out the secondary pool (full, and its last score above the bound).
// G: candidates a wave keeps on their way at once.  Their records are loaded together, then reduced one by one;
// then the dense rows of those that still need one are loaded together and multiplied one by one.  G = 1 is the
// plain order (record, sums, dense row); larger G trades registers for memory requests in flight, which pays where
// a large pool leaves a CU with few waves.  pre: the candidates' dense rows are requested along with their records (they
// got past their bounds, so nearly all of them need theirs).  The order of the additions inside a candidate does not depend on G.
// W0: the first of the NW waves that score (the waves before it do not take part).
template <int DT, int NV, bool TAB, bool KW, bool BIG, int NW, int G, int W0 = 0>
__device__ __forceinline__ int32_t ap_score_candidates(const ApVecs &D, const uint2 *rec, const float *qa, const uint64_t *qtab,
                                                       const ApLists &a, float wd, float ws, float wf, float qnorm, bool pool_full,
                                                       float worst_score, const uint4 *s_meta, int32_t c,
                                                       uint64_t *newk, const int32_t *s_kw, int32_t n_kw, bool kw_all,
                                                       bool second_full, float second_worst, uint32_t msp, uint32_t mtx, bool pre) {
    const int lane = threadIdx.x & 63, wave = ap_wave_id();
    int32_t skipped = 0;
    for (int32_t i0 = wave - W0; i0 < c; i0 += NW * G) {
        uint2 xs[G][2], xt[G][1];
        uint4 raw[G][NV];
        const uint2 *r[G];
        int32_t spn[G], txn[G], v[G];
        float dn[G];
#pragma unroll
        for (int gi = 0; gi < G; gi++) {
            const int32_t i = i0 + NW * gi;
            if (i < c) {
                const uint4 m = s_meta[i];
                // the descriptor is the same in every lane: keep the record's address in scalar registers
                r[gi] = rec + ap_uniform_u32(m.x);
                spn[gi] = __builtin_amdgcn_readfirstlane((int32_t)(m.y & 0xffffu));
                txn[gi] = __builtin_amdgcn_readfirstlane((int32_t)(m.y >> 16));
                dn[gi] = __uint_as_float(ap_uniform_u32(m.z));
                v[gi] = (int32_t)ap_uniform_u32(m.w);
                ap_rec_load_raw<2, 1>(r[gi], spn[gi], txn[gi], xs[gi], xt[gi]);
                if (pre) ap_dense_load_raw<DT, NV>(D, v[gi], raw[gi]);
            }
        }
        float ss[G], sf[G];
        uint32_t flags[G];
        bool need[G];      // uniform: the candidate's dense row has to be read
#pragma unroll
        for (int gi = 0; gi < G; gi++) {
            const int32_t i = i0 + NW * gi;
            need[gi] = false;
            if (i >= c) continue;
            int32_t si[2], ti[1];
            float sv[2], tv[1];
            ap_rec_decode<2, 1>(xs[gi], xt[gi], spn[gi], txn[gi], si, sv, ti, tv);
            if (TAB)   // bucketed tables, one read per look-up
                ap_rec_reduce_bucket<2, 1, ApQTab<BIG>::SPB, ApQTab<BIG>::TXB>(r[gi], (const AP_LDS uint64_t *)qtab,
                                                                               (const AP_LDS uint64_t *)(qtab + (1 << ApQTab<BIG>::SPB)),
                                                                               msp, mtx, spn[gi], txn[gi], si, sv, ti, tv, ss[gi], sf[gi]);
            else
                ap_rec_reduce_lists<2, 1>(r[gi], a, spn[gi], txn[gi], si, sv, ti, tv, ss[gi], sf[gi]);
            // upper bound of the fused score, with slack far above fp32 rounding
            const float dmax = fabsf(wd) * qnorm * dn[gi] * 1.0001f;
            const float part = fmaf(wf, sf[gi], ws * ss[gi]);
            const float ub = part + dmax + 1e-5f * (fabsf(ws * ss[gi]) + fabsf(wf * sf[gi]) + dmax);
            flags[gi] = 1u;
            if (KW && n_kw > 0) {
                uint32_t hit = 0;   // bit j: required term j occurs in the candidate's text
                for (int32_t e0 = 0; e0 < txn[gi]; e0 += 64) {
                    int32_t term = ti[0];
                    if (e0 > 0) term = e0 + lane < txn[gi] ? (int32_t)r[gi][spn[gi] + e0 + lane].x : -1;
                    for (int32_t j = 0; j < n_kw; j++) hit |= __ballot(term == s_kw[j]) != 0ull ? 1u << j : 0u;
                }
                const bool sat = kw_all ? hit == (1u << n_kw) - 1u : hit != 0u;
                flags[gi] |= sat ? 2u : 0u;
            }
            if (pool_full && ub < worst_score && (!(flags[gi] & 2u) || (second_full && ub < second_worst))) {
                if (lane == 0) newk[i] = (uint64_t)(uint32_t)(i + 1);   // ranks after every real key (score bits 0), distinct per candidate
                skipped++;
            } else {
                need[gi] = true;
            }
        }
#pragma unroll
        for (int gi = 0; gi < G; gi++)
            if (need[gi] && !pre) ap_dense_load_raw<DT, NV>(D, v[gi], raw[gi]);
#pragma unroll
        for (int gi = 0; gi < G; gi++) {
            if (need[gi]) {
                const float sd = ap_dense_dot_raw<DT, NV>(D, qa, raw[gi]);
                if (lane == 0) newk[i0 + NW * gi] = ap_pool_key<KW>(ap_fuse(wd, ws, wf, sd, ss[gi], sf[gi]), v[gi], flags[gi]);
            }
        }
    }
    return skipped;
}
