// S7-S9: batched best-first search (Algorithm 2 without its entity branches),
// one workgroup per query.  The KW instantiation adds the keyword branches of
// Section 4.2.2: keyword edges of parents that satisfy the query's keyword
// constraint, a secondary pool of satisfying documents the pool did not keep,
// and the final filter.
//
// Per query, in LDS: the candidate pool (one sorted array of 64-bit keys that
// plays both `cand` and `topk` of Algorithm 2; bit 0 of a key = "not yet
// expanded"), the descriptors and keys of the neighbours scored in this
// iteration, and the query's two sparse lists as look-up tables.  The query's
// dense slice stays in registers.  The visited set is an exact bitset (one bit
// per document): in LDS for small pools on small corpora, else in a global
// workspace of bounded size (large batches run in slabs of queries).
#include <math.h>
#include <stdlib.h>
#include <string.h>
#include <algorithm>
#include <mutex>
#include "ap_score.hpp"

int ap_validate_queries(const ap_queries *q);

struct ApSearchArgs {
    ApVecs D, Q;
    const int32_t *graph;
    const int32_t *entry;
    const float *w;     // per query (stride 3) or the index default (stride 0)
    int32_t w_stride;
    int32_t R, E, k, L, max_iters, width, cmax;
    int32_t icap;       // large pools: > 0: an iteration's neighbours are listed by their ids (this many at most) and scored cmax at a time; 0: all at once
    int32_t vis_lds;    // the visited sets live in LDS (words words after the kernel's other arrays), not in `visited`
    int32_t nxtw;       // words of the scratch that parks positions when more keys enter at once than the workgroup has threads (else 0)
    int32_t q0;         // the launch covers queries q0 .. q0 + gridDim.x (a slab of the batch)
    int32_t no_tables;  // debug: search the query's lists where they lie even when they fit the LDS tables
    uint32_t *visited;  // one bitset per query of the slab
    size_t words;       // visited words per query
    int32_t *out_ids;
    float *out_scores;
    int32_t *counts;    // nq x 3: candidates scored, iterations, candidates whose dense row was skipped (NULL: not wanted)
    const uint2 *rec;   // packed (term, weight) records of the documents' two sparse parts
    const uint4 *meta;  // per document: first entry, counts, |d_dense|
    const uint32_t *deleted;   // one bit per document, NULL = nothing is mark-deleted: left out of the answers only
    float *bound;              // upper bounds of the scores, a row of bound_ld documents per query of the slab; NULL: none
    const float4 *bound_floor; // per query of the slab: neighbours with a bound below it wait (see k_search); two lower ones; NULL: none wait
    uint64_t *marks;           // with bound_floor: per query of the slab a word for 32 documents, visited | bound reaches the floor << 32
    int64_t bound_ld;
    const int32_t *bound_col;  // keyword searches with bounds: head column of every lexical term (-1: the entry's count tells), bitmaps of the columns
    const uint32_t *bound_bits;
    int32_t tx_vocab;
    // keyword-constrained search only
    const int32_t *kw_edges;   // n x KR keyword edges, kw_count[u] of them valid
    const int32_t *kw_count;
    const int32_t *kw_terms;   // nq x kw_stride required terms, -1 = unused slot
    int32_t KR, kw_stride, kw_all, kw_use_edges;
};

// Number of entries of the descending array keys[0..n) that rank before `key`.
__device__ __forceinline__ int32_t ap_rank_in(const uint64_t *keys, int32_t n, uint64_t key) {
    int32_t lo = 0, hi = n;
    while (lo < hi) {
        const int32_t mid = (lo + hi) >> 1;
        if (keys[mid] > key) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// Candidates a wave keeps in flight (ap_score_candidates' G), by workgroup size, as measured on a million-document
// shape: a second candidate costs some 35 registers, which the four- and eight-wave workgroups that share a CU cannot
// spare (one is fastest there: other waves hide the latency); sixteen waves alone on a CU gain 6 % from a second one
// and nothing from a third.
#ifndef AP_SEARCH_G_256
#define AP_SEARCH_G_256 1
#endif
#ifndef AP_SEARCH_G_512
#define AP_SEARCH_G_512 1
#endif
#ifndef AP_SEARCH_G_1024
#define AP_SEARCH_G_1024 2
#endif
#ifndef AP_RANK_LANES
#define AP_RANK_LANES 16        // lanes that rank one entering key of a large pool (16, 32 or 64)
#endif
#define AP_RANK_SORT 128        // entering keys of a large pool beyond which they are sorted instead of ranked one against the other
// Two waves a query with keywords: at six waves a SIMD they spill less than at seven (768 f32 columns 6 registers instead of 13, 1,024 f32 17 and 29,
// 1,024 bf16 5 and 11); 2,500 queries of 768 f32 columns 11.05 -> 10.62 ms.
#define AP_SEARCH_WAVES_KW2 6
#define AP_SEARCH_LISTED 256    // listed neighbours that are scored at a time
#ifndef AP_SEARCH_WAVES_512
#define AP_SEARCH_WAVES_512 6
#endif
#define AP_SEARCH_G_LIST 2
template <int NT, bool LIST> struct ApSearchG { static constexpr int G = LIST ? AP_SEARCH_G_LIST : NT == 1024 ? AP_SEARCH_G_1024 : NT == 512 ? AP_SEARCH_G_512 : AP_SEARCH_G_256; };

// Profiling aid of debug builds (-DAP_SEARCH_PROFILE): thread 0 of every workgroup adds the time it spent in each
// phase of the loop (100 MHz ticks) to a device array that ap_debug_search_profile reads and clears.
#ifdef AP_SEARCH_PROFILE
__device__ unsigned long long g_search_prof[8];
#define AP_PROF_DECL unsigned long long prof_t = wall_clock64(), prof_acc[8] = {0, 0, 0, 0, 0, 0, 0, 0}
#define AP_PROF(i) do { const unsigned long long now_ = wall_clock64(); prof_acc[i] += now_ - prof_t; prof_t = now_; } while (0)
#define AP_PROF_FLUSH do { if (threadIdx.x == 0) for (int i_ = 0; i_ < 8; i_++) atomicAdd(&g_search_prof[i_], prof_acc[i_]); } while (0)
extern "C" int ap_debug_search_profile(unsigned long long out8[8]) {
    AP_CHECK_HIP(hipMemcpyFromSymbol(out8, HIP_SYMBOL(g_search_prof), sizeof(g_search_prof)));
    unsigned long long z[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    AP_CHECK_HIP(hipMemcpyToSymbol(HIP_SYMBOL(g_search_prof), z, sizeof(z)));
    return AP_OK;
}
#else
#define AP_PROF_DECL
#define AP_PROF(i)
#define AP_PROF_FLUSH
#endif

#define AP_CUS 256              // compute units of the chip
#define AP_LDS_BLOCKS 128       // what the LDS of one is handed out in ...
#define AP_LDS_BLOCK 1280       // ... bytes each
#define AP_SEARCH_STATIC 320    // bytes of k_search's static arrays beside its look-up tables, at most
// NT threads per workgroup.  256 (four waves) is the usual size: seven workgroups share a CU while the pool is small
// enough, and the register budget is the 72 VGPRs of seven waves per SIMD.  When the pool is so large that the LDS
// holds four workgroups or fewer, 512 or 1024 threads keep the CU's SIMDs occupied with one query's candidates.
#ifndef AP_SEARCH_WAVES_PER_SIMD
#define AP_SEARCH_WAVES_PER_SIMD 7
#endif
#ifndef AP_SEARCH_NT512_AT
#define AP_SEARCH_NT512_AT 4    // workgroups of 256 threads a CU's LDS holds at or below which 512 threads are used
#endif
#ifndef AP_SEARCH_NT1024_AT
#define AP_SEARCH_NT1024_AT 1   // ... and 1024 threads
#endif
// Wide bf16 rows (more than 1024 columns: 24 or 32 query values per lane) do not fit seven waves' registers without
// spilling; they run at five waves per SIMD.
template <int DT, int NV, int NT, bool LIST, bool KW> struct ApSearchWaves {
    static constexpr int MIN = LIST ? 4 : (DT == AP_BF16 && NV >= 3) ? (NT == 1024 ? 4 : 5) : NT == 128 && KW ? AP_SEARCH_WAVES_KW2 : NT <= 256 ? AP_SEARCH_WAVES_PER_SIMD : NT == 512 ? AP_SEARCH_WAVES_512 : 4;
};
// FLOOR: neighbours with a bound below the estimated end of the pool wait (large pools searched with bounds).
// LIST: an iteration's neighbours are listed by their ids and scored g.cmax at a time (large pools of which two then fit a CU).
template <int DT, int NV, bool KW, bool BIG, int NT, bool FLOOR, bool LIST = false>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(ApSearchWaves<DT, NV, NT, LIST, KW>::MIN, 8)))
void k_search(ApSearchArgs g) {
    static_assert(!LIST || (!KW && !BIG && NT == 512), "lists are for the plain search's large pools");
    static_assert(!FLOOR || (!KW && !BIG && NT >= 512), "the floor is for the plain search's large pools");
    extern __shared__ __attribute__((aligned(16))) uint64_t smem64[];   // 16-byte aligned: the descriptors are read as uint4
    // Large pools (workgroups of 512 or 1024 threads): the keys that cannot enter are dropped before sorting, and
    // parents are picked from a bitmap of the unexpanded entries.
    constexpr bool PIPE = !KW && !BIG && NT >= 512;
    constexpr int SPB = ApQTab<BIG>::SPB, TXB = ApQTab<BIG>::TXB;
    // The query's two look-up tables are a static array: at an address the compiler knows, so that a look-up's address
    // is the hash alone.  The dynamic part starts with this iteration's candidates: 16 bytes each, the document's
    // descriptor with its id in the fourth word.
    // PIPE: once the candidates are scored their space is free until the next gather, and holds the entering keys,
    // unordered (xk) and sorted (newS): what lets the largest pool (16384 entries) take sixteen parents' neighbours.
    __shared__ __attribute__((aligned(16))) uint64_t qtab[ApQTab<BIG>::SLOTS];
    uint4 *s_meta = reinterpret_cast<uint4 *>(smem64);
    uint64_t *cur = reinterpret_cast<uint64_t *>(s_meta + g.cmax);   // the pool: L keys, best first
    uint64_t *newk = cur + g.L;              // keys of this iteration's candidates, unordered
    uint64_t *newS = PIPE ? reinterpret_cast<uint64_t *>(s_meta) + g.cmax : newk + g.cmax;   // the same, sorted
    uint64_t *nxt = newk + (PIPE ? 1 : 2) * g.cmax;   // scratch of nxtw words (only wide searches of small pools need it)
    uint64_t *xk = PIPE ? reinterpret_cast<uint64_t *>(s_meta) : nxt + g.nxtw;   // cmax words.  KW: satisfying keys the pool did not keep in this iteration; PIPE: entering keys, unordered
    uint64_t *kwc = nxt + g.nxtw + (KW ? g.cmax : 0);   // KW: the secondary pool, k keys, best first
    uint64_t *umask = kwc + (KW ? g.k : 0);   // PIPE: one bit per pool entry; after it the visited set when it lives in LDS
    int32_t *s_ids = reinterpret_cast<int32_t *>(umask + (g.L + 63) / 64 + 1);   // LIST: the ids (umask also holds a word a block and one more)
    __shared__ int32_t s_cnt, s_nid, s_np, s_skip, s_drop, s_wait, s_stop, s_xn, s_kc, s_nin, s_rmin;
    __shared__ int32_t s_par[16], s_psat[16];
    __shared__ int32_t s_kw[AP_KW_MAX_TERMS], s_kwcol[AP_KW_MAX_TERMS];
    __shared__ int32_t s_seed[2];

    const int64_t q = (int64_t)g.q0 + blockIdx.x;
    const int lane = threadIdx.x & 63, wave = ap_wave_id();
    // the query's lists: look-up tables in LDS when they are short (the usual case), else left in global memory
    ApLists a;
    {
        const int64_t sb = g.Q.sp_indptr[q], tb = g.Q.tx_indptr[q];
        a.sp_n = (int32_t)(g.Q.sp_indptr[q + 1] - sb); a.tx_n = (int32_t)(g.Q.tx_indptr[q + 1] - tb);
        a.sp_idx = g.Q.sp_idx + sb; a.sp_val = g.Q.sp_val + sb; a.tx_idx = g.Q.tx_idx + tb; a.tx_val = g.Q.tx_val + tb;
    }
    // Wave 0 builds the two bucketed tables (lists of at most 64 / 32 entries; 256 / 128 for queries that are documents);
    // if no multiplier fits a list, or a list is longer, the lists are searched where they lie.
    bool use_tab = !g.no_tables && a.sp_n <= (1 << SPB) / 4 && a.tx_n <= (1 << TXB) / 4;   // uniform
    uint32_t msp = 0, mtx = 0;
    if (use_tab && wave == 0) {
        const int32_t s0 = ap_bucket_build<BIG ? 4 : 1>(a.sp_idx, a.sp_val, a.sp_n, qtab, SPB);
        const int32_t s1 = ap_bucket_build<BIG ? 2 : 1>(a.tx_idx, a.tx_val, a.tx_n, qtab + (1 << SPB), TXB);
        if (lane == 0) { s_seed[0] = s0; s_seed[1] = s1; }
    }
    __syncthreads();
    if (use_tab) {
        const int32_t seed0 = ap_uniform_i32(s_seed[0]), seed1 = ap_uniform_i32(s_seed[1]);
        use_tab = seed0 >= 0 && seed1 >= 0;
        if (use_tab) { msp = ap_seed_mult(seed0); mtx = ap_seed_mult(seed1); }
    }
    float qa[NV * ApDense<DT>::EPC];
    ap_load_aside<DT, NV, AP_F32>(g.Q.dense, q, g.D.dim, qa);
    float qnorm;
    {
        float p = 0.f;
#pragma unroll
        for (int i = 0; i < NV * ApDense<DT>::EPC; i++) p = fmaf(qa[i], qa[i], p);
        qnorm = sqrtf(ap_wave_sum(p));
    }
    const float wd = g.w[q * g.w_stride + 0], ws = g.w[q * g.w_stride + 1], wf = g.w[q * g.w_stride + 2];
    ApVisited vis{g.visited + (size_t)blockIdx.x * g.words, nullptr};
    uint64_t *marks = FLOOR ? g.marks + (size_t)blockIdx.x * g.words : nullptr;
    // marks document v as visited.  1: it was before; 2 (FLOOR): its bound reaches the floor
    auto meet = [&](int32_t v) -> uint32_t {
        if (!FLOOR) return vis.test_and_set(v) ? 1u : 0u;
        const uint64_t old = __hip_atomic_fetch_or(marks + (v >> 5), 1ull << (v & 31), __ATOMIC_RELAXED, AP_VIS_SCOPE);
        return ((uint32_t)old >> (v & 31) & 1u) | ((uint32_t)(old >> 32) >> (v & 31) & 1u) << 1;
    };
    if (g.vis_lds) {   // uniform
        vis.l = (AP_LDS uint32_t *)reinterpret_cast<uint32_t *>(umask + (PIPE ? (g.L + 63) / 64 : 0));
        for (size_t i = threadIdx.x; i < g.words; i += blockDim.x) vis.l[i] = 0u;
    }
    if (threadIdx.x == 0) { s_cnt = 0; s_nid = 0; s_skip = 0; s_drop = 0; s_wait = 0; s_xn = 0; s_kc = 0; s_nin = 0; }
    // the query's required terms, unused slots squeezed out (uniform)
    int32_t n_kw = 0;
    if (KW) {
        for (int32_t j = 0; j < g.kw_stride; j++) {
            const int32_t t = g.kw_terms[q * g.kw_stride + j];
            if (t >= 0) {
                if (threadIdx.x == 0) { s_kw[n_kw] = t; s_kwcol[n_kw] = g.bound && t < g.tx_vocab ? g.bound_col[t] : -1; }
                n_kw++;
            }
        }
    }
    const bool kw_on = KW && n_kw > 0;
    int32_t kc = 0;   // entries in the secondary pool (maintained by wave 0)
    __syncthreads();

    // S7: entry points
    for (int32_t i = threadIdx.x; i < g.E; i += blockDim.x) {
        const int32_t v = g.entry[i];
        if (v >= 0) {
            const bool seen = (meet(v) & 1u) != 0u;
            const uint4 m = g.meta[v];
            if (!seen) s_meta[atomicAdd(&s_cnt, 1)] = make_uint4(m.x, m.y, m.z, (uint32_t)v);
            if (FLOOR) reinterpret_cast<uint32_t *>(g.bound)[(int64_t)blockIdx.x * g.bound_ld + v] = 0xff800000u;   // -inf: scored
        }
    }
    __syncthreads();
    int32_t len = 0, it = 0, nscored = 0, nskipped = 0;
    int32_t fu = 0;   // every pool entry before this position has been expanded
    bool bound_on = false;  // the candidates of this iteration got past their bounds (uniform)
    int32_t ndropped = 0;   // per lane: neighbours its bound kept out
    uint32_t *bound = reinterpret_cast<uint32_t *>(g.bound) + (g.bound ? (int64_t)blockIdx.x * g.bound_ld : 0);
    // The floor: an estimate, from below, of the last score of the pool when the search ends (k_bound_floor).  Three
    // quarters of the documents that get past their bounds enter the pool early and leave it before they are ever expanded;
    // those with a bound below the floor are left waiting instead (marked visited, nothing read).  While every parent
    // scores at least the floor nothing that waits can rank before it, so the parents are the same; and when the pool is
    // full down to the floor nothing that waits can be in it.  Should the search get below the floor all the same, what
    // waits is found by its visited bits and bounds, scored and merged, and nothing waits from then on.  Documents that
    // were scored although their bound is below the floor (before waiting began) lose their bound, so that the scan passes
    // over them.  4,000 queries of 100,000 documents at beam 2112 : 16: 9,340 -> 4,740 documents scored, 39.0 -> 29.9 ms;
    // 2,000 of 500,000 at beam 8192 : 16: 34,900 -> 13,700, 102.6 -> 79.7 ms.
    // Whether a bound reaches the floor is a bit beside the visited bit, so that the one atomic tells both: of the neighbours met for the first time
    // only one in thirty has its bound read then, a line of memory each (all of them: as many bytes as the scoring reads).  The first
    // iterations, whose parents lie below the floor, take the highest of two lower floors that enough of the pool reaches.  Beam 2112 : 16
    // as above: 4,740 -> 3,820 documents scored, the search 26.7 -> 23.9 ms; beam 8192 : 16, where steps that wait for one another bound it: 13,700 ->
    // 13,070, 57.6 -> 56.5.
    const float4 floors = FLOOR ? g.bound_floor[blockIdx.x] : make_float4(0.f, 0.f, 0.f, 0.f);
    const float floor_score = floors.x;
    float level = -INFINITY;                      // uniform: the floor in force; what waits has a bound below it
    const uint32_t AP_NO_BOUND = 0xff800000u;   // -inf
    bool waiting = false, may_wait = FLOOR;       // uniform: something may wait; it may come to that
    int64_t scan = -1;                            // where the scan of what waits is, -1: none under way
    int32_t n_id = 0, next_id = 0;                // uniform: listed neighbours of this iteration, those taken from the list
    AP_PROF_DECL;
    for (;;) {
        AP_PROF(0);
        int32_t c = ap_uniform_i32(s_cnt);   // counts and keys that every thread reads alike are kept in scalar registers
        if (LIST && next_id < n_id) {   // uniform: the next of the listed neighbours
            c = n_id - next_id < g.cmax ? n_id - next_id : g.cmax;
            for (int32_t t = threadIdx.x; t < c; t += NT) {
                const int32_t v = s_ids[next_id + t];
                const uint4 m = g.meta[v];
                s_meta[t] = make_uint4(m.x, m.y, m.z, (uint32_t)v);
            }
            next_id += c;
            __syncthreads();
        }
        nscored += c;
        const bool pool_full = len == g.L;
        const uint64_t worst = pool_full ? ap_uniform_u64(cur[g.L - 1]) : 0ull;
        const float worst_score = ap_key_score(worst);
        const bool second_full = kw_on && s_kc == g.k;   // s_kc and kwc were last written before the previous barriers
        const float second_worst = second_full ? ap_key_score(kwc[g.k - 1]) : 0.f;
        constexpr int G = ApSearchG<NT, LIST>::G;
        if (use_tab)
            nskipped += ap_score_candidates<DT, NV, true, KW, BIG, NT / 64, G>(g.D, g.rec, qa, qtab, a, wd, ws, wf, qnorm, pool_full, worst_score,
                                                                 s_meta, c, newk, s_kw, n_kw, g.kw_all != 0, second_full, second_worst, msp, mtx, bound_on);
        else
            nskipped += ap_score_candidates<DT, NV, false, KW, BIG, NT / 64, G>(g.D, g.rec, qa, qtab, a, wd, ws, wf, qnorm, pool_full, worst_score,
                                                                  s_meta, c, newk, s_kw, n_kw, g.kw_all != 0, second_full, second_worst, 0u, 0u, bound_on);
        AP_PROF(1);
        __syncthreads();
        AP_PROF(2);
        if (threadIdx.x == 0) s_cnt = 0;   // every thread has read this iteration's count; the gather counts anew after further barriers
        int32_t cin;
        if (PIPE) {
            // Only keys that rank before the pool's last entry can enter (any key while the pool has room): late in a
            // search they are a small part of the iteration's candidates, so they are picked out first (unordered, in
            // xk) and ranked among themselves afterwards.
            for (int32_t t = threadIdx.x; t < c; t += blockDim.x) {
                const uint64_t key = newk[t];
                if ((key >> 32) != 0ull && key > worst) xk[atomicAdd(&s_nin, 1)] = key;
            }
            __syncthreads();
            cin = ap_uniform_i32(s_nin);
            // A group of AP_RANK_LANES lanes per entering key finds both of its ranks: among the entering keys (a compare
            // per lane and step) and among the pool (as many probes a step as the group has lanes: four steps of 16
            // for 16384 entries instead of fourteen halvings).  The first gives the key its place in newS, the second
            // goes to rr (in newk's space, which is free now).  Late in a search few keys enter, and what costs is the
            // chain of dependent LDS reads per key: four keys share a wave's steps.
            constexpr int GL = AP_RANK_LANES, GSH = GL == 64 ? 6 : GL == 32 ? 5 : 4, GPW = 64 / GL;
            static_assert(GL == 16 || GL == 32 || GL == 64, "lanes per key");
            const int grp = lane >> GSH, gl = lane & (GL - 1);
            auto group_count = [&](bool p) -> int32_t {   // lanes of this lane's group for which p holds
                const uint64_t m = __ballot(p);
                if (GL == 64) return (int32_t)__popcll(m);
                return (int32_t)__popc((uint32_t)(m >> (grp * GL)) & (GL == 32 ? 0xffffffffu : 0xffffu));
            };
            int32_t *rr = reinterpret_cast<int32_t *>(newk);
            // Many keys enter while the pool fills: from AP_RANK_SORT on they are sorted where they lie (the squared number of
            // compares is what costs there: 1,024 keys took 93 us of ranking; the array and newS behind it hold them padded
            // to a power of two).
            const bool sorted = cin > AP_RANK_SORT;   // uniform
            if (sorted) {
                int32_t n2 = AP_RANK_SORT;
                while (n2 < cin) n2 <<= 1;
                for (int32_t t = cin + (int32_t)threadIdx.x; t < n2; t += NT) xk[t] = 0ull;
                for (int32_t size = 2; size <= n2; size <<= 1)
                    for (int32_t stride = size >> 1; stride > 0; stride >>= 1) {
                        // pairs closer than 64 keys lie inside one wave's 128 keys: no barrier between those steps
                        if (stride >= 64 || stride == size >> 1) __syncthreads(); else ap_wave_sync();
                        for (int32_t t = threadIdx.x; t < (n2 >> 1); t += NT) {
                            const int32_t x = 2 * t - (t & (stride - 1)), y = x + stride;
                            const uint64_t kx = xk[x], ky = xk[y];
                            if ((kx < ky) == ((x & size) == 0)) { xk[x] = ky; xk[y] = kx; }
                        }
                    }
                __syncthreads();
                newS = xk;
            } else newS = reinterpret_cast<uint64_t *>(s_meta) + g.cmax;
            for (int32_t j0 = wave * GPW; j0 < cin; j0 += NT / 64 * GPW) {
                const int32_t j = j0 + grp;
                const bool on = j < cin;
                const uint64_t key = on ? xk[j] : 0ull;
                int32_t e = j;
                if (!sorted) {
                    e = 0;
                    for (int32_t i0 = 0; i0 < cin; i0 += GL) e += group_count(on && i0 + gl < cin && xk[i0 + gl] > key);
                }
                int32_t lo = 0, hi = on ? len : 0;   // the rank (number of pool entries that rank before the key) lies in [lo, hi]
                while (__any(hi > lo)) {
                    const int32_t step = (hi - lo + GL - 1) >> GSH;
                    const int32_t at = lo + (gl + 1) * step - 1;
                    const int32_t n_before = group_count(hi > lo && at < hi && cur[at] > key);
                    const int32_t nlo = lo + n_before * step, nhi = lo + (n_before + 1) * step - 1;
                    if (hi > lo) { lo = nlo; hi = nhi < hi ? nhi : hi; }
                }
                if (on && gl == 0) { if (!sorted) newS[e] = key; rr[e] = lo; }
            }
            __syncthreads();
            if (threadIdx.x == 0) s_nin = 0;   // next touched after the barriers of the merge or the pick
        } else {
            // sort the new keys by ranking them among themselves; only those that
            // rank before the pool's last entry (when the pool is full) can enter
            for (int32_t t = threadIdx.x; t < c; t += blockDim.x) {
                const uint64_t key = newk[t];
                int32_t r = 0;
                for (int32_t j = 0; j < c; j++) r += newk[j] > key;
                newS[r] = key;
            }
            __syncthreads();
            cin = ap_uniform_i32(ap_rank_in(newS, c, worst));   // new keys that rank before `worst` (all of them while the pool has room)
        }
        AP_PROF(3);
        if (kw_on) {
            // scored, satisfying, but ranked after the full pool's last entry: to the secondary pool
            for (int32_t t = cin + (int32_t)threadIdx.x; t < c; t += blockDim.x) {
                const uint64_t key = newS[t];
                if ((key >> 32) != 0ull && (key & 2ull)) xk[atomicAdd(&s_xn, 1)] = key;
            }
        }
        if (PIPE && cin > 0) {
            // In-place rank merge of a large pool.  The entering keys are few against the pool, so what costs is
            // latency and barriers: the number of entering keys that land before each 64-entry block of the pool is
            // tabulated, after which a pool entry finds how far it moves with two reads; entries from the first
            // insertion point on are read in chunks of 4 NT from the back of the pool to the front and written one
            // barrier later (a chunk's writes never reach below its own start).
            const int32_t *rr = reinterpret_cast<const int32_t *>(newk);   // rank of every entering key among the pool, ascending
            int32_t *bshift = reinterpret_cast<int32_t *>(umask);          // entering keys that land before block b
            const int32_t rmin = ap_uniform_i32(rr[0]);
            fu = fu < rmin ? fu : rmin;   // the best entering key lands at rmin, unexpanded; entries before it stay put
            const int32_t nb = (len + 63) >> 6;
            for (int32_t b = threadIdx.x; b <= nb; b += NT) {   // number of ranks below 64 b
                int32_t lo = 0, hi = cin;
                while (lo < hi) {
                    const int32_t mid = (lo + hi) >> 1;
                    if (rr[mid] < 64 * b) lo = mid + 1; else hi = mid;
                }
                bshift[b] = lo;
            }
            __syncthreads();
            constexpr int CH = 4;
            for (int32_t hi = len; hi > rmin; hi -= CH * NT) {
                const int32_t lo = hi - CH * NT > rmin ? hi - CH * NT : rmin;
                uint64_t held[CH]; int32_t dest[CH];
#pragma unroll
                for (int m = 0; m < CH; m++) {
                    const int32_t t = lo + (int32_t)threadIdx.x + NT * m;
                    dest[m] = g.L;
                    if (t < hi) {
                        held[m] = cur[t];
                        int32_t k = bshift[t >> 6];
                        while (k < cin && rr[k] <= t) k++;   // insertion points inside the entry's own block: rarely any
                        dest[m] = t + k;
                    }
                }
                __syncthreads();
#pragma unroll
                for (int m = 0; m < CH; m++)
                    if (dest[m] < g.L) cur[dest[m]] = held[m];
                // no barrier here: these writes land at or after `lo`, the next chunk's reads come before it
            }
            for (int32_t t = threadIdx.x; t < cin; t += NT) {
                const int32_t r = rr[t] + t;
                if (r < g.L) cur[r] = newS[t];
            }
            len = len + cin < g.L ? len + cin : g.L;
            __syncthreads();
        } else if (cin > 0) {
            // In-place rank merge.  A pool entry at position t moves up by the number of entering keys that rank
            // before it, so only entries from the first insertion point on move, and they only move towards the
            // end: chunks of 2 NT entries are read, then (one barrier later) written, from the back of the pool to the
            // front.  A chunk's writes never reach below its own start, so they need not be fenced from the reads of
            // the chunk before it; the barrier of that chunk orders them before its writes.
            uint64_t nkey = 0; int32_t npos = g.L;
            if ((int32_t)threadIdx.x < cin) { nkey = newS[threadIdx.x]; npos = (int32_t)threadIdx.x + ap_rank_in(cur, len, nkey); }
            if (threadIdx.x == 0) s_rmin = npos;   // where the best entering key lands
            for (int32_t t = (int32_t)threadIdx.x + NT; t < cin; t += NT) {   // more entering keys than threads (wide searches)
                const uint64_t key = newS[t];
                nxt[t] = (uint64_t)(uint32_t)(t + ap_rank_in(cur, len, key));   // park the positions in the scratch array
            }
            __syncthreads();
            const int32_t rmin = ap_uniform_i32(s_rmin);
            fu = fu < rmin ? fu : rmin;   // the best entering key lands at rmin, unexpanded; entries before it stay put
            for (int32_t hi = len; hi > rmin; hi -= 2 * NT) {
                const int32_t lo = hi - 2 * NT > rmin ? hi - 2 * NT : rmin;
                uint64_t held[2]; int32_t dest[2];
#pragma unroll
                for (int m = 0; m < 2; m++) {
                    const int32_t t = lo + (int32_t)threadIdx.x + NT * m;
                    dest[m] = g.L;
                    if (t < hi) { held[m] = cur[t]; dest[m] = t + ap_rank_in(newS, cin, held[m]); }
                }
                __syncthreads();
#pragma unroll
                for (int m = 0; m < 2; m++) {
                    if (dest[m] < g.L) cur[dest[m]] = held[m];
                    else if (kw_on && lo + (int32_t)threadIdx.x + NT * m < hi && (held[m] & 2ull)) xk[atomicAdd(&s_xn, 1)] = held[m];   // evicted
                }
                // no barrier here: these writes land at or after `lo`, the next chunk's reads come before it
            }
            if (npos < g.L) cur[npos] = nkey;
            else if (kw_on && (int32_t)threadIdx.x < cin && (nkey & 2ull)) xk[atomicAdd(&s_xn, 1)] = nkey;
            for (int32_t t = (int32_t)threadIdx.x + NT; t < cin; t += NT) {
                const int32_t r = (int32_t)(uint32_t)nxt[t];
                if (r < g.L) cur[r] = newS[t];
                else if (kw_on && (newS[t] & 2ull)) xk[atomicAdd(&s_xn, 1)] = newS[t];
            }
            len = len + cin < g.L ? len + cin : g.L;
            __syncthreads();
        }
        if (kw_on) {
            // the secondary pool keeps the k best of everything handed over so far (any order of arrival gives the same k)
            __syncthreads();
            if (wave == 0) {
                const int32_t m = s_xn;
                if (g.deleted) {   // a mark-deleted document cannot be an answer: it does not take a place here
                    for (int32_t j = lane; j < m; j += 64) {
                        const int32_t v = ap_pool_id<KW>(xk[j]);
                        if ((g.deleted[v >> 5] >> (v & 31)) & 1u) xk[j] = 0ull;
                    }
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                }
                for (int32_t j = 0; j < m; j++) {
                    const uint64_t key = xk[j] & ~1ull;
                    if (key == 0ull || (kc == g.k && key < kwc[kc - 1])) continue;
                    int32_t pos = 0;
                    for (int32_t base = 0; base < kc; base += 64) {
                        const int32_t i = base + lane;
                        pos += __popcll(__ballot(i < kc && kwc[i] > key));
                    }
                    const int32_t last = kc < g.k ? kc : g.k - 1;   // entries [pos, last) move one place towards the end
                    for (int32_t hi = last; hi > pos; hi -= 64) {
                        const int32_t lo = hi - 64 > pos ? hi - 64 : pos;
                        const int32_t i = lo + lane;
                        uint64_t h = 0;
                        if (i < hi) h = kwc[i];
                        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                        __builtin_amdgcn_wave_barrier();
                        if (i < hi) kwc[i + 1] = h;
                        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                        __builtin_amdgcn_wave_barrier();
                    }
                    if (lane == 0) kwc[pos] = key;
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    kc = kc < g.k ? kc + 1 : g.k;
                }
                if (lane == 0) { s_xn = 0; s_kc = kc; }
            }
        }
        AP_PROF(4);
        if (LIST && next_id < n_id) {
            if (cin == 0) __syncthreads();   // else the merge has ended with one
            continue;
        }
        if (g.max_iters > 0 && it >= g.max_iters) break;
        // S8: pick the best `width` unexpanded entries (wave 0), mark them expanded
        int32_t pipe_np = 0;
        // Parents below the floor, or too few of them, while documents wait that the pool might hold: those come first.
        auto release = [&](int32_t found, bool below) -> bool {
            if (found == g.width && !below) return false;
            return !(len == g.L && ap_key_score(ap_uniform_u64(cur[g.L - 1])) >= level);
        };
        if (!FLOOR || scan < 0) {
        if (FLOOR && may_wait && !waiting) waiting = ap_uniform_i32(s_wait) != 0;   // not again once what waited has been scanned
        if (PIPE) {
            // Late in a search the unexpanded entries are few and far apart, and a scan by one wave would walk most of
            // the pool: every wave reduces its share of the pool from the cursor on to one bit per entry, and wave 0
            // picks from the bits.
            const int32_t b0 = fu >> 6, nb = (len + 63) >> 6;
            for (int32_t b = b0 + wave; b < nb; b += NT / 64) {
                const int32_t i = b * 64 + lane;
                const uint64_t m = __ballot(i < len && (cur[i] & 1ull));
                if (lane == 0) umask[b] = m;
            }
            __syncthreads();
            // Every wave picks for itself (the same scalar steps over the same bits, so the same parents): the first
            // `width` set bits are found with uniform steps and lane j takes the j-th.  No barrier is needed between
            // the pick and the gather of the parents' neighbours; wave 0 marks the parents expanded.
            int32_t found = 0, last = -1, mine = -1;
            for (int32_t base = b0; base < nb && found < g.width; base += 64) {
                const int32_t b = base + lane;
                const uint64_t m = b < nb ? umask[b] : 0ull;
                uint64_t nz = __ballot(m != 0ull);
                while (nz != 0ull && found < g.width) {
                    const int32_t src = (int32_t)__builtin_ctzll(nz);
                    nz &= nz - 1ull;
                    uint64_t word = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int32_t)(m >> 32), src) << 32) |
                                    (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int32_t)(uint32_t)m, src);
                    while (word != 0ull && found < g.width) {
                        last = (base + src) * 64 + (int32_t)__builtin_ctzll(word);
                        word &= word - 1ull;
                        if (lane == found) mine = last;
                        found++;
                    }
                }
            }
            const uint64_t pkey = mine >= 0 ? cur[mine] : 0ull;
            if (FLOOR && waiting && release(found, __any(mine >= 0 && !(ap_key_score(pkey) >= level)))) scan = 0;   // a NaN counts as below
            else {
                if (mine >= 0) {
                    s_par[lane] = ap_pool_id<KW>(pkey);     // every wave stores the same ids
                    if (wave == 0) cur[mine] = pkey & ~1ull;   // only the flag changes: a wave that reads the entry meanwhile gets the same id
                }
                ap_wave_sync();
                pipe_np = found;
                fu = last >= 0 ? last + 1 : len;   // everything up to the last entry taken is expanded now
            }
        } else if (wave == 0) {
            int32_t found = 0, last = -1;
            for (int32_t base = fu & ~63; base < len && found < g.width; base += 64) {   // the scan starts where it can first succeed
                const int32_t i = base + lane;
                const bool un = i < len && (cur[i] & 1ull);
                const uint64_t mask = __ballot(un);
                const int32_t rank = __popcll(mask & ((1ull << lane) - 1ull));
                const bool take = un && found + rank < g.width;
                if (take) {
                    s_par[found + rank] = ap_pool_id<KW>(cur[i]);
                    if (KW) s_psat[found + rank] = (int32_t)((cur[i] >> 1) & 1ull);
                    cur[i] &= ~1ull;
                }
                const uint64_t tmask = __ballot(take);
                if (tmask) last = base + 63 - (int32_t)__builtin_clzll(tmask);
                found += __popcll(mask);
            }
            fu = last >= 0 ? last + 1 : len;   // everything up to the last entry taken is expanded now
            if (lane == 0) s_np = found < g.width ? found : g.width;
        }
        if (!PIPE) __syncthreads();
        AP_PROF(5);
        }
        if (FLOOR && scan >= 0) {
            // what waits, as many documents at a time as the candidates' array holds; then nothing waits any more
            if (scan == 0 && threadIdx.x == 0) s_stop = 0x7fffffff;
            waiting = false; may_wait = false; bound_on = len == g.L;
            const float lowest = bound_on ? ap_key_score(ap_uniform_u64(cur[g.L - 1])) : -INFINITY;
            __syncthreads();
            constexpr int SU = 8;
            int32_t taken = 0;
            while (scan < g.D.n && taken < g.cmax) {   // uniform
                for (int j = 0; j < SU; j++) {
                    const int64_t v = scan + j * NT + threadIdx.x;
                    if (v >= g.D.n) continue;
                    const uint64_t mark = __hip_atomic_load(marks + (v >> 5), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> (v & 31);
                    if ((mark & (1ull | 1ull << 32)) != 1ull) continue;   // met, with a bound below the floor
                    const uint32_t e = bound[v];
                    const float ub = __uint_as_float(e & ~AP_BOUND_COUNT);
                    if (e == AP_NO_BOUND || !(ub < floor_score) || ub < lowest) continue;
                    const int32_t pos = atomicAdd(&s_cnt, 1);
                    if (pos >= g.cmax) { atomicMin(&s_stop, (int32_t)v); continue; }
                    const uint4 m = g.meta[v];
                    s_meta[pos] = make_uint4(m.x, m.y, m.z, (uint32_t)v);
                    bound[v] = AP_NO_BOUND;
                    ndropped--;   // it will be counted with the candidates
                }
                __syncthreads();
                taken = ap_uniform_i32(s_cnt);
                scan += SU * NT;
                __syncthreads();   // everyone has read the count before the next documents are added to it
            }
            if (taken > g.cmax) scan = ap_uniform_i32(s_stop);   // the array is full: on from the first document it could not take
            __syncthreads();
            if (threadIdx.x == 0) { if (taken > g.cmax) s_cnt = g.cmax; s_stop = 0x7fffffff; }
            if (scan >= g.D.n) scan = -1;
            __syncthreads();
            continue;
        }
        const int32_t np = PIPE ? pipe_np : ap_uniform_i32(s_np);
        if (np == 0) break;
        // neighbours of the parents that were never seen before; a parent that satisfies the keyword
        // constraint also brings its keyword edges
        // The bounds of all documents, where the call has them, are looked at first: while the pool is full, a neighbour
        // whose bound lies below the pool's last score cannot enter (nor, with keywords, the secondary pool) and is only
        // marked visited: its descriptor, record and dense row are not read.
        const int32_t per = g.R + (KW ? g.KR : 0);
        bound_on = g.bound && len == g.L;
        const float b_worst = bound_on ? ap_key_score(ap_uniform_u64(cur[g.L - 1])) : -INFINITY;
        const bool b_second_full = kw_on && s_kc == g.k;
        // Waiting begins once the pool holds a few iterations' parents that score at least the floor; below a lower floor, which far more
        // of the neighbours to come reach, once it holds the next iteration's.
        if (FLOOR && may_wait && level < floor_score) {
            const int32_t m_on = 4 * g.width + 16 < g.L ? 4 * g.width + 16 : g.L;
            const int64_t next = (int64_t)(it + 1) * g.width + (g.width > 16 ? g.width : 16);
            if (len >= m_on && ap_key_score(ap_uniform_u64(cur[m_on - 1])) >= floor_score) level = floor_score;
            else if (len >= next) {
                const float at = ap_key_score(ap_uniform_u64(cur[next - 1]));
                level = fmaxf(level, at >= floors.y ? floors.y : at >= floors.z ? floors.z : -INFINITY);
            }
        }
        const bool wait_on = FLOOR && may_wait && level > -INFINITY;
        const bool by_bit = wait_on && level == floor_score;   // whether a neighbour waits is its bit
        const float b_second = b_second_full ? ap_key_score(kwc[g.k - 1]) : 0.f;
        auto neighbour = [&](int32_t i) -> int32_t {
            if (KW) {
                const int32_t pi = i / per, sl = i % per, u = s_par[pi];
                if (sl < g.R) return g.graph[(int64_t)u * g.R + sl];
                return g.kw_use_edges && s_psat[pi] && sl - g.R < g.kw_count[u] ? g.kw_edges[(int64_t)u * g.KR + (sl - g.R)] : -1;
            }
            return g.graph[(int64_t)s_par[i / g.R] * g.R + (i % g.R)];
        };
        if (bound_on || wait_on) {
            // two neighbours a thread at a time, step by step, so that the round trips of one run beside the other's
            constexpr int GU = 2;
            for (int32_t i0 = threadIdx.x; i0 < np * per; i0 += GU * NT) {
                int32_t v[GU];
                uint32_t e[GU];
                bool low[GU];
#pragma unroll
                for (int j = 0; j < GU; j++) v[j] = i0 + j * NT < np * per ? neighbour(i0 + j * NT) : -1;
#pragma unroll
                for (int j = 0; j < GU; j++) {
                    low[j] = false;
                    if (v[j] < 0) continue;
                    const uint32_t met = meet(v[j]);
                    low[j] = FLOOR && may_wait && !(met & 2u);   // its bound lies below the floor
                    if (met & 1u) v[j] = -1;
                    else if (FLOOR && by_bit && low[j]) {   // waits, or cannot enter anyway
                        if (!(b_worst >= floor_score)) s_wait = 1;
                        ndropped++;
                        v[j] = -1;
                    }
                }
#pragma unroll
                for (int j = 0; j < GU; j++) e[j] = v[j] >= 0 && (!FLOOR || bound_on || low[j]) ? bound[v[j]] : 0x7f800000u;
#pragma unroll
                for (int j = 0; j < GU; j++) {
                    if (v[j] < 0) continue;
                    const float ub = __uint_as_float(e[j] & ~AP_BOUND_COUNT);
                    bool out = bound_on && ub < b_worst;
                    const bool wait = FLOOR && wait_on && ub < level && !out;
                    if (kw_on && out) {
                        int32_t held = (int32_t)(e[j] & AP_BOUND_COUNT);
                        for (int32_t t = 0; t < n_kw; t++)
                            if (s_kwcol[t] >= 0) held += (int32_t)((g.bound_bits[(int64_t)s_kwcol[t] * (int64_t)g.words + (v[j] >> 5)] >> (v[j] & 31)) & 1u);
                        if (g.kw_all ? held == n_kw : held > 0) out = b_second_full && ub < b_second;
                    }
                    if (out) { ndropped++; continue; }
                    if (wait) { s_wait = 1; ndropped++; continue; }
                    if (FLOOR && low[j]) bound[v[j]] = AP_NO_BOUND;
                    if (LIST) { s_ids[atomicAdd(&s_nid, 1)] = v[j]; continue; }
                    const uint4 m = g.meta[v[j]];
                    s_meta[atomicAdd(&s_cnt, 1)] = make_uint4(m.x, m.y, m.z, (uint32_t)v[j]);
                }
            }
        } else {
            for (int32_t i = threadIdx.x; i < np * per; i += NT) {
                const int32_t v = neighbour(i);
                if (v >= 0) {
                    // the descriptor (where the record is, how long, the dense norm) is fetched along with the visited
                    // test, not after it: one memory round trip less per iteration for 16 bytes per neighbour already seen
                    const uint32_t met = meet(v);
                    const bool seen = (met & 1u) != 0u;
                    if (LIST) { if (!seen) s_ids[atomicAdd(&s_nid, 1)] = v; }
                    else {
                        const uint4 m = g.meta[v];
                        if (!seen) s_meta[atomicAdd(&s_cnt, 1)] = make_uint4(m.x, m.y, m.z, (uint32_t)v);
                    }
                    if (FLOOR && met == 0u && may_wait) bound[v] = AP_NO_BOUND;
                }
            }
        }
        __syncthreads();
        if (LIST) {
            n_id = ap_uniform_i32(s_nid);
            next_id = 0;
            __syncthreads();   // everyone has read the count
            if (threadIdx.x == 0) s_nid = 0;   // next touched after further barriers
        }
        AP_PROF(6);
        it++;
    }
    AP_PROF_FLUSH;
    if (lane == 0) atomicAdd(&s_skip, nskipped);
    if (g.bound && ndropped) atomicAdd(&s_drop, ndropped);
    __syncthreads();
    nscored += s_drop;   // a dropped neighbour counts like any other that was decided without its dense row
    if (threadIdx.x == 0 && g.counts) { g.counts[q * 3] = nscored; g.counts[q * 3 + 1] = it; g.counts[q * 3 + 2] = s_skip + s_drop; }
    // S9
    if (kw_on) {
        // Everything in the secondary pool ranked after the pool's last entry when it was handed over, and that
        // entry only ever improves: the satisfying pool entries in order, then the secondary pool, is the merged order.
        if (wave == 0) {
            int32_t o = 0;
            for (int32_t base = 0; base < len && o < g.k; base += 64) {
                const int32_t i = base + lane;
                bool sat = i < len && (cur[i] & 2ull);
                if (sat && g.deleted) { const int32_t v = ap_pool_id<KW>(cur[i]); sat = !((g.deleted[v >> 5] >> (v & 31)) & 1u); }
                const uint64_t mask = __ballot(sat);
                const int32_t at = o + __popcll(mask & ((1ull << lane) - 1ull));
                if (sat && at < g.k) {
                    g.out_ids[q * g.k + at] = ap_pool_id<KW>(cur[i]);
                    g.out_scores[q * g.k + at] = ap_key_score(cur[i]);
                }
                o += __popcll(mask);
            }
            o = o < g.k ? o : g.k;
            for (int32_t i = o + lane; i < g.k; i += 64) {
                const bool have = i - o < kc;
                g.out_ids[q * g.k + i] = have ? ap_pool_id<KW>(kwc[i - o]) : -1;
                g.out_scores[q * g.k + i] = have ? ap_key_score(kwc[i - o]) : -INFINITY;
            }
        }
        return;
    }
    if (KW && g.deleted) {
        // mark-deletion (searches on an index with deletions always run this instantiation): the best k live pool entries
        if (wave == 0) {
            int32_t o = 0;
            for (int32_t base = 0; base < len && o < g.k; base += 64) {
                const int32_t i = base + lane;
                bool live = i < len;
                if (live) { const int32_t v = ap_pool_id<KW>(cur[i]); live = !((g.deleted[v >> 5] >> (v & 31)) & 1u); }
                const uint64_t mask = __ballot(live);
                const int32_t at = o + __popcll(mask & ((1ull << lane) - 1ull));
                if (live && at < g.k) {
                    g.out_ids[q * g.k + at] = ap_pool_id<KW>(cur[i]);
                    g.out_scores[q * g.k + at] = ap_key_score(cur[i]);
                }
                o += __popcll(mask);
            }
            for (int32_t i = (o < g.k ? o : g.k) + lane; i < g.k; i += 64) { g.out_ids[q * g.k + i] = -1; g.out_scores[q * g.k + i] = -INFINITY; }
        }
        return;
    }
    for (int32_t i = threadIdx.x; i < g.k; i += blockDim.x) {
        g.out_ids[q * g.k + i] = i < len ? ap_pool_id<KW>(cur[i]) : -1;
        g.out_scores[q * g.k + i] = i < len ? ap_key_score(cur[i]) : -INFINITY;
    }
}

// Default cap of the index-owned workspace: 2 GiB of visited bits (16,384 queries of a million documents at a time).
#define AP_SEARCH_WS_BYTES ((size_t)2 << 30)

// What the bounds of all documents cost, by what was measured (microseconds): a document's columns are read once (0.4 ns), a
// tile of 256 queries takes 3.1 ps a pair at 1,280 columns and 1.1 ps for the tail of 165 entries a document, which grows with the lists (519 entries 3.1,
// 1,254 7.3, 2,259 12); up to 64 queries take one pass over the columns (0.54 to 0.97 ns a document; 37 queries of 1,254 entries 25 us more for 20,000).
static double ap_list_share(const ap_index *ix) { return std::max(1.0, (double)(ix->sp_nnz + ix->tx_nnz) / (165.0 * (double)ix->docs.n)); }
double ap_bound_cost(const ap_index *ix, int64_t nq) {
    const double cols = (double)((ix->bd_kd ? ix->bd_kd : ix->docs.dim) + ix->bd_kh) / 1280.0, tiles = (double)((nq + 255) / 256), lists = ap_list_share(ix);
    if (nq <= AP_BOUND_FEW) return 15.0 + (double)ix->docs.n * ((0.55e-3 + 7e-6 * (double)nq) * cols + 5e-6 * (double)nq * (lists - 1.0));
    return 15.0 + (double)ix->docs.n * (0.4e-3 * cols + tiles * 256.0 * (3.1e-6 * cols + 1.1e-6 * lists));
}

// Whether that is less than they save:
//  - a search that does without: 0.22 ns more for every document it reaches while the chip is full (10,000 queries of 100,000
//    documents: 0.22 to 0.28 where both take the same time, which is at pools of 16, 25 and 36 entries for 128 f32, 768 f32 and
//    1,024 bf16 columns; at 128 entries of 768 f32 columns 22.1 ms without bounds, 10.5 with them);
//  - while it is not, so much more an iteration (60,000 to 150,000 documents of 128 and 768 f32 and 1,024 bf16 columns, pools of 10 and 16, where the line lies):
//      degree      1 query      8      29      64     200   1,000
//        64         11..22  16..29  24..34  29..36  32..44  37..49 us
//        32          5..11   9..12  10..17  13..21  14..22  17..25
//        16          2.. 4   3.. 4   4.. 8   5.. 9   6..12   8..15
//    and 10 to 20 at degree 64 with pools of 128, where it no longer matters (one query 2.53 and 0.79 ms).  1,000 queries of 100,000 f32 documents at degree 16, pool 16:
//    0.32 ms without bounds, 0.67 with them; 24 at degree 64, pool 10: 0.47 and 0.23;
//  - with keywords, whose parents have half as many edges again, 0.26 to 0.41 ns a document and 0.30 to 0.71 us an edge that an iteration of 200 to 1,000 queries has (4,000
//    queries of 60,000 bf16 documents at degree 64, pool 16: 2.84 ms without bounds, 1.99 with them; 1,000 of 128 f32 columns at degree 32, pool 10: 0.66 and 0.48);
//  - more where documents have long lists, which a search without bounds reads (1,254 entries, 768 f32 columns, degree 64: 2.4 to 3.5 ns a document, and an
//    iteration of one query 80 us, of 24 to 1,000 190 to 240).  4,000 queries of 100,000 such documents, pools of 10, 16 and 24: 9.2, 13.1 and 19.2 ms
//    without bounds, 5.0, 5.4 and 6.0 with them.
bool ap_bound_pays(const ap_index *ix, int64_t nq, int32_t beam, int32_t width, int32_t max_iters, bool keywords) {
    if (!ix->bd_mem || g_ap_debug.search_bounds == 1 || nq < 1) return false;
    const double n = (double)ix->docs.n;
    if ((double)AP_BOUND_WS_BYTES / (4.0 * n) < (double)std::min<int64_t>(nq, 256)) return false;   // slabs too small to fill the chip
    if (g_ap_debug.search_bounds == 2) return true;
    double iters = (double)beam / width;
    if (max_iters > 0) iters = std::min(iters, (double)max_iters);
    const double edges = ix->params.degree * (keywords ? 1.5 : 1.0), reached = n * (1.0 - exp(-iters * width * edges / n));
    const double iteration = std::min(40.0, 12.0 + 4.0 * log2((double)nq)) * pow(std::min(edges, 96.0) / 64.0, 1.25);
    const double lists = ap_list_share(ix);
    return std::max((double)nq * reached * (keywords ? 0.35e-3 : 0.22e-3) * (1.5 * lists - 0.5), iters * iteration * lists) > ap_bound_cost(ix, nq);
}

// Queries per slab when `cap_words` words are available: as many as fit, then evened out over the slabs.
static int32_t ap_slab_size(int32_t nq, size_t words, size_t cap_words) {
    size_t fit = std::max<size_t>(1, cap_words / std::max<size_t>(words, 1));
    fit = std::min<size_t>(fit, (size_t)1 << 21);   // a launch of workgroups of up to 1024 threads holds fewer than 2^32 threads
    if (fit >= (size_t)nq) return nq;
    const size_t slabs = ((size_t)nq + fit - 1) / fit;
    return (int32_t)(((size_t)nq + slabs - 1) / slabs);
}

// Sizes the workspace an index owns (grow only) for a call of nq queries.
int ap_search_reserve(ap_index *ix, int32_t nq, hipStream_t st, ApSearchWs *ws, bool bounds, const ApWalkPlan &plan, bool marks) {
    const size_t words = ((size_t)ix->docs.n + 31) / 32;
    const size_t cap_bytes = g_ap_debug.search_workspace_bytes > 0 ? (size_t)g_ap_debug.search_workspace_bytes : AP_SEARCH_WS_BYTES;
    ws->slab = ap_slab_size(nq, words, cap_bytes / 4);
    const size_t need = words * (size_t)ws->slab;
    if (need > ix->visited_words) {
        if (ix->visited) { AP_CHECK_HIP(hipStreamSynchronize(st)); (void)hipFree(ix->visited); ix->visited = nullptr; ix->visited_words = 0; }
        AP_TRY(ap_bound_make_room(ix, st, &ix->visited, need));
        ix->visited_words = need;
    }
    if ((size_t)nq * 3 > ix->search_counts_cap) {
        if (ix->search_counts) { AP_CHECK_HIP(hipStreamSynchronize(st)); (void)hipFree(ix->search_counts); ix->search_counts = nullptr; ix->search_counts_cap = 0; }
        AP_TRY(ap_dev_alloc(&ix->search_counts, (size_t)nq * 3));
        ix->search_counts_cap = (size_t)nq * 3;
    }
    if (!ix->ev_search[0]) {
        AP_CHECK_HIP(hipEventCreate(&ix->ev_search[0]));
        AP_CHECK_HIP(hipEventCreate(&ix->ev_search[1]));
    }
    ws->visited = ix->visited;
    ws->counts = ix->search_counts;
    ws->ev0 = ix->ev_search[0]; ws->ev1 = ix->ev_search[1];
    ix->last_nq = nq;
    // The bounds come last, and what the search cannot do without is sized as if there were none: they never take the memory
    // of a search that used to fit, and the same batch can run without them afterwards (captured, say) and allocate nothing.
    if (plan.mode != 0 && ws->slab == nq) {   // a small batch, as a whole or not at all
        AP_TRY(ap_bound_reserve(ix, nq, AP_BOUND_WHOLE, AP_BOUND_WS_BYTES, plan.mode == 1 ? 2 : 1, st, &ws->bound));
        if (ws->bound.table) {
            ws->walk.bound = plan.mode == 1 ? ws->bound.table : nullptr;
            ws->walk.exact = plan.mode == 1 ? ws->bound.second : ws->bound.table;
            ws->walk.line = ws->bound.floor;
            ws->walk.ld = ws->bound.ld;
            for (int i = 0; i < 4; i++) ws->walk.share[i] = plan.share[i];
            return AP_OK;
        }
    }
    if (bounds) {
        AP_TRY(ap_bound_reserve(ix, ws->slab, 2048, AP_BOUND_WS_BYTES, marks ? AP_BOUND_MARKS : 1, st, &ws->bound));
        if (ws->bound.table) ws->slab = ws->bound.slab;
    }
    return AP_OK;
}

// LDS of a search's arrays.  k: of the secondary pool, with keywords.
static size_t ap_search_lds(int32_t L, bool kw, int32_t k, bool big_tables, int32_t nt, int32_t cmax, int32_t icap) {
    const bool pipe = !kw && !big_tables && nt >= 512;   // the large-pool path: entering keys in the candidates' space, a bitmap of the pool
    const int32_t nxtw = !pipe && cmax > nt ? cmax : 0;
    return (size_t)(L + (pipe ? 1 : 2) * cmax + nxtw + (kw ? cmax + k : 0)) * 8 + (size_t)cmax * 16 +
           (size_t)(big_tables ? ApQTab<true>::SLOTS : ApQTab<false>::SLOTS) * 8 + (pipe ? (size_t)((L + 63) / 64) * 8 : 0) + (pipe && icap ? 8 + (size_t)icap * 4 : 0);
}
// Workgroup size (plain search): four waves as long as the LDS holds at least five workgroups per CU; a pool
// that leaves room for two to four gets eight waves, one that fills the CU alone sixteen (measured: each is the
// fastest in its range).
static int32_t ap_search_threads(int32_t L, int32_t cmax) {
    const size_t per_cu = (size_t)160 * 1024 / ap_search_lds(L, false, 0, false, 256, cmax, 0);
    return per_cu > AP_SEARCH_NT512_AT ? 256 : per_cu > AP_SEARCH_NT1024_AT ? 512 : 1024;
}
// Whether a plain search may take a floor below which neighbours wait: where it ends by itself, in large pools.  In small ones (256 threads) what
// it keeps from being scored is little -- 590 instead of 730 documents at beam 128 -- and its code costs more.  A pool for (nearly) all documents has no floor.
static bool ap_search_waits(const ap_index *ix, int32_t beam, int32_t width, int32_t max_iters) {
    return max_iters == 0 && !ix->deleted && g_ap_debug.search_floor != 1 && ap_bound_floor_share(ix, beam) < 1.0 && ap_search_threads(beam, std::max(ix->params.n_entry, width * ix->params.degree)) >= 512;
}

// The launch itself.  Q: the queries (any view with f32 dense rows); w_dev / w_stride: device weights, one triple
// per query (stride 3) or one for all (stride 0).  kw_terms == NULL: the plain search; otherwise the
// keyword-constrained one.  The queries run in slabs of ws.slab, one launch each, that share the workspace.
// Nothing here allocates: the workspace comes from the caller.
static int ap_search_launch(const ap_index *ix, const ApSearchWs &ws, const ApVecs &Q, const float *w_dev, int32_t w_stride, int32_t k,
                            int32_t beam, int32_t max_iters, int32_t width, const int32_t *kw_terms, int32_t kw_stride,
                            uint32_t kw_flags, bool big_tables, int32_t *out_ids, float *out_scores, hipStream_t st) {
    // The keyword instantiation also serves plain searches on an index with mark-deleted documents (it carries the
    // answer filter; without required terms it searches exactly like the plain one), so that the plain
    // instantiation stays free of both.
    const bool kw = kw_terms != nullptr || ix->deleted != nullptr;
    const int32_t nq = (int32_t)Q.n;
    auto note_form = [&](int32_t threads, int32_t listed, int32_t vis_lds) {   // where the call may write to the index
        if (!ws.counts) return;
        ix->search_form[0] = threads; ix->search_form[1] = listed; ix->search_form[2] = vis_lds;
    };
    if (ws.walk.exact) {
        note_form(0, 0, 0);
        if (ws.ev0) AP_CHECK_HIP(hipEventRecord(ws.ev0, st));
        if (ws.walk.bound) AP_TRY(ap_bound_fill(ix, ws.bound, Q, w_dev, w_stride, 0, nq, nullptr, 0, st));
        AP_TRY(ap_walk_launch(ix, ws.walk, ws.visited, Q, w_dev, w_stride, k, beam, width, ws.counts, out_ids, out_scores, st));
        if (ws.ev1) AP_CHECK_HIP(hipEventRecord(ws.ev1, st));
        return AP_OK;
    }
    if (!kw_terms) kw_stride = 0;
    ApSearchArgs g;
    g.D = ix->docs;
    g.Q = Q;
    g.graph = ix->graph;
    g.entry = ix->entry;
    g.w = w_dev;
    g.w_stride = w_stride;
    g.R = ix->params.degree;
    g.E = ix->params.n_entry;
    g.k = k; g.L = beam; g.max_iters = max_iters; g.width = width;
    g.KR = kw_terms ? ix->params.degree / 2 : 0;
    g.kw_edges = ix->kw; g.kw_count = ix->kw_count; g.kw_terms = kw_terms; g.kw_stride = kw_stride;
    g.kw_all = (kw_flags & AP_KW_ALL) ? 1 : 0;
    g.kw_use_edges = (kw_flags & AP_KW_NO_EDGES) ? 0 : 1;
    g.cmax = g.E > g.width * (g.R + g.KR) ? g.E : g.width * (g.R + g.KR);
    g.words = ((size_t)ix->docs.n + 31) / 32;
    g.visited = ws.visited;
    g.out_ids = out_ids;
    g.out_scores = out_scores;
    g.counts = ws.counts;
    g.rec = ix->rec;
    g.meta = ix->meta;
    g.deleted = ix->deleted;
    g.bound = ws.bound.table;
    g.bound_ld = ws.bound.ld;
    g.bound_col = ix->bd_mem ? ix->bd_col + ix->corpus.sp_vocab : nullptr;
    g.bound_bits = ix->bd_bits;
    g.tx_vocab = ix->corpus.tx_vocab;
    auto lds_bytes = [&](int32_t nt, int32_t cmax, int32_t icap) { return ap_search_lds(beam, kw, kw ? k : 0, big_tables, nt, cmax, icap); };
    const int64_t at_once = std::min(ws.slab, nq);
    int32_t nt = 256;
    g.icap = 0;
    if (!kw && !big_tables) {
        nt = ap_search_threads(beam, g.cmax);
        // A pool that fills the CU alone because of the candidates beside it: their descriptors and keys take 28 bytes each, their ids 4,
        // and what gets past the bounds is a few dozen an iteration.  Listed and scored AP_SEARCH_LISTED at a time, two queries
        // of eight waves share the CU, and one reads while the other ranks and merges.  2,000 queries of 500,000 bf16 documents,
        // pool 8,192, sixteen parents: 79.6 -> 64.3 ms; 300 of 100,000 f32 13.8 -> 10.5, 1,500 43.6 -> 36.9.  (Pools of which three would fit then instead of two keep their candidates:
        // three take the registers of the second candidate in flight.)
        if (nt == 1024 && at_once > AP_CUS && ws.bound.table && g.cmax > AP_SEARCH_LISTED && 2 * (lds_bytes(512, AP_SEARCH_LISTED, g.cmax) + 640) <= (size_t)160 * 1024) {
            nt = 512;
            g.icap = g.cmax;
            g.cmax = AP_SEARCH_LISTED;   // at least the 256 entry points an index may have
        }
    }
    // Two waves a query, twice as many queries on the chip at a time: a query then takes some 1.2 times as long (its few candidates
    // an iteration keep four waves no busier than two, the steps between them wait for memory either way), so this pays where it saves
    // a second, half empty round.  2,500 queries (1,792 of four waves run at a time, 3,584 of two), pool 512: 100,000 f32 documents
    // with keywords 14.6 -> 10.9 ms, plain 9.32 -> 8.36; 60,000 bf16 10.6 -> 8.6 and 7.25 -> 6.32; 10,000 narrow ones 6.6 -> 4.5 and 4.3 -> 3.1.
    // Not where the batch fits one round of four waves (400 to 1,500 queries: 0.67 to 0.98 of the speed) nor without bounds or with
    // more candidates an iteration, where two waves have more to score than they hide (0.6 to 0.9; 128 candidates: 0.7).  With keywords 1.05 to 1.5
    // up to the 3,072 that run at once.  A plain search has less to hide behind, and that shows in three places (speeds by two waves, pools 48 to 1,400):
    //  - wide bf16 rows, of which five waves a SIMD run: 0.77 to 1.05 for 1,300 to 2,560 queries of 1,536 and 2,048 columns (1,280 and 2,560 run at a time);
    //    with keywords 0.85 to 1.15 up to 1,800, 1.03 to 1.22 from 2,100 on;
    //  - bf16 rows of 513 to 1,024 columns where only four waves have their visited sets in LDS: 0.90 to 1.03 (where both do or neither does 0.98 to 1.17);
    //  - other rows where only four waves do, towards two full rounds: rows of 768 f32 columns 1.02 to 1.14 up to 2,500 queries, 0.99 to 1.02 at 2,750 (1.53
    //    rounds), 0.96 to 1.0 at 3,000; 1,024 columns 1.03 to 1.05 at 2,750 and 1.0 to 1.02 at 3,000; shorter rows (128 and 384 f32, 512 bf16) 0.97 to 1.13 from
    //    2,250 to 3,300 queries (1.84 rounds), 0.96 to 1.04 at 3,550.
    // Beyond one round of two waves four are taken, though they are not always the faster: from 3,900 to 7,000 queries two would run plain searches at
    // 0.80 to 1.38 times the speed (f32 0.80 to 0.97, bf16 0.82 to 1.0, narrow rows 1.05 to 1.38) and those with keywords at 0.86 to 1.16 with a
    // pool of 32 and 1.01 to 1.34 with pools of 128 and 512.
    const int32_t slots_of = ix->dtype == AP_BF16 && ix->docs.dim > 1024 ? 5 : AP_SEARCH_WAVES_PER_SIMD;   // waves a SIMD holds (ApSearchWaves)
    auto slots = [&](int32_t threads, size_t bytes) -> int64_t {
        const int32_t waves = threads == 128 && kw ? std::min(slots_of, AP_SEARCH_WAVES_KW2) : slots_of;
        // LDS is handed out in 128 blocks of 1,280 bytes a CU.  (By bytes alone 2,500 queries of 50,000 documents, pool 512, were taken to run
        // at once with their visited sets in LDS: 10 workgroups of 15,592 bytes a CU, where 9 do.  8.90 ms before, 9.71 with them, 7.54 now.)
        return AP_CUS * (int64_t)std::min<size_t>((size_t)waves * 256 / threads, AP_LDS_BLOCKS / ((bytes + AP_SEARCH_STATIC + AP_LDS_BLOCK - 1) / AP_LDS_BLOCK));
    };
    // Visited sets in LDS (small workgroups only).  Four waves: when the bitset fits beside the kernel's other arrays without
    // taking a workgroup's place on the CU (seven of them run on one while the pool is small).  Measured on 100,000
    // documents (12.5 KB a set): 4 to 5 % faster up to beam 512, 29 % slower at beam 2144 where it costs two of the
    // seven workgroups, which is why the rule is about occupancy.  Two waves: as long as the whole batch runs at once.  Same results either way.
    auto visited_fit = [&](int32_t threads) {
        if (threads > 256 || g_ap_debug.search_visited_global != 0) return false;
        const size_t without = lds_bytes(threads, g.cmax, 0), with = without + g.words * 4 + 8, lds = (size_t)160 * 1024;
        if (with > lds) return false;
        if (threads == 128) return slots(128, with) >= at_once;
        return lds / with >= std::min<size_t>(7, lds / without);
    };
    if (nt == 256 && !big_tables && ws.bound.table && g.cmax <= 96) {
        const int64_t four = slots(256, lds_bytes(256, g.cmax, 0));
        const bool bf16 = ix->dtype == AP_BF16;
        int32_t least = 11, most = 20;   // tenths of a round of four waves
        if (bf16 && ix->docs.dim > 1024) { least = 15; most = kw ? 20 : 0; }
        else if (!kw && !visited_fit(128) && visited_fit(256)) most = bf16 && ix->docs.dim > 512 ? 0 : !bf16 && ix->docs.dim > 512 ? 16 : 19;
        if (at_once * 10 > four * least && at_once * 10 <= four * most && at_once <= slots(128, lds_bytes(128, g.cmax, 0))) nt = 128;
    }
    g.bound_floor = ws.bound.table && ws.bound.marks ? reinterpret_cast<const float4 *>(ws.bound.floor) : nullptr;   // the caller asked for marks: ap_search_waits
    g.marks = ws.bound.marks;
    g.nxtw = nt <= 256 && g.cmax > nt ? g.cmax : 0;
    g.vis_lds = visited_fit(nt) ? 1 : 0;
    const size_t smem = lds_bytes(nt, g.cmax, g.icap) + (g.vis_lds ? g.words * 4 + 8 : 0);
    // the kernel's static arrays (counters, parents, required terms) take a few hundred bytes more
    AP_REQUIRE(smem + 512 <= 160 * 1024, "beam and search_width need %zu bytes of LDS (limit 160 KiB)", smem + 512);
    note_form(nt, g.icap > 0, g.vis_lds);
    const size_t dyn = smem - (size_t)(big_tables ? ApQTab<true>::SLOTS : ApQTab<false>::SLOTS) * 8;   // the tables are a static array
    hipError_t le = hipSuccess;
#define AP_LAUNCH_SEARCH(KWF, BIGF, NTF, ...)                                                                                         \
    AP_DISPATCH_DENSE(ix->dtype, ix->docs.dim, {                                                                                  \
        if (smem > 48 * 1024)                                                                                                     \
            le = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_search<DT, NV, KWF, BIGF, NTF, __VA_ARGS__>),                           \
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)dyn);                                       \
        if (le == hipSuccess) hipLaunchKernelGGL((k_search<DT, NV, KWF, BIGF, NTF, __VA_ARGS__>), dim3((unsigned)qn), dim3(NTF), dyn, st, g);  \
    })
    for (int32_t q0 = 0; q0 < nq; q0 += ws.slab) {
        const int32_t qn = std::min(ws.slab, nq - q0);
        g.q0 = q0;
        g.no_tables = g_ap_debug.search_query_lists != 0;
        // every slab starts from empty visited sets (a fill kernel, not a memset: callers may capture the stream)
        if (!g.vis_lds && !g.bound_floor) AP_TRY(ap_fill_u32(ws.visited, g.words * (size_t)qn, 0u, st));
        if (q0 == 0 && ws.ev0) AP_CHECK_HIP(hipEventRecord(ws.ev0, st));
        if (ws.bound.table) {
            AP_TRY(ap_bound_fill(ix, ws.bound, Q, w_dev, w_stride, q0, qn, kw_terms, kw_stride, st));
            if (g.bound_floor) AP_TRY(ap_bound_floors(ix, ws.bound, qn, beam, st));
        }
        if (kw && nt == 128) AP_LAUNCH_SEARCH(true, false, 128, false);
        else if (kw) AP_LAUNCH_SEARCH(true, false, 256, false);
        else if (big_tables) AP_LAUNCH_SEARCH(false, true, 256, false);
        else if (nt == 128) AP_LAUNCH_SEARCH(false, false, 128, false);
        else if (nt == 256) AP_LAUNCH_SEARCH(false, false, 256, false);
        else if (g.icap && g.bound_floor) AP_LAUNCH_SEARCH(false, false, 512, true, true);
        else if (g.icap) AP_LAUNCH_SEARCH(false, false, 512, false, true);
        else if (nt == 512 && g.bound_floor) AP_LAUNCH_SEARCH(false, false, 512, true);
        else if (nt == 512) AP_LAUNCH_SEARCH(false, false, 512, false);
        else if (g.bound_floor) AP_LAUNCH_SEARCH(false, false, 1024, true);
        else AP_LAUNCH_SEARCH(false, false, 1024, false);
        AP_CHECK_HIP(le);
        AP_CHECK_HIP(hipGetLastError());
    }
#undef AP_LAUNCH_SEARCH
    if (ws.ev1) AP_CHECK_HIP(hipEventRecord(ws.ev1, st));
    return AP_OK;
}

// Argument checks shared by every entry into the search.
static int ap_search_check(const ap_index *ix, int32_t nq, int32_t k, int32_t beam, int32_t max_iters, int32_t width, bool kw,
                           const int32_t *out_ids, const float *out_scores) {
    if (!ix->has_graph) { ap_set_error("index has no graph: build or import one first"); return AP_ESTATE; }
    AP_REQUIRE(nq == 0 || (out_ids && out_scores), "NULL output");
    AP_REQUIRE(beam >= 1 && beam <= AP_MAX_BEAM, "beam = %d must be in [1, %d]", beam, AP_MAX_BEAM);
    AP_REQUIRE(k >= 1 && k <= beam, "k = %d must be in [1, beam]", k);
    AP_REQUIRE(width >= 1 && width <= 16, "search_width = %d must be in [1, 16]", width);
    AP_REQUIRE(max_iters >= 0, "max_iters must be >= 0");
    AP_REQUIRE(!(kw || ix->deleted) || ix->docs.n < (1ll << 29), "keyword search and searches on an index with deletions need n < 2^29");
    return AP_OK;
}

int ap_search_core(ap_index *ix, const ApVecs &Q, const float *w_dev, int32_t w_stride, int32_t k, int32_t beam, int32_t max_iters,
                   int32_t width, bool big_tables, int32_t *out_ids, float *out_scores, hipStream_t st) {
    AP_TRY(ap_search_check(ix, (int32_t)Q.n, k, beam, max_iters, width, false, out_ids, out_scores));
    if (Q.n == 0) return AP_OK;
    ApSearchWs ws;
    AP_TRY(ap_search_reserve(ix, (int32_t)Q.n, st, &ws, ap_bound_pays(ix, Q.n, beam, width, max_iters)));
    return ap_search_launch(ix, ws, Q, w_dev, w_stride, k, beam, max_iters, width, nullptr, 0, 0u, big_tables, out_ids, out_scores, st);
}

static int ap_search_impl(ap_index *ix, const ap_queries *q, const float *per_query_w, const ap_search_params *p,
                          const int32_t *kw_terms, int32_t kw_stride, uint32_t kw_flags, int32_t *out_ids, float *out_scores,
                          void *stream) {
    AP_REQUIRE(ix && p, "NULL argument");
    AP_TRY(ap_validate_queries(q));
    AP_TRY(ap_search_check(ix, q->nq, p->k, p->beam, p->max_iters, p->search_width, kw_terms != nullptr, out_ids, out_scores));
    if (q->nq == 0) return AP_OK;
    const ApVecs Q{q->nq, ix->docs.dim, q->dense, q->sp_indptr, q->sp_idx, q->sp_val, q->tx_indptr, q->tx_idx, q->tx_cnt};
    ApSearchWs ws;
    const bool bounds = ap_bound_pays(ix, q->nq, p->beam, p->search_width, p->max_iters, kw_terms && !(kw_flags & AP_KW_NO_EDGES));
    const ApWalkPlan plan = kw_terms ? ApWalkPlan() : ap_walk_plan(ix, q->nq, p->beam, p->search_width, p->max_iters, bounds, true);
    AP_TRY(ap_search_reserve(ix, q->nq, (hipStream_t)stream, &ws, bounds, plan, !kw_terms && ap_search_waits(ix, p->beam, p->search_width, p->max_iters)));
    return ap_search_launch(ix, ws, Q, per_query_w ? per_query_w : ix->w_dev, per_query_w ? 3 : 0, p->k, p->beam, p->max_iters,
                            p->search_width, kw_terms, kw_stride, kw_flags, false, out_ids, out_scores, (hipStream_t)stream);
}

extern "C" int ap_search_batch(ap_index *ix, const ap_queries *q, const float *per_query_w,
                               const ap_search_params *p, int32_t *out_ids, float *out_scores, void *stream) {
    return ap_search_impl(ix, q, per_query_w, p, nullptr, 0, 0u, out_ids, out_scores, stream);
}

// ---- the search for callers that cannot allocate ---------------------------------------------------------------
// The visited sets live in a file-scope device array instead of an index-owned allocation.  Each GPU holds its own
// copy of the array at its own address; host code uses the address hipGetSymbolAddress returns for the current
// device, never the array's name (which is only a host-side stand-in).
static __device__ __align__(256) unsigned char scratch[AP_NOALLOC_WORKSPACE_BYTES];

#define AP_MAX_DEVICES 64
static std::mutex g_scratch_lock;
static void *g_scratch_ptr[AP_MAX_DEVICES];   // per device, filled on first use

// The address of `scratch` on the current device (looked up once per device).
int ap_static_scratch(void **out) {
    int dev = -1;
    AP_CHECK_HIP(hipGetDevice(&dev));
    AP_REQUIRE(dev >= 0 && dev < AP_MAX_DEVICES, "device %d is beyond the %d devices this library keeps a workspace for", dev, AP_MAX_DEVICES);
    std::lock_guard<std::mutex> hold(g_scratch_lock);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        AP_CHECK_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        AP_REQUIRE(p != nullptr, "the static search workspace has no address on device %d", dev);
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return AP_OK;
}

extern "C" int ap_search_batch_noalloc(const ap_index *ix, const ap_queries *q, const float *per_query_w,
                                       const ap_search_params *p, int32_t *out_ids, float *out_scores, void *stream) {
    AP_REQUIRE(ix && p, "NULL argument");
    AP_TRY(ap_validate_queries(q));
    AP_TRY(ap_search_check(ix, q->nq, p->k, p->beam, p->max_iters, p->search_width, false, out_ids, out_scores));
    const size_t words = ((size_t)ix->docs.n + 31) / 32;
    // the debug setting that caps the index-owned workspace caps this one too (never beyond the array)
    const size_t cap = g_ap_debug.search_workspace_bytes > 0 ? std::min<size_t>((size_t)g_ap_debug.search_workspace_bytes, AP_NOALLOC_WORKSPACE_BYTES)
                                                             : AP_NOALLOC_WORKSPACE_BYTES;
    AP_REQUIRE(words * 4 <= cap,
               "the corpus has %lld documents: one visited bit per document does not fit the static workspace of %zu bytes "
               "(at most %zu documents); use ap_search_batch",
               (long long)ix->docs.n, cap, cap * 8);
    if (q->nq == 0) return AP_OK;
    void *base = nullptr;
    AP_TRY(ap_static_scratch(&base));
    ApSearchWs ws;                       // no counters, no events: nothing of the index is written
    ws.visited = static_cast<uint32_t *>(base);
    ws.slab = ap_slab_size(q->nq, words, cap / 4);
    // a small batch by the walk, with every document scored ahead, where the scores fit the array beside the visited sets
    const ApWalkPlan plan = ap_walk_plan(ix, q->nq, p->beam, p->search_width, p->max_iters, false, false);
    const size_t ld = ((size_t)ix->docs.n + 63) / 64 * 64, at = (words * (size_t)q->nq + 63) / 64 * 64;
    if (plan.mode == 2 && (at + (ld + 5) * (size_t)q->nq) * 4 <= cap) {
        ws.walk.exact = static_cast<float *>(base) + at;
        ws.walk.line = ws.walk.exact + ld * (size_t)q->nq;
        ws.walk.ld = (int64_t)ld;
        for (int i = 0; i < 4; i++) ws.walk.share[i] = plan.share[i];
    }
    const ApVecs Q{q->nq, ix->docs.dim, q->dense, q->sp_indptr, q->sp_idx, q->sp_val, q->tx_indptr, q->tx_idx, q->tx_cnt};
    return ap_search_launch(ix, ws, Q, per_query_w ? per_query_w : ix->w_dev, per_query_w ? 3 : 0, p->k, p->beam, p->max_iters,
                            p->search_width, nullptr, 0, 0u, false, out_ids, out_scores, (hipStream_t)stream);
}

extern "C" int ap_search_batch_keywords(ap_index *ix, const ap_queries *q, const float *per_query_w,
                                        const ap_search_params *p, const int32_t *kw_terms, int32_t kw_stride,
                                        uint32_t kw_flags, int32_t *out_ids, float *out_scores, void *stream) {
    AP_REQUIRE(ix && q, "NULL argument");
    AP_REQUIRE(kw_stride >= 1 && kw_stride <= AP_KW_MAX_TERMS, "kw_stride = %d must be in [1, %d]", kw_stride, AP_KW_MAX_TERMS);
    AP_REQUIRE(kw_terms || q->nq == 0, "kw_terms is NULL");
    AP_REQUIRE((kw_flags & ~(uint32_t)(AP_KW_ALL | AP_KW_NO_EDGES)) == 0, "unknown bits in kw_flags");
    if (!ix->has_graph) { ap_set_error("index has no graph: build or import one first"); return AP_ESTATE; }
    AP_REQUIRE(ix->kw && ix->kw_count, "index has no keyword edges");
    AP_REQUIRE(ix->docs.n < (1ll << 29), "keyword search needs n < 2^29");
    if (q->nq == 0) return ap_search_impl(ix, q, per_query_w, p, nullptr, 0, 0u, out_ids, out_scores, stream);
    return ap_search_impl(ix, q, per_query_w, p, kw_terms, kw_stride, kw_flags, out_ids, out_scores, stream);
}

extern "C" int ap_search_form(const ap_index *ix, int32_t out3[3]) {
    AP_REQUIRE(ix && out3, "NULL argument");
    if (ix->last_nq == 0) { ap_set_error("no search has run on this index"); return AP_ESTATE; }
    memcpy(out3, ix->search_form, sizeof(ix->search_form));
    return AP_OK;
}

extern "C" int ap_search_stats(const ap_index *ix, int32_t *out_counts, int32_t nq, float *kernel_ms, void *stream) {
    AP_REQUIRE(ix, "index is NULL");
    if (!ix->ev_search[1] || ix->last_nq == 0) { ap_set_error("no search has run on this index"); return AP_ESTATE; }
    AP_CHECK_HIP(hipEventSynchronize(ix->ev_search[1]));
    if (kernel_ms) AP_CHECK_HIP(hipEventElapsedTime(kernel_ms, ix->ev_search[0], ix->ev_search[1]));
    if (out_counts) {
        AP_REQUIRE(nq == ix->last_nq, "nq = %d does not match the last search (%d)", nq, ix->last_nq);
        AP_CHECK_HIP(hipMemcpyAsync(out_counts, ix->search_counts, (size_t)nq * 3 * sizeof(int32_t), hipMemcpyDeviceToDevice,
                                    (hipStream_t)stream));
    }
    return AP_OK;
}
