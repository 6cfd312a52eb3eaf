// The search for batches too small to fill the chip (Algorithm 2, as k_search runs it, with the same results).
//
// Such a batch is bound by the chain of its iterations: in k_search each is a gather (edge, visited bit, bound,
// descriptor: one round trip to memory after the other), a list of documents to score (another two) and half a dozen
// barriers, 5.5 us together, while most of the chip idles.  Here
//  - the scores come first: k_walk_score lets the whole chip score the documents that the search may want, those whose
//    upper bound reaches a quantile of the query's bounds (or, of a small corpus, all of them), and leaves the scores in
//    a row of floats per query;
//  - one wave walks the graph (k_walk), 1.05 to 1.25 us an iteration: a round trip for the parent's edges, unless it was foreseen
//    (every other one is), one for its neighbours' scores, and LDS for the rest; nothing in the loop waits for another wave.
// A score is computed by the code that k_search runs, so the results have the same bits.
#include <math.h>
#include <algorithm>
#include <type_traits>
#include "ap_score.hpp"

#define AP_WALK_LIST_NT 256      // threads of the walk with lists: one wave walks
#define AP_WALK_NT 1024          // threads of the one with a sorted pool: the others step in to score
#define AP_WALK_SCORE_NT 512
#define AP_WALK_LIST 1024        // candidates a block of k_walk_score gathers before it scores them
#define AP_WALK_SAMPLE 1024      // bounds the quantiles are taken from
#define AP_WALK_LEVELS 4
#define AP_WALK_GOOD 3           // documents above the first line that the way into the graph has to lead to
#define AP_WALK_STEPS 6          // steps it is followed for that

typedef uint32_t ap_u32x4_w __attribute__((ext_vector_type(4)));

struct ApWalkArgs {
    ApVecs D, Q;
    const int32_t *graph, *entry;
    const float *w;
    int32_t w_stride, no_tables;
    int32_t R, E, k, L, width, cmax, vis_lds, warm;
    int32_t vis_at;             // where in the dynamic LDS the visited set lies (8-byte words)
    uint32_t *visited;          // per query `words` words, where the sets do not live in LDS
    size_t words;
    int32_t *out_ids;
    float *out_scores;
    int32_t *counts;
    const uint2 *rec;
    const uint4 *meta;
    const uint32_t *deleted;
    uint32_t *bound;            // upper bounds, bit 0 set where `exact` holds the score (NULL: it holds all of them)
    float *exact;
    int64_t ld;                 // of both, per query
    const float *line;          // per query AP_WALK_LEVELS lines: documents with bounds from the first on are scored ahead
    int32_t *undecided;         // per query: 1 where the walk with lists did not decide it
    int32_t cap, done_cap;      // entries of a lane's list, of the list of expanded documents
    int64_t per_block;          // documents a block of k_walk_score looks at
};

// The query's tables and dense slice, as k_search sets them up; all threads of the workgroup take part.
template <int DT, int NV> struct ApWalkQuery {
    ApLists a;
    bool use_tab;
    uint32_t msp, mtx;
    float qa[NV * ApDense<DT>::EPC], qnorm, wd, ws, wf;
    __device__ __forceinline__ void load(const ApWalkArgs &g, int64_t q, uint64_t *qtab, int32_t *s_seed) {
        constexpr int SPB = ApQTab<false>::SPB, TXB = ApQTab<false>::TXB;
        const int64_t sb = g.Q.sp_indptr[q], tb = g.Q.tx_indptr[q];
        a.sp_n = (int32_t)(g.Q.sp_indptr[q + 1] - sb); a.tx_n = (int32_t)(g.Q.tx_indptr[q + 1] - tb);
        a.sp_idx = g.Q.sp_idx + sb; a.sp_val = g.Q.sp_val + sb; a.tx_idx = g.Q.tx_idx + tb; a.tx_val = g.Q.tx_val + tb;
        use_tab = !g.no_tables && a.sp_n <= (1 << SPB) / 4 && a.tx_n <= (1 << TXB) / 4;   // uniform
        msp = mtx = 0;
        if (use_tab && ap_wave_id() == 0) {
            const int32_t s0 = ap_bucket_build<1>(a.sp_idx, a.sp_val, a.sp_n, qtab, SPB);
            const int32_t s1 = ap_bucket_build<1>(a.tx_idx, a.tx_val, a.tx_n, qtab + (1 << SPB), TXB);
            if ((threadIdx.x & 63) == 0) { s_seed[0] = s0; s_seed[1] = s1; }
        }
        __syncthreads();
        if (use_tab) {
            const int32_t seed0 = ap_uniform_i32(s_seed[0]), seed1 = ap_uniform_i32(s_seed[1]);
            use_tab = seed0 >= 0 && seed1 >= 0;
            if (use_tab) { msp = ap_seed_mult(seed0); mtx = ap_seed_mult(seed1); }
        }
        ap_load_aside<DT, NV, AP_F32>(g.Q.dense, q, g.D.dim, qa);
        float p = 0.f;
#pragma unroll
        for (int i = 0; i < NV * ApDense<DT>::EPC; i++) p = fmaf(qa[i], qa[i], p);
        qnorm = sqrtf(ap_wave_sum(p));
        wd = g.w[q * g.w_stride + 0]; ws = g.w[q * g.w_stride + 1]; wf = g.w[q * g.w_stride + 2];
    }
    // scores the c documents of s_meta into newk (ap_score_candidates)
    template <int NW, int G, int W0 = 0>
    __device__ __forceinline__ int32_t score(const ApWalkArgs &g, const uint64_t *qtab, const uint4 *s_meta, int32_t c, uint64_t *newk, bool pool_full,
                                             float worst_score, bool pre) const {
        if (use_tab)
            return ap_score_candidates<DT, NV, true, false, false, NW, G, W0>(g.D, g.rec, qa, qtab, a, wd, ws, wf, qnorm, pool_full, worst_score, s_meta, c, newk,
                                                                          nullptr, 0, false, false, 0.f, msp, mtx, pre);
        return ap_score_candidates<DT, NV, false, false, false, NW, G, W0>(g.D, g.rec, qa, qtab, a, wd, ws, wf, qnorm, pool_full, worst_score, s_meta, c, newk,
                                                                       nullptr, 0, false, false, 0.f, 0u, 0u, pre);
    }
};

// Largest value of the wave, in every lane: by its upper halves first, by the lower ones where those agree.
__device__ __forceinline__ uint32_t ap_wave_max_u32(uint32_t v) {
    auto step = [](uint32_t a, uint32_t b) { return a > b ? a : b; };
    v = step(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xf, 0xf, true));
    v = step(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xf, 0xf, true));
    v = step(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xf, 0xf, true));
    v = step(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xf, 0xf, true));
    const uint32_t r0 = (uint32_t)__builtin_amdgcn_readlane((int)v, 0), r1 = (uint32_t)__builtin_amdgcn_readlane((int)v, 16),
                   r2 = (uint32_t)__builtin_amdgcn_readlane((int)v, 32), r3 = (uint32_t)__builtin_amdgcn_readlane((int)v, 48);
    return step(step(r0, r1), step(r2, r3));
}
__device__ __forceinline__ uint64_t ap_wave_max_u64(uint64_t v) {
    const uint32_t hi = ap_wave_max_u32((uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | ap_wave_max_u32((uint32_t)(v >> 32) == hi ? (uint32_t)v : 0u);
}

// One block per query: the values (bounds, or scores) that four falling shares of the documents reach, from a sample of at
// most AP_WALK_SAMPLE of them (64 runs of 16 spread over the corpus).
__global__ __launch_bounds__(512) void k_walk_lines(const uint32_t *__restrict__ table, int64_t ld, int64_t n, float4 shares, float *__restrict__ line) {
    __shared__ uint32_t keys[AP_WALK_SAMPLE];
    const uint32_t *row = table + (int64_t)blockIdx.x * ld;
    const int32_t m = n < AP_WALK_SAMPLE ? (int32_t)n : AP_WALK_SAMPLE;
    for (int32_t i = threadIdx.x; i < AP_WALK_SAMPLE; i += 512) {
        const int64_t d = n <= AP_WALK_SAMPLE ? i : (int64_t)(i >> 4) * ((n - 16) / 63) + (i & 15);
        keys[i] = i < m ? ap_f2ord(__uint_as_float(row[d])) : 0u;
    }
    for (int32_t size = 2; size <= AP_WALK_SAMPLE; size <<= 1)
        for (int32_t stride = size >> 1; stride > 0; stride >>= 1) {
            // pairs closer than 64 keys lie inside one wave's 128 keys
            if (stride >= 64 || stride == size >> 1) __syncthreads(); else ap_wave_sync();
            const int32_t t = threadIdx.x, lo = 2 * t - (t & (stride - 1)), hi = lo + stride;
            const uint32_t x = keys[lo], y = keys[hi];
            if ((x < y) == ((lo & size) == 0)) { keys[lo] = y; keys[hi] = x; }
        }
    __syncthreads();
    if (threadIdx.x < AP_WALK_LEVELS) {
        const float share = threadIdx.x == 0 ? shares.x : threadIdx.x == 1 ? shares.y : threadIdx.x == 2 ? shares.z : shares.w;
        const int32_t at = (int32_t)(share * (float)m);
        line[blockIdx.x * (int64_t)AP_WALK_LEVELS + threadIdx.x] = at < m ? ap_ord2f(keys[at]) : -INFINITY;
    }
}

// blockIdx.y = query, blockIdx.x = a run of per_block documents: those whose bound is not below the query's first line (all of
// them where there are no bounds) are gathered and scored, eight waves a candidate each.  With bounds a last block follows
// the search's way into the graph, scoring all it meets, until a few documents above the line wait to be followed: entry
// points and their neighbours are no better than any documents, and where none of them is above the line the walk would not
// get started (one query in 200 with 64 and 64 of them and a line at 5 %).
template <int DT, int NV, bool ALL>
__global__ __launch_bounds__(AP_WALK_SCORE_NT) void k_walk_score(ApWalkArgs g) {
    __shared__ __attribute__((aligned(16))) uint64_t qtab[ApQTab<false>::SLOTS];
    __shared__ __attribute__((aligned(16))) uint4 s_meta[AP_WALK_LIST];
    __shared__ uint64_t newk[AP_WALK_LIST];
    __shared__ int32_t s_seed[2], s_cnt;
    const int64_t q = blockIdx.y, d0 = (int64_t)blockIdx.x * g.per_block, d1 = d0 + g.per_block < g.D.n ? d0 + g.per_block : g.D.n;
    if (threadIdx.x == 0) s_cnt = 0;
    ApWalkQuery<DT, NV> Q;
    Q.load(g, q, qtab, s_seed);
    uint32_t *bound = ALL ? nullptr : g.bound + q * g.ld;
    float *exact = g.exact + q * g.ld;
    const float line = ALL ? 0.f : g.line[q * AP_WALK_LEVELS];
    __syncthreads();
    // the c candidates of the list: their scores, noted
    auto score = [&](int32_t c) {
        (void)Q.template score<AP_WALK_SCORE_NT / 64, 2>(g, qtab, s_meta, c, newk, false, 0.f, true);
        __syncthreads();
        if (threadIdx.x == 0) s_cnt = 0;
        for (int32_t i = threadIdx.x; i < c; i += AP_WALK_SCORE_NT) {
            const int32_t at = ap_key_id(newk[i]);
            exact[at] = ap_key_score(newk[i]);
            if (!ALL) bound[at] |= 1u;
        }
    };
    if constexpr (!ALL) {
        if (blockIdx.x == gridDim.x - 1) {   // uniform
            __shared__ uint64_t pool[AP_WALK_LIST], red[AP_WALK_SCORE_NT / 64];   // what was scored here and not followed yet
            __shared__ int32_t s_pool, s_good[AP_WALK_STEPS + 1];
            if (threadIdx.x == 0) s_pool = 0;
            if (threadIdx.x <= AP_WALK_STEPS) s_good[threadIdx.x] = 0;
            __syncthreads();
            int64_t parent = -1, before = -1;
            for (int32_t step = 0; step <= AP_WALK_STEPS; step++) {
                const int32_t total = step == 0 ? g.E : g.R;
                for (int32_t i0 = 0; i0 < total; i0 += AP_WALK_SCORE_NT) {
                    // some are scored by another block as well, to the same bits
                    const int32_t i = i0 + (int32_t)threadIdx.x, v = i < total ? (step == 0 ? g.entry[i] : g.graph[parent * g.R + i]) : -1;
                    if (v >= 0 && v != before) {
                        const uint4 m = g.meta[v];
                        s_meta[atomicAdd(&s_cnt, 1)] = make_uint4(m.x, m.y, m.z, (uint32_t)v);
                    }
                    __syncthreads();
                    const int32_t c = ap_uniform_i32(s_cnt);
                    score(c);
                    for (int32_t j = threadIdx.x; j < c; j += AP_WALK_SCORE_NT) {
                        const int32_t at = atomicAdd(&s_pool, 1);
                        if (at < AP_WALK_LIST) pool[at] = newk[j];
                    }
                    __syncthreads();
                }
                const int32_t m = s_pool < AP_WALK_LIST ? s_pool : AP_WALK_LIST;
                uint64_t best = 0ull;
                for (int32_t j = threadIdx.x; j < m; j += AP_WALK_SCORE_NT) {
                    best = pool[j] > best ? pool[j] : best;
                    if (pool[j] != 0ull && ap_key_score(pool[j]) >= line) atomicAdd(&s_good[step], 1);
                }
                best = ap_wave_max_u64(best);
                if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = best;
                __syncthreads();
                for (int j = 0; j < AP_WALK_SCORE_NT / 64; j++) best = red[j] > best ? red[j] : best;
                if (s_good[step] > AP_WALK_GOOD || best == 0ull) return;   // uniform
                for (int32_t j = threadIdx.x; j < m; j += AP_WALK_SCORE_NT)
                    if (pool[j] == best) pool[j] = 0ull;
                before = parent;
                parent = ap_key_id(best);
                __syncthreads();
            }
            return;
        }
    }
    for (int64_t d = d0; d < d1; d += AP_WALK_SCORE_NT) {   // uniform
        const int64_t v = d + threadIdx.x;
        if (v < d1 && (ALL || !(__uint_as_float(bound[v] & ~AP_BOUND_COUNT) < line))) {
            const uint4 m = g.meta[v];
            s_meta[atomicAdd(&s_cnt, 1)] = make_uint4(m.x, m.y, m.z, (uint32_t)v);
        }
        __syncthreads();
        const int32_t c = ap_uniform_i32(s_cnt);
        if (c > AP_WALK_LIST - AP_WALK_SCORE_NT || d + AP_WALK_SCORE_NT >= d1) {
            score(c);
        }
        __syncthreads();
    }
}

// What the walking wave and the scoring waves share, and the arrays in LDS.
struct ApWalkLds {
    uint4 *meta;          // candidates to score
    uint64_t *newk, *cur; // their keys; the pool
    uint64_t *list, *done; // the lanes' lists; the expanded documents
    int32_t *c, *full, *par;
    float *worst;
};
// All waves of the workgroup meet; what any wrote before is seen by all afterwards.
__device__ __forceinline__ void ap_walk_meet() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// The walk of one wave with lists: what the documents met ahead of it hold, and no more.  Everything scored ahead that may
// still matter goes into the list of the lane that met it, the best of a list in a register, so that an entering document
// costs a store wherever it ranks and the next parent is a maximum over the wave.  Nothing is ever taken out but parents:
//  - documents whose bound lies below the first line were not scored (entry points aside) and wait: while every parent scores
//    at least the line, none of them can rank before it.  Once the search has met as many documents above a line as the pool
//    holds, nothing below that line can be in the pool any more (`cut`);
//  - the best unexpanded document ranks behind expanded ones only, so it is in the pool as long as fewer of those than the pool
//    holds rank before it: when it is not, all of the pool has been expanded, and the search is over.
// Returns false where that does not decide the search: a parent below the line, or a pool not full down to it, while documents
// wait; a score that is a NaN, a list that is full.  ONE: one parent an iteration, at most 64 neighbours, visited set in LDS:
// the edges of the next parent are requested as soon as it is known, those of the one after it ahead of time.
template <bool ALL, bool ONE>
__device__ __forceinline__ bool ap_walk_lists(const ApWalkArgs &g, int64_t q, const ApVisited &vis, const ApWalkLds &l, int32_t &n_done) {
    const int lane = threadIdx.x & 63;
    const uint32_t *bound = ALL ? nullptr : g.bound + q * g.ld;
    const float *exact = g.exact + q * g.ld;
    const int32_t stride = g.cap + 1;   // odd: the lanes' stores fall in distinct banks
    uint64_t *const mine = l.list + lane * stride;
    const float *line = g.line + q * AP_WALK_LEVELS;
    const float t0 = line[0], t1 = line[1], t2 = line[2], t3 = line[3];
    float cut = -INFINITY;
    int32_t c0 = 0, c1 = 0, c2 = 0, c3 = 0;     // documents met at or above the lines
    int32_t it = 0, nscored = 0, nwait = 0, n = 0;
    bool bad = false;
    // per lane
    uint64_t head = 0ull;   // the best unexpanded document of the list, 0: none
    int32_t held = 0;       // entries of the list besides
    auto fresh = [&](int32_t v) -> bool {   // marks document v, tells whether it had not been marked before
        if constexpr (ONE) {                // no branch that a load on its way would have to be waited for at
            const uint32_t bit = 1u << (v & 31);
            return (__hip_atomic_fetch_or(vis.l + (v >> 5), bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) & bit) == 0u;
        } else return !vis.test_and_set(v);
    };
    auto fetch = [&](int32_t v, uint32_t &e, float &x) {
        const int32_t at = v < 0 ? 0 : v;
        if constexpr (!ALL) e = bound[at];
        x = exact[at];
    };
    auto take = [&](int32_t v, bool on, uint32_t e, float x) {
        const bool known = on && (ALL || (e & 1u));
        const bool has = known && x >= cut;
        const int32_t m = (int32_t)__popcll(__ballot(on));
        nscored += m;
        if constexpr (!ALL) nwait += m - (int32_t)__popcll(__ballot(known));
        if (c3 < g.L) {   // uniform
            c0 += (int32_t)__popcll(__ballot(known && x >= t0));
            c1 += (int32_t)__popcll(__ballot(known && x >= t1));
            c2 += (int32_t)__popcll(__ballot(known && x >= t2));
            c3 += (int32_t)__popcll(__ballot(known && x >= t3));
            cut = c3 >= g.L ? t3 : c2 >= g.L ? t2 : c1 >= g.L ? t1 : c0 >= g.L ? t0 : -INFINITY;
        }
        bool lost = known && !(x == x);
        if (has) {
            const uint64_t key = ap_make_key(x, v, 1u);
            const uint64_t low = key < head ? key : head;
            head = key < head ? head : key;
            if (low) {
                if (held < g.cap) mine[held++] = low;
                else lost = true;
            }
        }
        bad = bad || __ballot(lost) != 0ull;
    };
    // the best head, and takes it out
    auto best = [&](int32_t &owner) -> uint64_t {
        const uint32_t top = ap_wave_max_u32((uint32_t)(head >> 32));
        const uint64_t same = __ballot((uint32_t)(head >> 32) == top);
        owner = (int32_t)__builtin_ctzll(same);
        if ((same & (same - 1ull)) == 0ull)
            return ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int32_t)top) << 32) | (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int32_t)(uint32_t)head, owner);
        const uint64_t key = ap_uniform_u64(ap_wave_max_u64(head));
        owner = (int32_t)__builtin_ctzll(__ballot(head == key));
        return key;
    };
    auto refill = [&](int32_t owner) {
        const int32_t m = __builtin_amdgcn_readlane(held, owner);
        uint64_t *from = l.list + owner * stride;
        uint64_t top = 0ull;
        ap_wave_sync();
        if (m <= 64) {   // uniform
            const uint64_t k = lane < m ? from[lane] : 0ull;
            const uint32_t hi = ap_wave_max_u32((uint32_t)(k >> 32));
            uint64_t same = __ballot((uint32_t)(k >> 32) == hi);
            if (same & (same - 1ull)) same = __ballot(k == ap_wave_max_u64(k));
            const int32_t at = (int32_t)__builtin_ctzll(same);
            auto key_at = [&](int32_t j) -> uint64_t {
                return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int32_t)(k >> 32), j) << 32) | (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int32_t)(uint32_t)k, j);
            };
            top = key_at(at);
            const uint64_t last = key_at(m > 0 ? m - 1 : 0);
            if (lane == at && at < m) from[at] = last;
        } else {
            uint64_t key = 0ull;
            for (int32_t i = lane; i < m; i += 64) { const uint64_t k = from[i]; key = k > key ? k : key; }
            top = ap_uniform_u64(ap_wave_max_u64(key));
            const uint64_t last = from[m - 1];
            for (int32_t i = lane; i < m; i += 64)
                if (from[i] == top) from[i] = last;
        }
        ap_wave_sync();
        if (lane == owner) { head = top; held = m > 0 ? m - 1 : 0; }
    };
    // Whether all of the pool has been expanded, with `key` the best unexpanded document.
    auto over = [&](uint64_t key) -> bool {
        int32_t before = 0;
        for (int32_t i = lane; i < n; i += 64) before += l.done[i] > key ? 1 : 0;
        for (int32_t o = 1; o < 64; o <<= 1) before += __shfl_xor(before, o, 64);
        return __builtin_amdgcn_readfirstlane(before) >= g.L;
    };
    // Whether nothing that waits can be in the pool: enough documents are above the first line, or none wait.
    auto sure = [&]() -> bool { return c0 >= g.L || nwait == 0; };
    // Whether `key`, the best unexpanded document, is the next parent.
    auto parent = [&](uint64_t key) -> bool { return key != 0ull && !(n >= g.L && over(key)) && (ap_key_score(key) >= t0 || sure()); };
    for (int32_t i0 = 0; i0 < g.E; i0 += 64) {   // S7: entry points
        const int32_t v = i0 + lane < g.E ? g.entry[i0 + lane] : -1;
        uint32_t e = 0;
        float x = 0.f;
        fetch(v, e, x);
        take(v, v >= 0 && fresh(v), e, x);
    }
    if constexpr (ONE) {
        const int32_t el = lane < g.R ? lane : g.R - 1;
        auto edges = [&](int32_t u) -> int32_t { return g.graph[(int64_t)u * g.R + el]; };
        int32_t v = -1, u1 = -1, v1 = -1;
        for (;;) {
            int32_t owner;
            const uint64_t key = best(owner);
            if (bad || n >= g.done_cap || !parent(key)) break;
            const int32_t u = ap_key_id(key);
            const bool there = u == u1;
            uint32_t e = 0;
            float x = 0.f;
            if (there) {
                v = lane < g.R ? v1 : -1;
                fetch(v, e, x);
            } else v = edges(u);
            if (lane == 0) l.done[n] = key;
            n++;
            refill(owner);
            // the document after it, its edges (which of two with the same score does not matter here)
            const uint32_t top = ap_wave_max_u32((uint32_t)(head >> 32));
            const int32_t at = (int32_t)__builtin_ctzll(__ballot((uint32_t)(head >> 32) == top));
            u1 = __builtin_amdgcn_readfirstlane((int32_t)top) != 0 ? (int32_t)(0x3fffffffu - ((uint32_t)__builtin_amdgcn_readlane((int32_t)(uint32_t)head, at) >> 1)) : -1;
            v1 = edges(u1 < 0 ? 0 : u1);
            if (!there) {
                v = lane < g.R ? v : -1;
                fetch(v, e, x);
            }
            const bool on = v >= 0 && fresh(v);
            take(v, on, e, x);
            it++;
        }
    } else {
        for (;;) {
            int32_t found = 0;
            while (found < g.width && n < g.done_cap) {
                int32_t owner;
                const uint64_t key = best(owner);
                if (!parent(key)) break;
                if (lane == 0) { l.done[n] = key; l.par[found] = ap_key_id(key); }
                n++;
                found++;
                refill(owner);
            }
            // too few parents, and what waits may be better than none
            if (bad || n >= g.done_cap || found == 0 || (found < g.width && !sure())) break;
            ap_wave_sync();
            const int32_t total = found * g.R;
            const int32_t par = l.par[lane & 15];
            constexpr int CH = 4;
            for (int32_t base = 0; base < total; base += CH * 64) {
                int32_t v[CH];
                uint32_t e[CH];
                float x[CH];
#pragma unroll
                for (int c = 0; c < CH; c++) {
                    const int32_t i = base + c * 64 + lane, p = i < total ? i / g.R : 0;
                    const int32_t u = __shfl(par, p, 64);
                    v[c] = i < total ? g.graph[(int64_t)u * g.R + (i - p * g.R)] : -1;
                }
#pragma unroll
                for (int c = 0; c < CH; c++) { e[c] = 0; fetch(v[c], e[c], x[c]); }
#pragma unroll
                for (int c = 0; c < CH; c++)
                    if (base + c * 64 < total) take(v[c], v[c] >= 0 && fresh(v[c]), e[c], x[c]);
            }
            it++;
        }
    }
    n_done = n;
    if (bad || n >= g.done_cap || !sure()) return false;
    if (lane == 0 && g.counts) { g.counts[q * 3] = nscored; g.counts[q * 3 + 1] = it; g.counts[q * 3 + 2] = nwait; }   // the rows of what waits were not read
    return true;
}

// The walk of one wave with a sorted pool, as k_search's, for what the one with lists leaves undecided: every document it meets
// that was not scored ahead, and that its bound does not rule out, is scored by the other waves.
template <bool ALL>
__device__ __forceinline__ void ap_walk_sorted(const ApWalkArgs &g, int64_t q, const ApVisited &vis, const ApWalkLds &l) {
    const int lane = threadIdx.x & 63;
    uint64_t *const cur = l.cur;
    const uint32_t *bound = ALL ? nullptr : g.bound + q * g.ld;
    const float *exact = g.exact + q * g.ld;
    // uniform
    int32_t len = 0, fu = 0, it = 0, nscored = 0, nunread = 0, cnt = 0;   // fu: every entry of the pool before it has been expanded
    uint64_t worst = 0ull;      // the pool's last key while it is full, else 0: a key has to rank before it
    // Puts the keys of the lanes that hold one (each ranks before `worst`) into the pool.  The pool's entries are read in
    // chunks from the back; every entering key is compared with all of them at once, which gives the key its rank (a
    // ballot) and the entries their shift (they only move towards the end, so a chunk's writes land at or after the chunk's
    // own start).  The chunk in which the first entry stays put is the last: everything before it ranks before every key.
    auto merge = [&](bool has, uint64_t key) {
        const uint64_t mask = __ballot(has);
        if (mask == 0ull) return;
        const int32_t m = (int32_t)__popcll(mask);
        int32_t after = 0, e = 0;   // per lane: pool entries that rank after this lane's key, entering keys that rank before it
        int32_t hi = len;
        bool more = true, first = true;
        auto chunk = [&](auto width) {
            constexpr int CB = decltype(width)::value;
            const int32_t lo = hi > 0 ? (hi - 1) / (CB * 64) * (CB * 64) : 0;
            uint64_t r[CB];
            int32_t sh[CB];
#pragma unroll
            for (int b = 0; b < CB; b++) {   // what lies past the end ranks after every key
                const int32_t i = lo + b * 64 + lane;
                r[b] = i < hi ? cur[i] : 0ull;
                sh[b] = 0;
            }
            for (uint64_t bits = mask; bits; bits &= bits - 1ull) {
                const int32_t j = (int32_t)__builtin_ctzll(bits);
                const uint64_t k = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int32_t)(key >> 32), j) << 32) |
                                   (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int32_t)(uint32_t)key, j);
                int32_t below = 0;
#pragma unroll
                for (int b = 0; b < CB; b++) {
                    const uint64_t lt = __ballot(k > r[b]);
                    below += (int32_t)__popcll(lt);
                    sh[b] += k > r[b] ? 1 : 0;
                }
                after += lane == j ? below : 0;
                if (first) e += k > key ? 1 : 0;
            }
#pragma unroll
            for (int b = 0; b < CB; b++) {
                const int32_t i = lo + b * 64 + lane, d = i + sh[b];
                if (i < hi && sh[b] > 0 && d < g.L) cur[d] = r[b];
            }
            after -= lo + CB * 64 - hi;
            more = lo > 0 && __builtin_amdgcn_readfirstlane(sh[0]) != 0;
            hi = lo;
            first = false;
        };
        if (len <= 128) chunk(std::integral_constant<int, 2>());
        else while (more) chunk(std::integral_constant<int, 4>());
        const int32_t pos = len - after + e;
        if (has && pos < g.L) cur[pos] = key;
        const int32_t rmin = __builtin_amdgcn_readlane(pos, (int32_t)__builtin_ctzll(__ballot(has && e == 0)));
        fu = fu < rmin ? fu : rmin;
        len = len + m < g.L ? len + m : g.L;
        ap_wave_sync();
        if (len == g.L) worst = ap_uniform_u64(cur[g.L - 1]);
    };
    // One document a lane, `on` where it is a new one, with its bound and score as read: scored ones that rank before `worst`
    // enter (the answer, and their keys), other scored ones are done with; of the rest, those the bound does not rule out
    // are noted for scoring.
    auto take = [&](int32_t v, bool on, uint32_t e, float x, uint64_t &key) -> bool {
        const bool full = len == g.L;
        const bool known = on && (ALL || (e & 1u));
        key = ap_make_key(x, v < 0 ? 0 : v, 1u);
        const bool has = known && key > worst;
        const bool ask = on && !known && !(full && __uint_as_float(e & ~AP_BOUND_COUNT) < ap_key_score(worst));
        nscored += (int32_t)__popcll(__ballot(on));
        if constexpr (!ALL) {
            const uint64_t am = __ballot(ask);
            nunread += (int32_t)__popcll(__ballot(on && !known && !ask));
            if (am) {
                if (ask) {
                    const uint4 m = g.meta[v];
                    l.meta[cnt + (int32_t)__popcll(am & ((1ull << lane) - 1ull))] = make_uint4(m.x, m.y, m.z, (uint32_t)v);
                }
                cnt += (int32_t)__popcll(am);
            }
        }
        return has;
    };
    auto fetch = [&](int32_t v, uint32_t &e, float &x) {
        const int32_t at = v < 0 ? 0 : v;
        if constexpr (!ALL) e = bound[at];
        x = exact[at];
    };
    // the other waves score what was noted; their keys are merged
    auto help = [&]() {
        if constexpr (!ALL) {
            if (cnt == 0) return;
            if (lane == 0) { *l.c = cnt; *l.full = len == g.L; *l.worst = ap_key_score(worst); }
            ap_walk_meet();
            ap_walk_meet();
            for (int32_t c0 = 0; c0 < cnt; c0 += 64) {
                const uint64_t key = c0 + lane < cnt ? l.newk[c0 + lane] : 0ull;
                merge(key > worst, key);   // a candidate that was skipped has a key below every real one
            }
            cnt = 0;
        }
    };
    for (int32_t i0 = 0; i0 < g.E; i0 += 64) {   // S7: entry points
        const int32_t v = i0 + lane < g.E ? g.entry[i0 + lane] : -1;
        uint32_t e = 0;
        float x = 0.f;
        fetch(v, e, x);
        uint64_t key;
        const bool has = take(v, v >= 0 && !vis.test_and_set(v), e, x, key);
        merge(has, key);
    }
    help();
    for (;;) {
        // S8: the best `width` unexpanded entries, marked expanded
        int32_t found = 0, last = -1;
        for (int32_t base = fu & ~63; base < len && found < g.width; base += 64) {
            const int32_t i = base + lane;
            const uint64_t k = i < len ? cur[i] : 0ull;
            const uint64_t mask = __ballot((k & 1ull) != 0ull);
            if (mask == 0ull) continue;
            const int32_t rank = (int32_t)__popcll(mask & ((1ull << lane) - 1ull));
            const bool mine = (k & 1ull) != 0ull && found + rank < g.width;
            if (mine) { l.par[found + rank] = ap_key_id(k); cur[i] = k & ~1ull; }
            const uint64_t tm = __ballot(mine);
            last = base + 63 - (int32_t)__builtin_clzll(tm);
            found += (int32_t)__popcll(tm);
        }
        fu = last >= 0 ? last + 1 : len;
        if (found == 0) break;
        ap_wave_sync();
        const int32_t total = found * g.R;
        const int32_t par = l.par[lane & 15];
        constexpr int CH = 4;
        for (int32_t base = 0; base < total; base += CH * 64) {
            int32_t v[CH];
            uint32_t e[CH];
            float x[CH];
#pragma unroll
            for (int c = 0; c < CH; c++) {
                const int32_t i = base + c * 64 + lane, p = i < total ? i / g.R : 0;
                const int32_t u = __shfl(par, p, 64);
                v[c] = i < total ? g.graph[(int64_t)u * g.R + (i - p * g.R)] : -1;
            }
#pragma unroll
            for (int c = 0; c < CH; c++) { e[c] = 0; fetch(v[c], e[c], x[c]); }
            for (int c = 0; c < CH; c++)
                if (base + c * 64 < total) {
                    uint64_t key;
                    const bool has = take(v[c], v[c] >= 0 && !vis.test_and_set(v[c]), e[c], x[c], key);
                    merge(has, key);
                }
        }
        it++;
        help();
    }
    if (lane == 0 && g.counts) { g.counts[q * 3] = nscored; g.counts[q * 3 + 1] = it; g.counts[q * 3 + 2] = nunread; }
    // S9: the best k entries that are not mark-deleted
    int32_t o = 0;
    for (int32_t base = 0; base < len && o < g.k; base += 64) {
        const int32_t i = base + lane;
        const uint64_t k = i < len ? cur[i] : 0ull;
        const int32_t v = ap_key_id(k);
        const bool live = i < len && !(g.deleted && ((g.deleted[v >> 5] >> (v & 31)) & 1u));
        const uint64_t mask = __ballot(live);
        const int32_t at = o + (int32_t)__popcll(mask & ((1ull << lane) - 1ull));
        if (live && at < g.k) { g.out_ids[q * g.k + at] = v; g.out_scores[q * g.k + at] = ap_key_score(k); }
        o += (int32_t)__popcll(mask);
    }
    for (int32_t i = (o < g.k ? o : g.k) + lane; i < g.k; i += 64) { g.out_ids[q * g.k + i] = -1; g.out_scores[q * g.k + i] = -INFINITY; }
}

__device__ __forceinline__ ApVisited ap_walk_visited(const ApWalkArgs &g, int64_t q, uint64_t *lds, bool in_lds) {
    ApVisited vis{g.visited + (size_t)q * g.words, nullptr};
    if (in_lds) {
        vis.l = (AP_LDS uint32_t *)reinterpret_cast<uint32_t *>(lds + g.vis_at);
        for (size_t i = threadIdx.x; i < g.words; i += blockDim.x) vis.l[i] = 0u;
    }
    return vis;
}

// One workgroup per query.  Wave 0 walks; the others bring the rows of bounds and scores near, and rank the answer at the end.
template <bool ALL, bool ONE>
__global__ __launch_bounds__(AP_WALK_LIST_NT) void k_walk(ApWalkArgs g) {
    extern __shared__ __attribute__((aligned(16))) uint64_t walk_lds[];
    __shared__ int32_t s_done, s_par[16];
    ApWalkLds l;
    l.list = walk_lds;
    l.done = l.list + 64 * (g.cap + 1);
    l.par = s_par;
    const int64_t q = blockIdx.x;
    const ApVisited vis = ap_walk_visited(g, q, walk_lds, ONE || g.vis_lds);
    __syncthreads();
    if (ap_wave_id() == 0) {
        int32_t n_done = 0;
        const bool ok = ap_walk_lists<ALL, ONE>(g, q, vis, l, n_done);
        if (threadIdx.x == 0) { s_done = ok ? n_done : -1; g.undecided[q] = ok ? 0 : 1; }
    } else if (g.warm) {
        // the rows the walk reads one word at a time were written all over the chip: into this XCD's L2
        const float *exact = g.exact + q * g.ld;
        for (int64_t i = (threadIdx.x - 64) * 4; i < g.D.n; i += (AP_WALK_LIST_NT - 64) * 4) {
            const ap_u32x4_w x = *reinterpret_cast<const ap_u32x4_w *>(exact + i);
            asm volatile("" ::"v"(x));
            if constexpr (!ALL) {
                const ap_u32x4_w y = *reinterpret_cast<const ap_u32x4_w *>(g.bound + q * g.ld + i);
                asm volatile("" ::"v"(y));
            }
        }
    }
    __syncthreads();
    // S9: the best k of the pool (the best L of the expanded documents) that are not mark-deleted, all threads counting what
    // ranks before each
    const int32_t n = ap_uniform_i32(s_done);
    if (n < 0) return;
    if (g.deleted) {
        uint32_t out = 0u;   // a bit per document of this thread's (at most 32, see walk_lds_sizes): left out
        int32_t b = 0;
        for (int32_t i = threadIdx.x; i < n; i += AP_WALK_LIST_NT, b++) {
            const uint64_t k = l.done[i];
            const int32_t v = ap_key_id(k);
            int32_t at = 0;
            for (int32_t j = 0; j < n; j++) at += l.done[j] > k ? 1 : 0;
            if (at >= g.L || ((g.deleted[v >> 5] >> (v & 31)) & 1u)) out |= 1u << b;
        }
        __syncthreads();
        b = 0;
        for (int32_t i = threadIdx.x; i < n; i += AP_WALK_LIST_NT, b++)
            if ((out >> b) & 1u) l.done[i] = 0ull;
        __syncthreads();
    }
    int32_t live = 0;
    for (int32_t i0 = 0; i0 == 0 || i0 < n; i0 += AP_WALK_LIST_NT) {
        const int32_t i = i0 + (int32_t)threadIdx.x;
        const uint64_t k = i < n ? l.done[i] : 0ull;
        int32_t at = 0;
        live = 0;
        for (int32_t j = 0; j < n; j++) { const uint64_t o = l.done[j]; at += o > k ? 1 : 0; live += o != 0ull ? 1 : 0; }
        if (k != 0ull && at < g.k) { g.out_ids[q * g.k + at] = ap_key_id(k); g.out_scores[q * g.k + at] = ap_key_score(k); }
    }
    for (int32_t i = live + (int32_t)threadIdx.x; i < g.k; i += AP_WALK_LIST_NT) { g.out_ids[q * g.k + i] = -1; g.out_scores[q * g.k + i] = -INFINITY; }
}

// The queries the walk with lists left undecided, once more with a sorted pool: wave 0 walks, the others wait until there are
// documents to score (two barriers a time: when it has noted some, and when their keys are there).
template <int DT, int NV, bool ALL>
__global__ __launch_bounds__(AP_WALK_NT) void k_walk_rest(ApWalkArgs g) {
    extern __shared__ __attribute__((aligned(16))) uint64_t walk_lds[];
    __shared__ __attribute__((aligned(16))) uint64_t qtab[ApQTab<false>::SLOTS];
    __shared__ int32_t s_seed[2], s_c, s_full, s_par[16];
    __shared__ float s_worst;
    const int64_t q = blockIdx.x;
    if (g.undecided[q] == 0) return;   // uniform
    ApWalkLds l;
    l.meta = reinterpret_cast<uint4 *>(walk_lds);
    l.newk = reinterpret_cast<uint64_t *>(l.meta + g.cmax);
    l.cur = l.newk + g.cmax;
    l.c = &s_c; l.full = &s_full; l.par = s_par; l.worst = &s_worst;
    const ApVisited vis = ap_walk_visited(g, q, walk_lds, g.vis_lds);
    if (!g.vis_lds) for (size_t i = threadIdx.x; i < g.words; i += AP_WALK_NT) vis.g[i] = 0u;
    if (threadIdx.x == 0) s_c = 0;
    ApWalkQuery<DT, NV> Q;
    Q.load(g, q, qtab, s_seed);
    __threadfence_block();
    __syncthreads();
    if (ap_wave_id() == 0) {
        ap_walk_sorted<ALL>(g, q, vis, l);
        if (threadIdx.x == 0) s_c = -1;
        ap_walk_meet();
        return;
    }
    for (;;) {
        ap_walk_meet();
        const int32_t c = ap_uniform_i32(s_c);
        if (c < 0) break;
        (void)Q.template score<AP_WALK_NT / 64 - 1, 2, 1>(g, qtab, l.meta, c, l.newk, s_full != 0, s_worst, s_full != 0);   // rows requested along with the records
        ap_walk_meet();
    }
}

// Entries of a lane's list and of the list of expanded documents, and the dynamic LDS they take: the arrays of the sorted walk
// (candidates, unless all documents are scored ahead, and pool) lie in the same place.
static bool walk_lds_sizes(int32_t beam, int32_t cmax, int32_t *cap, int32_t *done_cap, size_t *bytes) {
    const size_t lds = (size_t)160 * 1024 - 4096;   // the static arrays take the rest
    *done_cap = beam + beam / 4 + 64;
    const size_t most = lds > (size_t)*done_cap * 8 ? (lds - (size_t)*done_cap * 8) / 512 : 0;
    *cap = (int32_t)std::min<size_t>(std::max(32, beam * 12 / 64), most > 2 ? most - 2 : 0) / 2 * 2;   // even
    *bytes = std::max(((size_t)64 * (size_t)(*cap + 1) + (size_t)*done_cap) * 8, (size_t)beam * 8 + (size_t)cmax * 24);
    return *cap >= 32 && *bytes <= lds && *done_cap <= 32 * AP_WALK_LIST_NT;
}

int ap_walk_launch(const ap_index *ix, const ApWalk &walk, uint32_t *visited, const ApVecs &Q, const float *w, int32_t w_stride, int32_t k, int32_t beam,
                   int32_t width, int32_t *counts, int32_t *out_ids, float *out_scores, hipStream_t st) {
    const bool all = walk.bound == nullptr;
    const int64_t nq = Q.n, n = ix->docs.n;
    ApWalkArgs g;
    g.D = ix->docs; g.Q = Q; g.graph = ix->graph; g.entry = ix->entry; g.w = w; g.w_stride = w_stride;
    g.no_tables = g_ap_debug.search_query_lists != 0;
    g.R = ix->params.degree; g.E = ix->params.n_entry; g.k = k; g.L = beam; g.width = width;
    g.cmax = std::max(g.E, g.width * g.R);
    g.words = ((size_t)n + 31) / 32;
    g.visited = visited;
    g.out_ids = out_ids; g.out_scores = out_scores; g.counts = counts;
    g.rec = ix->rec; g.meta = ix->meta; g.deleted = ix->deleted;
    g.bound = reinterpret_cast<uint32_t *>(walk.bound);
    g.exact = walk.exact; g.ld = walk.ld; g.line = walk.line;
    g.undecided = reinterpret_cast<int32_t *>(walk.line + nq * AP_WALK_LEVELS);
    g.warm = (double)nq * (double)g.ld * (all ? 4 : 8) <= 24e6;   // the rows fit the L2 of the eight XCDs
    size_t smem = 0;
    AP_REQUIRE(walk_lds_sizes(beam, g.cmax, &g.cap, &g.done_cap, &smem), "beam and search_width need too much LDS");
    g.vis_at = (int32_t)(smem / 8);
    g.vis_lds = g_ap_debug.search_visited_global == 0 && smem + g.words * 4 <= (size_t)160 * 1024 - 4096 ? 1 : 0;
    if (g.vis_lds) smem += g.words * 4;
    else AP_TRY(ap_fill_u32(visited, g.words * (size_t)nq, 0u, st));
    auto lines = [&](const float *table) {
        hipLaunchKernelGGL(k_walk_lines, dim3((unsigned)nq), dim3(512), 0, st, reinterpret_cast<const uint32_t *>(table), g.ld, n,
                           make_float4(walk.share[0], walk.share[1], walk.share[2], walk.share[3]), walk.line);
    };
    if (!all) lines(walk.bound);
    // four blocks a CU, of a multiple of the block's threads
    const int64_t runs = std::max<int64_t>(1, std::min<int64_t>((n + AP_WALK_SCORE_NT - 1) / AP_WALK_SCORE_NT, (1024 + nq - 1) / nq));
    g.per_block = all ? (n + runs - 1) / runs : ((n + runs - 1) / runs + AP_WALK_SCORE_NT - 1) / AP_WALK_SCORE_NT * AP_WALK_SCORE_NT;
    const dim3 grid((unsigned)((n + g.per_block - 1) / g.per_block) + (all ? 0u : 1u), (unsigned)nq);
    const bool one = width == 1 && g.R <= 64 && g.vis_lds;
    hipError_t e = hipSuccess;
    auto launch = [&](auto kernel, unsigned nt) {
        if (e == hipSuccess && smem > 48 * 1024) e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        if (e == hipSuccess) hipLaunchKernelGGL(kernel, dim3((unsigned)nq), dim3(nt), smem, st, g);
    };
    if (all) {
        AP_DISPATCH_DENSE(ix->dtype, ix->docs.dim, hipLaunchKernelGGL((k_walk_score<DT, NV, true>), grid, dim3(AP_WALK_SCORE_NT), 0, st, g));
        lines(walk.exact);
        if (one) launch(&k_walk<true, true>, AP_WALK_LIST_NT); else launch(&k_walk<true, false>, AP_WALK_LIST_NT);
        launch(&k_walk_rest<AP_F32, 1, true>, AP_WALK_NT);   // nothing is left to score: any instantiation serves
    } else {
        AP_DISPATCH_DENSE(ix->dtype, ix->docs.dim, hipLaunchKernelGGL((k_walk_score<DT, NV, false>), grid, dim3(AP_WALK_SCORE_NT), 0, st, g));
        if (one) launch(&k_walk<false, true>, AP_WALK_LIST_NT); else launch(&k_walk<false, false>, AP_WALK_LIST_NT);
        AP_DISPATCH_DENSE(ix->dtype, ix->docs.dim, launch(&k_walk_rest<DT, NV, false>, AP_WALK_NT));
    }
    AP_CHECK_HIP(e);
    AP_CHECK_HIP(hipGetLastError());
    return AP_OK;
}

// Whether a batch is searched by the walk, and whether out of the bounds (1) or with every document scored ahead (2), by what was
// measured (microseconds; f32 rows of 768 columns and bf16 rows of 1,024, 3,000 to 100,000 documents, 1 to 1,000 queries):
//  - the walk: 60 and 1.1 an entry of the pool (2.0 at 2,048 entries, whose lists are longer than a wave), whatever the number
//    of parents, out of the bounds 45 more (several parents: 90 either way); a batch that does not fit the chip at once takes that several times;
//  - scoring ahead: the documents' bytes at 5 TB/s, 0.4 ns a document at least; all documents of a corpus that the last-level
//    cache holds, at 16 TB/s from the second query on;
//  - k_search with bounds: 80, per iteration 5.5 with one parent (6.6 from 90 queries on), 13.6 with four, 18 with sixteen (0.45 of that on 3,000
//    documents, whose descriptors and rows are all close by; 18 and more where it runs without bounds), 0.09 ns for every document it reaches
//    while the chip is full (0.24 without bounds).
// One query of 100,000 documents, pool 128: 867 -> 254 us (all scored ahead: the scores 92, the lines 11, the walk 137);
// 37 of 120,011, pool 512: 3.17 -> 0.93 ms (out of the bounds: these 0.10 ms, the lines 0.01, the scores 0.14, the walk 0.63).  Where the walk would not be an eighth faster by this count (a fifth with more parents, for which
// the 60, the 80, the 6.6 and the 45 were not measured), k_search stays:
// 16 queries of 20,000 documents of 768 columns, pool 128, four parents: 482 and 316 us. 300 queries with a pool of 128, 1.2 and 1.6 ms.  16 queries of 60,000 documents of 128 columns, pool 32: 293 and 178 us, 64 of 100,000 of 768, pool 128: 1,067 and 647.
// A way whose lists would not hold what enters them is not taken: a query whose list is full is searched twice (43,000 documents, degree 32,
// 3 queries, pool 2,048: 10.9 ms by k_search, 13.3 scored ahead, 4.3 out of the bounds; degree 64, pool 3,600: 14.8, 29.0 and 7.9).  Documents that are
// met enter while they score at least the last line that the pool has filled, taking those met for any of the corpus; what leaves as a parent
// makes up for lanes that get more than others.  Lists stayed whole up to 1.0 of their room by this count and were full from 1.1 on.
// The first line: three times the share of the documents that the pool holds of those a search reaches, if it met them at
// random, and so many that six of the entry points and first neighbours are above it; a search that finds less runs twice.
ApWalkPlan ap_walk_plan(const ap_index *ix, int64_t nq, int32_t beam, int32_t width, int32_t max_iters, bool bounds, bool can_bound) {
    ApWalkPlan p;
    const int forced = (int)g_ap_debug.search_walk;
    if (forced == 1 || (forced == 0 && g_ap_debug.search_bounds != 0) || nq < 1 || nq > 4096 || max_iters > 0) return p;
    int32_t cap, done_cap;
    size_t bytes;
    if (!walk_lds_sizes(beam, std::max(ix->params.n_entry, width * ix->params.degree), &cap, &done_cap, &bytes)) return p;
    const double n = (double)ix->docs.n, q = (double)nq, iters = (double)beam / width;
    const double met = n * (1.0 - exp(-(double)beam * ix->params.degree / n)), share = beam / met;
    const double first = std::min(1.0, std::max(3.0 * share, 6.0 / (ix->params.n_entry + ix->params.degree)));
    const double row = (double)ix->docs.dim * (ix->dtype == AP_BF16 ? 2 : 4) + 8.0 * (double)(ix->sp_nnz + ix->tx_nnz) / n;   // bytes of a document
    const double per_cu = std::min(8.0, floor(160.0 * 1024 / (double)(bytes + 1024 + (n <= 65536 ? n / 8 : 0))));
    const bool single = width == 1;
    const double walk = (single ? 60.0 : 90.0) + beam * (1.1 + std::max(0, beam - 512) * 6e-4) * ceil(q / (256.0 * std::max(1.0, per_cu)));
    const double table = ap_bound_cost(ix, nq);
    const double out_of_bounds = walk + (single ? 45.0 : 0.0) + table + q * first * n * std::max(0.4e-3, row / 5e6);
    const double all = walk + n * row / 5e6 + (q - 1) * n * std::max(0.16e-3, row / (n * row <= 2e8 ? 16e6 : 7.5e6));
    const double near = std::min(1.2, std::max(0.4, 0.45 + 0.36 * log10(n / 3000.0)));
    const double other = bounds ? table + (single ? 80.0 : 0.0) + std::max(iters * near * (5.5 + (single ? 0.012 * std::min(q, 90.0) : std::min(2.7 * (width - 1), 12.5))), q * met * 0.09e-3)
                                : std::max(iters * near * 18.0, q * met * 0.24e-3);
    double lines[2][4] = {{first, first / 2, 1.5 * share, share}, {std::max(0.5, 8 * share), 8 * share, 3 * share, 1.2 * share}};
    for (auto &l : lines) for (double &s : l) s = std::min(1.0, s);
    // a lane's list takes the neighbours at its own places of the parents' edges
    const double edges = (double)width * ix->params.degree, room = cap * edges / ceil(edges / 64.0);
    auto fits = [&](int mode) {
        const double *s = lines[mode - 1];
        double enter = 0.0, seen = 0.0, part = mode == 1 ? first : 1.0;   // out of the bounds nothing enters that was not scored ahead
        for (int i = 0; i < 5; i++) {
            const double until = i < 4 ? std::min(met, beam / s[i]) : met;
            if (until > seen) { enter += (until - seen) * part; seen = until; }
            if (i < 4) part = s[i];
        }
        return enter <= room;
    };
    const bool some = can_bound && ix->bd_mem != nullptr;
    if (forced != 0) p.mode = some && forced == 2 ? 1 : 2;
    else {
        const double cost[2] = {some && fits(1) ? out_of_bounds : INFINITY, fits(2) ? all : INFINITY};
        p.mode = cost[0] < cost[1] ? 1 : 2;
        if (cost[p.mode - 1] > (single ? 0.88 : 0.8) * other) { p.mode = 0; return p; }
    }
    for (int i = 0; i < 4; i++) p.share[i] = (float)lines[p.mode - 1][i];
    return p;
}
