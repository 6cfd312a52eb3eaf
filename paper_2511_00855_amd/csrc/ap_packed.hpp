// Packed lists (ap_packed.hip): a document's learned-sparse and lexical entries, three bytes each, in units of four entries
// (12 bytes): four weights, rounded up to 8 bits of the list's largest, then the slots of their four terms (16 bits each; several
// rare terms may share a slot).  Unit 0 holds the scales of the two lists and the norm of the dense row.  A record begins
// on a line of 64 bytes.
#pragma once
#include "ap_common.hpp"

#define AP_PK_LINE 64
#define AP_PK_DIRECT 16384   // slots of frequent terms, one each
#define AP_PK_SP 4096        // slots that the other learned-sparse terms share
#define AP_PK_TX 12288       // ... and the other lexical terms
#define AP_PK_SLOTS (AP_PK_DIRECT + AP_PK_SP + AP_PK_TX)
#define AP_PK_LEAST 512      // documents below which nothing is packed
// Entries times K below which nothing is packed either: it takes some 0.1 ms then, and saves less.  Construction, records read -> packed: 1,000
// documents of 31 entries, K = 32 (1.0 million) 1.09 -> 1.17 ms, K = 64 (2.0 million) 1.83 -> 1.90; 513 of 190 entries, K = 32 (3.1 million) 1.35 -> 1.10.
#define AP_PK_WORK ((int64_t)1 << 21)
#define AP_PK_VOCAB ((int64_t)1 << 24)   // terms of both vocabularies together a table of slots is made for

// The line a record begins on, from the entries before it and its number: a record of e entries takes at most 12 + 3 e + 18
// bytes, and successive records begin at least 3 e + 96 - 63 bytes apart, so no sum over the documents is needed.
__host__ __device__ static inline int64_t ap_pk_line(int64_t entries_before, int64_t v) { return (3 * entries_before + 96 * v + AP_PK_LINE - 1) / AP_PK_LINE; }

struct ApPacked {
    size_t bytes = 0;
    void *mem = nullptr;             // one allocation; NULL: no packed lists
    const uint32_t *rec = nullptr;
    const uint2 *at = nullptr;       // per document: its line, units of either list (16 bits each)
};
int ap_pack_lists(const ap_index *ix, hipStream_t st, ApPacked *out);

#ifdef __HIPCC__
struct ApPkUnit { uint32_t w, s01, s23; };
// One side's weights by slot, a byte each, in LDS, against the four entries of a unit.
__device__ __forceinline__ uint32_t ap_pk_dot(const AP_LDS uint8_t *tab, const ApPkUnit &u) {
    const uint32_t a = (uint32_t)tab[u.s01 & 0xffffu] | ((uint32_t)tab[u.s01 >> 16] << 8) | ((uint32_t)tab[u.s23 & 0xffffu] << 16) | ((uint32_t)tab[u.s23 >> 16] << 24);
    return __builtin_amdgcn_udot4(u.w, a, 0u, false);
}
#endif
