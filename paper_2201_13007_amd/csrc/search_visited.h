// The visited set of the search kernels that do not need to know which worker reached a
// vertex first: sets of exact tags in LDS, and behind them a table in the query's workspace
// region.
#pragma once
#include "search_body.h"

namespace sa {
namespace search_detail {

// Whether a set's word (a count in the top two bits, that many tags of tb bits below) holds
// tag.  (Written without conditions on lanes: those cost more than the selects.)
__device__ __forceinline__ bool in_set(uint32_t word, uint32_t tag, uint32_t tb)
{
    const uint32_t t1 = word >> tb;
    const uint32_t w0 = __builtin_amdgcn_ubfe(word, 0u, tb) == tag ? 0u : 3u;
    const uint32_t w1 = __builtin_amdgcn_ubfe(t1, 0u, tb) == tag ? 1u : 3u;
    const uint32_t w2 = __builtin_amdgcn_ubfe(t1, tb, tb) == tag ? 2u : 3u;
    return min(min(w0, w1), w2) < (word >> 30);
}

// The first vertices visited, in sets in LDS.  A vertex's id u is mapped by
// h = u * K_B mod 2^B, with K_B the odd number nearest 2^B / golden ratio (Fibonacci hashing
// at B bits: one-to-one on ids of B bits, and ids close together land in sets far apart); the
// top log2 bits of h pick one of 2^log2 sets and the other tb = B - log2 bits are the tag, so a
// tag names one vertex exactly.  A set's word holds a count of tags in its top two bits and
// up to W = min(3, 30 / tb) tags below.  Tags stay: as long as a set has room, a vertex that
// is not in it is new and is put there, with no access to the workspace table; a vertex that
// finds its set full is claimed in the table.  (Ids of more than 15 + log2 bits: every vertex
// is.)  Behind the sets, a quarter as many of vertices lately claimed or found in the table,
// by the same hash with two tag bits more, the newest tag lowest; a new tag pushes the
// oldest out.  Both are zero at first.  Any number of lanes and wavefronts of the workgroup
// may claim at once.
struct Seen {
    uint32_t *const sets, *const recent;
    const int hbits, tbits, rbits;
    const uint32_t hmul;

    // words of LDS: 5/4 2^log2, 16-byte aligned
    __device__ __forceinline__ Seen(uint32_t *lds, int log2, int idbits)
        : sets(lds), recent(lds + (1 << log2)), hbits(idbits > log2 ? idbits : log2 + 1), tbits(hbits - log2),
          rbits(tbits + 2), hmul((2654435769u >> (32 - hbits)) | 1u)
    {
    }

    __device__ __forceinline__ uint32_t hash(uint32_t u) const { return (u * hmul) & (0xFFFFFFFFu >> (32 - hbits)); }

    // the first vertex of a search, into the empty set; false: it belongs in the table
    __device__ __forceinline__ bool put_first(uint32_t u) const
    {
        if (tbits > 15) return false;
        const uint32_t h = hash(u);
        sets[h >> tbits] = (1u << 30) | (h & ((1u << tbits) - 1u));
        return true;
    }

    // *fresh: u is new, and now in the set.  True: the table has to tell (and is told: u
    // counts as claimed or found there from now on).
    __device__ __forceinline__ bool claim(uint32_t u, bool *fresh) const
    {
        bool ask = true;
        const uint32_t h = hash(u);
        if (tbits <= 15) {
            const uint32_t ways = tbits <= 10 ? 3u : 2u;
            uint32_t *const set = sets + (h >> tbits);
            const uint32_t tag = h & ((1u << tbits) - 1u);
            uint32_t sw = *set;
            for (;;) {
                const uint32_t cnt = sw >> 30;
                const bool known = in_set(sw, tag, tbits);
                ask = !known;
                if (known | (cnt == ways)) break;
                const uint32_t old = atomicCAS(set, sw, (sw + (1u << 30)) | (tag << (cnt * tbits)));
                if (old == sw) {
                    *fresh = true;
                    ask = false;
                    break;
                }
                sw = old;   // another lane put a vertex into the set
            }
        }
        if (ask && rbits <= 15) {
            const uint32_t rways = rbits <= 10 ? 3u : 2u;
            const uint32_t tag = h & ((1u << rbits) - 1u);
            uint32_t *const set = recent + (h >> rbits);
            const uint32_t sw = *set;
            ask = !in_set(sw, tag, rbits);
            if (ask)
                *set = (min((sw >> 30) + 1u, rways) << 30) | (((sw << rbits) | tag) & ((1u << (rways * rbits)) - 1u));
        }
        return ask;
    }
};

// Slots of vertex u in a table of 2^t entries (t >= 6).  The first probe keeps the 32
// vertices of one id block (u / 32) together in one 128-byte line, each at its own offset:
// neighbours that a breadth-first numbering gave nearby ids then share lines, within a
// step and from one step to the next, so a step's claims touch about half as many lines
// and most of them are still in the L2 from the step before.  Later probes move by an odd
// stride 32 r + 1 (r odd): a new line every time, and every slot of the table in turn.
__device__ __forceinline__ uint32_t block_slot(uint32_t u, int t)
{
    return ((((u >> 5) * 2654435761u) >> (37 - t)) << 5) | (u & 31u);
}

__device__ __forceinline__ uint32_t block_stride(uint32_t u, int t)
{
    const uint32_t r = (((u ^ 0x9E3779B9u) * 2654435761u) >> (37 - t)) | 1u;
    return ((r << 5) | 1u) & ((1u << t) - 1u);
}

// find or insert u; *fresh tells whether this call inserted it.  NO_SLOT: table full.
__device__ __forceinline__ uint32_t claim(uint32_t *T, int log2cap, uint32_t u, bool *fresh)
{
    const uint32_t mask = (1u << log2cap) - 1u;
    uint32_t s = block_slot(u, log2cap);
    const uint32_t step = block_stride(u, log2cap);
    *fresh = false;
    for (uint32_t probe = 0; probe <= mask; ++probe) {
        const uint32_t old = atomicCAS(&T[s], 0u, u + 1u);
        if (old == 0u) {
            *fresh = true;
            return s;
        }
        if (old == u + 1u) return s;
        s = (s + step) & mask;
    }
    return NO_SLOT;
}

// The rest of claim() after its first probe, given what that probe's compare-and-swap at
// block_slot(u, log2cap) returned: lets the caller issue the first probes of a step, go on
// with other loads, and read the results later.
__device__ __forceinline__ uint32_t claim_rest(uint32_t *T, int log2cap, uint32_t u, uint32_t old, bool *fresh)
{
    const uint32_t mask = (1u << log2cap) - 1u;
    uint32_t s = block_slot(u, log2cap);
    *fresh = old == 0u;
    if (old == 0u || old == u + 1u) return s;
    const uint32_t step = block_stride(u, log2cap);
    for (uint32_t probe = 1; probe <= mask; ++probe) {
        s = (s + step) & mask;
        old = atomicCAS(&T[s], 0u, u + 1u);
        if (old == 0u) {
            *fresh = true;
            return s;
        }
        if (old == u + 1u) return s;
    }
    return NO_SLOT;
}

// Moves the visited set from the table in use (2^t1 entries) into one twice as large,
// 2^t2 entries at the same address (the region holds the largest; past the table in use
// it is zero).  The entries are copied out to scratch (the second half of the region) and
// the table is cleared; then they are inserted again and scratch is cleared.  Returns the
// number of entries moved.  The whole wavefront takes part.
__device__ __forceinline__ int grow_table(uint32_t *tbl, uint32_t *scratch, int t1, int t2)
{
    const int lane = __lane_id();
    int cnt = 0;
    for (int b = 0; b < (1 << t1); b += 64) {   // 2^t1 >= 64 entries
        const uint32_t e = tbl[b + lane];
        const uint64_t m = __ballot(e != 0u);
        if (e != 0u) scratch[cnt + bits_below(m)] = e;
        tbl[b + lane] = 0u;
        cnt += __popcll(m);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    __builtin_amdgcn_wave_barrier();
    for (int i = lane; i < cnt; i += 64) {
        bool fresh;
        (void)claim(tbl, t2, scratch[i] - 1u, &fresh);
        scratch[i] = 0u;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    __builtin_amdgcn_wave_barrier();
    return cnt;
}

// Zeroes the first 2^t entries of tbl (2^t >= 64, 16-byte aligned) with 16-byte stores.
__device__ __forceinline__ void clear_table(uint32_t *tbl, int t)
{
    uint4 *const p = reinterpret_cast<uint4 *>(tbl);
    const uint4 z = make_uint4(0u, 0u, 0u, 0u);
    for (int i = __lane_id(); i < (1 << (t - 2)); i += 64) p[i] = z;
}

}  // namespace search_detail
}  // namespace sa
