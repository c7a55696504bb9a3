// A sorted queue of keys in the registers of a wavefront: NI slots per lane, entry p in slot
// p / 64 of lane p % 64, and wave-uniform masks of its unchecked entries.
#pragma once
#include "search_body.h"

namespace sa {
namespace search_detail {

template <int NI>
struct Queue {
    uint64_t k[NI];    // keys; KEY_EMPTY past the end
    uint64_t un[NI];   // unchecked entries (wave-uniform; zero past the end)
    uint64_t top;      // NI > 4: in lane i the last key of slot i, KEY_EMPTY in the other lanes
    int len;
};

// Calls f with the constant s (uniform, in [LO, HI)), by halving: an access to the queue
// indexed by a variable would make the compiler move the arrays to scratch memory.
template <int LO, int HI, typename F>
__device__ __forceinline__ void at_slot(int s, F f)
{
    if constexpr (HI - LO == 1) {
        f(std::integral_constant<int, LO>{});
    } else {
        constexpr int MID = (LO + HI) / 2;
        if (s < MID) at_slot<LO, MID>(s, f);
        else at_slot<MID, HI>(s, f);
    }
}

// Calls f with the constants first .. NI - 1, and I .. first downwards.
template <int NI, int I = 0, typename F>
__device__ __forceinline__ void slots_from(int first, F f)
{
    if constexpr (I < NI) {
        if (I >= first) f(std::integral_constant<int, I>{});
        slots_from<NI, I + 1>(first, f);
    }
}

template <int I, typename F>
__device__ __forceinline__ void slots_down(int first, F f)
{
    if constexpr (I >= 0) {
        if (I < first) return;
        f(std::integral_constant<int, I>{});
        slots_down<I - 1>(first, f);
    }
}

// Takes the first entry of the masks m (one bit per queue entry) out of them and returns its
// id, or -1 if they are empty.
template <int NI, int I = 0>
__device__ __forceinline__ int32_t take_first(const uint64_t (&k)[NI], uint64_t (&m)[NI])
{
    if constexpr (I < NI) {
        if (m[I] != 0ull) {
            const int b = __builtin_ctzll(m[I]);
            m[I] &= m[I] - 1ull;
            return (int32_t)rdlane((uint32_t)k[I], b);
        }
        return take_first<NI, I + 1>(k, m);
    }
    return -1;
}

template <int NI>
__device__ __forceinline__ bool any_unchecked(const Queue<NI> &Q)
{
    uint64_t b = 0;
#pragma unroll
    for (int i = 0; i < NI; ++i) b |= Q.un[i];
    return b != 0ull;
}

// key at the uniform position p
template <int NI>
__device__ __forceinline__ uint64_t get_key(const Queue<NI> &Q, int p)
{
    uint64_t r;
    at_slot<0, NI>(p >> 6, [&](auto i) { r = rdlane64(Q.k[i], p & 63); });
    return r;
}

// Inserts the unchecked keys mk of the lanes in sbits (distinct, none in the queue),
// keeping at most L entries, and returns the update position: the best position one of
// them takes (L if none stays).  Every new key finds its place (the queue keys below it) by
// compares with whole slots: all of them up to four slots, beyond only the slot that the
// slots' last keys give.  Its rank among the new keys is added per lane.  An old entry moves
// up by the new keys below it.  Then the slots from the first that changes on are put
// together in LDS: in one exchange where STAGE holds all slots (few queries: one round trip
// through LDS instead of one per slot), else slot by slot from the last down, each from its
// own entries that stay in it, those that come up from the slot below (none moves by more
// than 64) and the new ones.  The unchecked flags travel as bit 31 of the ids.
// stage: 64 keys (STAGE: 64 NI) and one that takes what lands elsewhere.
//
// This replaced a form that kept a landing mask per slot and pulled every entry with
// cross-lane permutes: some 60 instructions per new key and 30 per slot against 25 and 25 at
// three slots.  With 10 new keys a step that was half of a step's 1,300 instructions.
template <int NI, bool STAGE>
__device__ __forceinline__ int insert_batch(Queue<NI> &Q, int L, uint64_t mk, uint64_t sbits, uint64_t *stage)
{
    constexpr bool ALL = NI <= 4;   // compare with every slot, and keep the entries' moves from it
    const int lane = __lane_id();
    int shift[ALL ? NI : 1];
#pragma unroll
    for (int i = 0; i < (ALL ? NI : 1); ++i) shift[i] = 0;
    int f = 1 << 20;   // where this lane's new key lands
    int r = 0;         // new keys below it
    int fmin = L;
    for (uint64_t b = sbits; b; b &= b - 1) {
        const int j = __builtin_ctzll(b);
        const uint64_t kj = rdlane64(mk, j);
        int below;
        if constexpr (ALL) {
            below = 64 * NI;
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const bool above = Q.k[i] > kj;
                shift[i] += above ? 1 : 0;
                below -= __popcll(__ballot(above));
            }
        } else {
            // (the last key of a full queue is above kj, so the slot exists)
            const int s = __popcll(__ballot(Q.top < kj));
            at_slot<0, NI>(s, [&](auto i) { below = 64 * i + __popcll(__ballot(Q.k[i] < kj)); });
        }
        r += kj < mk ? 1 : 0;
        f = lane == j ? below : f;
        fmin = min(fmin, below);   // the best new key has no other below it
    }
    if (fmin >= L) return L;
    const int place = f;
    f += r;
    const int nlen = min(L, Q.len + __popcll(sbits));
    const int i_first = fmin >> 6;
    // by how much this lane's entry of slot i moves up, and the same for the slots above
    const auto moves = [&](int i) {
        if constexpr (ALL) return shift[i];
        int c = __popcll(__ballot(place < 64 * i));   // (lanes without a new key: 2^20)
        for (uint64_t b = __ballot((place >> 6) == i); b; b &= b - 1)
            c += (int)rdlane((uint32_t)place, __builtin_ctzll(b)) <= 64 * i + lane ? 1 : 0;
        return c;
    };
    const auto flagged = [&](uint64_t key, uint64_t un) {
        return key | (__builtin_amdgcn_inverse_ballot_w64(un) ? 0x80000000ull : 0ull);
    };
    const auto take = [&](auto i, uint64_t v) {
        const bool keep = lane < nlen - 64 * i;
        Q.un[i] = __ballot(keep && ((uint32_t)v >> 31) != 0u);
        Q.k[i] = keep ? v & ~0x80000000ull : KEY_EMPTY;
        if constexpr (!ALL) {
            const uint64_t last = rdlane64(Q.k[i], 63);
            Q.top = lane == i ? last : Q.top;
        }
    };
    if constexpr (STAGE) {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            if (i < i_first) continue;
            stage[min((uint32_t)(64 * i + lane + moves(i)), 64u * NI)] = flagged(Q.k[i], Q.un[i]);
        }
        stage[min((uint32_t)f, 64u * NI)] = mk | 0x80000000ull;
        __builtin_amdgcn_wave_barrier();
        uint64_t v[NI];
#pragma unroll
        for (int i = 0; i < NI; ++i) v[i] = stage[64 * i + lane];
        __builtin_amdgcn_wave_barrier();
        slots_from<NI>(i_first, [&](auto i) { take(i, v[i]); });
    } else {
        int mine = moves(NI - 1);
        slots_down<NI - 1>(i_first, [&](auto ii) {
            constexpr int i = ii, h = i > 0 ? i - 1 : 0;
            const int below = i > 0 ? moves(h) : 0;   // moves of the slot below
            // offsets within the slot, 64 for what lands elsewhere
            const uint32_t own = min((uint32_t)(lane + mine), 64u);
            const uint32_t add = min((uint32_t)(f - 64 * i), 64u);
            stage[own] = flagged(Q.k[i], Q.un[i]);
            if (i > 0) stage[min((uint32_t)(lane + below - 64), 64u)] = flagged(Q.k[h], Q.un[h]);
            stage[add] = mk | 0x80000000ull;
            __builtin_amdgcn_wave_barrier();
            const uint64_t v = stage[lane];
            __builtin_amdgcn_wave_barrier();
            take(ii, v);
            mine = below;
        });
    }
    Q.len = nlen;
    return fmin;
}

}  // namespace search_detail
}  // namespace sa
