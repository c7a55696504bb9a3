// The general search kernel: several workers that merge when Algorithm 2 says so (or every so
// many steps), and one worker with an LDS visited table.
//
// One workgroup runs one query; worker t of Algorithm 3 is wavefront t.  Between two merges a
// worker's local queue is S with the worker's own new entries among it, cut at L, and it may
// expand its share of S and its own new entries.  So the local queue is never built: S stands
// once in LDS, the same for all workers, a worker's share is a bit mask per 64 entries, and
// only its own new entries are its own, in registers and in no order: a sort would be wasted,
// with a merge every other local step.  The place of an entry in the local queue is the
// count of smaller entries in S and among the own ones; one whose place is L or more has
// fallen out and is never expanded (places only grow), and a merge drops it, since L
// smaller ones exist.
//
// A local step: expand the first entry of the share or the smallest own one, whichever is
// smaller; claim its neighbours; a barrier; the distances of those this worker got, appended
// to the own entries; the next entry to expand is picked and the test of Algorithm 2 taken on
// the other side of a second barrier.  The row of the entry that looks next is read ahead.
// A merge publishes the own entries to LDS, counts for each the smaller ones in S and among
// the published, writes it to its place in the next S, and fills the other places from S in
// order (as search_bsp.hip does).  One active worker (the first step of a staged search, half
// of the local steps of some) takes its local steps in one wavefront, as search_single.h does.
//
// Every entry of S is a key with the id moved up by one bit and the unchecked flag below it.
//
// A vertex reached by several workers in one local step goes to the lowest (worker,
// adjacency slot): claims carry that order in their tag and the smallest tag of the step wins
// (two phases around the first barrier), which is the order a sequential emulation visits
// them in.  The visited set is an open-addressing hash of 64-bit entries
// ((id + 1) << 32 | tag), zero meaning empty, kept in LDS or in the query's region of the
// workspace (a query moves it there when the LDS table passes half full); workspace slots
// a query writes are listed and zeroed again before it ends.
//
// Bound by latency: a local step is the row (when not read ahead), the claims, two barriers,
// the gather and some eight round trips through LDS.  The form before this held every
// worker's copy of S in registers with a tag per entry: a new key was compared with all of
// it, a merge reloaded it, and all of it was published.  Over 200K x 128, adaptive: 33 queries
// with 8 workers, L = 272 903 -> 793 us, L = 512 1,520 -> 1,093; with 16 workers, L = 768
// 2,043 -> 1,302; four workers, L = 192, 1,000 queries 1,124 -> 900 and 10,000 5,947 -> 4,997.
#pragma once
#include "search_body.h"
#include "search_queue.h"
#include "search_visited.h"

#include <algorithm>
#include <atomic>
#include <climits>

namespace sa {
namespace search_detail {

constexpr int MAXW = 16;
constexpr int PUBCAP = 512;   // new keys published per round of a merge

// Room for them: no more than the workers can have (the 1 KB less at L <= 64 lets a fourth
// query of three workers into a CU).
__host__ __device__ inline uint32_t pub_room(int L, int M)
{
    const int all = 64 * M * (queue_slots_bucket(L, 2) + 1);
    return (uint32_t)(all < PUBCAP ? all : PUBCAP);
}

struct Ctrl {
    int32_t U[MAXW];
    int32_t work[MAXW];
    int32_t nnew[MAXW];
    int32_t hcount;   // visited vertices
    int32_t nexp;     // expansions
    int32_t mode;     // 0: visited set in LDS, 1: in the workspace
    int32_t flags;
    int32_t nslot;    // workspace-table slots written (zeroed again at the end)
    int32_t slen, substeps, steps, epoch, stop;   // handed over by the one active worker
    int32_t job;      // persistent form: the job the workgroup runs next
};

struct MultiLds {
    uint32_t o_key, o_pub, o_stage, o_un, o_ids, o_mark, o_ctrl, o_q, o_hash, total;   // o_key: S, S'
};

__host__ __device__ inline MultiLds multi_lds(int L, int M, int lpv, int llog2)
{
    MultiLds Y;
    const uint32_t Lp = (uint32_t)(L + 63) / 64 * 64;
    uint32_t o = 0;
    Y.o_key = o; o += 8u * 2u * Lp;
    Y.o_pub = o; o += 8u * pub_room(L, M);
    Y.o_stage = o; o += 8u * 66u * M;   // a worker's new keys, then its insert
    Y.o_un = o; o += 8u * 16u;
    Y.o_ids = o; o += 4u * 64u * M;
    Y.o_mark = o; o += 4u * 32u;
    Y.o_ctrl = o; o += (uint32_t)(sizeof(Ctrl) + 15) / 16 * 16;
    Y.o_q = o; o += 64u * (uint32_t)lpv;
    Y.o_hash = o; o += llog2 > 0 ? 8u << llog2 : 0u;
    Y.total = o;
    return Y;
}

__device__ __forceinline__ uint32_t hash_slot(uint32_t id, int log2cap)
{
    return (id * 2654435761u) >> (32 - log2cap);
}

// Phase one of a claim: find or insert u, leaving the smallest tag of this local step
// in its slot.  Returns the slot, or NO_SLOT if the table is full; *fresh tells whether
// this call inserted u.
__device__ __forceinline__ uint32_t visit_claim(unsigned long long *H, int log2cap, uint32_t u, uint32_t tag,
                                                uint32_t epoch, bool *fresh)
{
    const uint32_t mask = (1u << log2cap) - 1u;
    uint32_t s = hash_slot(u, log2cap);
    const unsigned long long want = ((unsigned long long)(u + 1) << 32) | tag;
    *fresh = false;
    for (uint32_t probe = 0; probe <= mask; ++probe) {
        unsigned long long old = atomicCAS(&H[s], 0ull, want);
        if (old == 0ull) {
            *fresh = true;
            return s;
        }
        if ((uint32_t)(old >> 32) == u + 1) {
            if (((uint32_t)old >> 10) == epoch) atomicMin(&H[s], want);
            return s;
        }
        s = (s + 1) & mask;
    }
    return NO_SLOT;
}

__device__ __forceinline__ unsigned long long read_slot_global(unsigned long long *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Records workspace slots written by fresh claims of this wave (prefix over the wave,
// then one reservation) so they can be zeroed at the end of the query.
__device__ __forceinline__ void record_slots(bool rec, uint32_t slot, int32_t *base_counter, uint32_t *slots)
{
    const uint64_t b = __ballot(rec);
    if (!b) return;
    int base = 0;
    if (__lane_id() == 0) base = atomicAdd(base_counter, __popcll(b));
    base = __builtin_amdgcn_readfirstlane(base);
    if (rec) slots[base + bits_below(b)] = slot;
}

// Moves the LDS visited table into the (zero-filled) workspace table.
__device__ __forceinline__ void migrate_table(const unsigned long long *lh, int llog2, unsigned long long *gh,
                                              int glog2, uint32_t *gslots, int32_t *nslot, int tid, int nthr)
{
    const uint32_t gm = (1u << glog2) - 1u;
    for (int base = 0; base < (1 << llog2); base += nthr) {
        const int i = base + tid;
        bool rec = false;
        uint32_t s = 0;
        if (i < (1 << llog2)) {
            const unsigned long long h = lh[i];
            if (h != 0ull) {
                s = hash_slot((uint32_t)(h >> 32) - 1u, glog2);
                while (atomicCAS(&gh[s], 0ull, h) != 0ull) s = (s + 1) & gm;
                rec = true;
            }
        }
        record_slots(rec, s, nslot, gslots);
    }
}

// Entries of the sorted S (slen of them, nslots slots) below e, which all lanes hold.
__device__ __forceinline__ int count_below(const uint64_t *S, int slen, int nslots, uint64_t e)
{
    const int lane = __lane_id();
    const int i = lane * nslots + nslots - 1;
    const int base = nslots * __popcll(__ballot(i < slen && S[i < slen ? i : 0] < e));
    const int j = base + lane;
    const bool in = lane < nslots && j < slen;
    return base + __popcll(__ballot(in && S[in ? j : 0] < e));
}

// What a worker may expand between two merges: its share of S (bit masks, entry j in bit
// j % 64 of mask j / 64) and its own new entries, unordered, entry p in lane p % 64 of slot
// p / 64 (KEY_EMPTY past the end), with masks of the unchecked ones.  One slot more than
// S has, so that a step's entries fit when those that fell out are dropped.
template <int NI>
struct Worker {
    uint64_t share[NI];
    uint64_t k[NI + 1], un[NI + 1];
    int len;
};

// Calls f with the slots in use.
template <int N, int I = 0, typename F>
__device__ __forceinline__ void slots_used(int len, F f)
{
    if constexpr (I < N) {
        if (64 * I < len) {
            f(std::integral_constant<int, I>{});
            slots_used<N, I + 1>(len, f);
        }
    }
}

template <int NI>
__device__ __forceinline__ int own_below(const Worker<NI> &W, uint64_t key)
{
    int c = 0;
    slots_used<NI + 1>(W.len, [&](auto i) { c += __popcll(__ballot(W.k[i] < key)); });
    return c;
}

// Appends the keys of the lanes in b, unchecked where the lane's flag says so.  stage: 64 keys.
template <int NI>
__device__ __forceinline__ void append(Worker<NI> &W, uint64_t key, uint64_t b, bool unchecked, uint64_t *stage)
{
    const int lane = __lane_id(), cnt = __popcll(b), at = W.len & 63;
    if ((b >> lane) & 1ull) stage[(W.len + bits_below(b)) & 63] = key | (unchecked ? 0x80000000ull : 0ull);
    __builtin_amdgcn_wave_barrier();
    const uint64_t v = stage[lane];
    __builtin_amdgcn_wave_barrier();
    // (every slot each time: stores in the branch of their slot would be merged into one store
    // through a pointer, and the slots put into scratch memory)
    const int first = W.len >> 6;
#pragma unroll
    for (int i = 0; i <= NI; ++i) {
        const int p = 64 * (i - first) + lane;
        const bool here = p >= at && p < at + cnt;
        W.un[i] |= __ballot(here && ((uint32_t)v >> 31) != 0u);
        W.k[i] = here ? v & ~0x80000000ull : W.k[i];
    }
    W.len += cnt;
}

// A bound t such that entries whose distance bits are t or more have fallen out of the first L
// of the local queue: the smallest that has L entries below it (all ones if there is none).
template <int NI>
__device__ __forceinline__ uint32_t fallen_from(const Worker<NI> &W, const uint64_t *S, int slen, int nslots, int L)
{
    uint32_t t = 0;   // the largest with fewer than L entries below it
    for (uint32_t bit = 0x80000000u; bit; bit >>= 1) {
        const uint64_t e = (uint64_t)(t | bit) << 32;
        if (own_below(W, e) + count_below(S, slen, nslots, e) < L) t |= bit;
    }
    return t == 0xFFFFFFFFu ? t : t + 1u;
}

// Drops the own entries whose distance bits are at least t; EXACT: those that have fallen out
// of the first L of the local queue.  Slot by slot in place.  (Places are counted among the
// entries kept and those to come: an entry with L smaller ones still has L smaller ones
// then, as the L smallest of all are kept.)
template <int NI, bool EXACT>
__device__ __forceinline__ void drop_dead(Worker<NI> &W, const uint64_t *S, int slen, int L, uint32_t t,
                                          uint64_t *stage)
{
    const int lane = __lane_id(), old = W.len;
    W.len = 0;
    for (int i = 0; 64 * i < old; ++i) {
        uint64_t key = KEY_EMPTY, un = 0;
#pragma unroll
        for (int c = 0; c <= NI; ++c) {
            key = c == i ? W.k[c] : key;
            un = c == i ? W.un[c] : un;
        }
        bool keep = 64 * i + lane < old && (uint32_t)(key >> 32) < t;
        if constexpr (EXACT) {
            int r = lower_bound(S, slen, entry_of(key, 1u));
            for (int j = 0; 64 * j < old; ++j) {
                uint64_t other = KEY_EMPTY;
#pragma unroll
                for (int c = 0; c <= NI; ++c) other = c == j ? W.k[c] : other;
                for (int l = 0; l < 64; ++l) r += rdlane64(other, l) < key ? 1 : 0;
            }
            keep = keep && r < L;
        }
#pragma unroll
        for (int c = 0; c <= NI; ++c) {
            W.k[c] = c == i ? KEY_EMPTY : W.k[c];
            W.un[c] = c == i ? 0ull : W.un[c];
        }
        const uint64_t alive = __ballot(keep);
        if (alive) append(W, key, alive, __builtin_amdgcn_inverse_ballot_w64(un), stage);
    }
}

struct Pick {
    int32_t v;     // the vertex, -1: none
    int32_t at;    // its place in S or among the own entries
    bool own;
};

// The first entry worker W may expand, if it is among the first L of the local queue.
// S: slen entries.
template <int NI>
__device__ __forceinline__ Pick pick_next(const Worker<NI> &W, const uint64_t *S, int slen, int L)
{
    int js = -1;
#pragma unroll
    for (int i = NI - 1; i >= 0; --i)
        if (W.share[i] != 0ull) js = 64 * i + __builtin_ctzll(W.share[i]);
    const uint64_t es = js >= 0 ? rdlane64(S[js], 0) : ~0ull;
    // the smallest unchecked own entry
    uint64_t mine = KEY_EMPTY;
    int slot = 0;   // of this lane's
    slots_used<NI + 1>(W.len, [&](auto i) {
        const uint64_t c = __builtin_amdgcn_inverse_ballot_w64(W.un[i]) ? W.k[i] : KEY_EMPTY;
        slot = c < mine ? (int)i : slot;
        mine = c < mine ? c : mine;
    });
    uint64_t ko = KEY_EMPTY;
    int lo = 0;
    if (W.len > 0) ko = min_key(mine, &lo);
    const uint64_t eo = ko != KEY_EMPTY ? entry_of(ko, 1u) : ~0ull;
    if (es < eo) {   // (different vertices: the flags do not decide)
        // it has fallen out if L - js or more own entries are below it
        if (js + W.len >= L && js + own_below(W, key_of(es)) >= L) return {-1, 0, false};
        return {entry_id(es), js, false};
    }
    if (ko == KEY_EMPTY) return {-1, 0, false};
    const int c = L - 1 - own_below(W, ko);   // at most c entries of S may be below it
    if (c < 0 || (c < slen && rdlane64(S[c], 0) < eo)) return {-1, 0, false};
    return {key_id(ko), 64 * (int)rdlane((uint32_t)slot, lo) + lo, true};
}

// Takes a picked entry out of the masks.
template <int NI>
__device__ __forceinline__ void take(Worker<NI> &W, const Pick &p)
{
    const uint64_t bit = 1ull << (p.at & 63);
    // (both masks each time: a choice between them would put them into scratch memory)
#pragma unroll
    for (int i = 0; i < NI; ++i) W.share[i] &= ~((p.at >> 6) == i && !p.own ? bit : 0ull);
#pragma unroll
    for (int i = 0; i <= NI; ++i) W.un[i] &= ~((p.at >> 6) == i && p.own ? bit : 0ull);
}

// Job `job` runs query order[job] (or job) in workspace region `region`.
// PBMAX: vectors per lane group in flight in a gather pass
template <int LPV, int NI, int DT, int PBMAX>
__device__ __forceinline__ void multi_body(const KArgs &A, int64_t job, int64_t region)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr int PB = PBMAX < LPV / 2 ? PBMAX : (LPV >= 2 ? LPV / 2 : 1);   // at most 32 in all
    const int tid = threadIdx.x, lane = __lane_id(), nthr = blockDim.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t qi = A.order ? __builtin_amdgcn_readfirstlane(A.order[job]) : job;
    const int L = A.qL ? __builtin_amdgcn_readfirstlane(A.qL[qi]) : A.L, M = A.M, R = A.R;
    const int kq = A.qk ? __builtin_amdgcn_readfirstlane(A.qk[qi]) : A.k;
    const int nslots = (L + 63) >> 6;

    const MultiLds Y = multi_lds(A.L, M, LPV, A.llog2);
    uint64_t *S = reinterpret_cast<uint64_t *>(smem + Y.o_key);
    uint64_t *Sn = S + (A.L + 63) / 64 * 64;
    uint64_t *const pub = reinterpret_cast<uint64_t *>(smem + Y.o_pub);            // [pub_room]
    uint64_t *const stage = reinterpret_cast<uint64_t *>(smem + Y.o_stage) + 66 * w;
    uint64_t *const un = reinterpret_cast<uint64_t *>(smem + Y.o_un);              // [16] unchecked entries of S
    int32_t *const claimed_ids = reinterpret_cast<int32_t *>(smem + Y.o_ids) + 64 * w;
    uint32_t *const mark = reinterpret_cast<uint32_t *>(smem + Y.o_mark);          // [32]
    Ctrl *const C = reinterpret_cast<Ctrl *>(smem + Y.o_ctrl);
    float *const qs = reinterpret_cast<float *>(smem + Y.o_q);
    unsigned long long *const lh = reinterpret_cast<unsigned long long *>(smem + Y.o_hash);
    unsigned long long *const gh = A.ghash + ((size_t)region << (A.glog2 + 1));
    uint32_t *const gslots = reinterpret_cast<uint32_t *>(gh + (1ull << A.glog2));

    const uint64_t t_start = __builtin_amdgcn_s_memrealtime();
    const int llog2 = A.llog2, glog2 = A.glog2;
    const bool l2 = A.metric == SA_L2;
    const VecSrc V{A.codes, A.scale, A.ldc};
    const int32_t n = (int32_t)A.n;
    // this lane's entry of an adjacency row (R <= 64); lanes past R load entry 0 and drop it
    const int32_t *const adj_lane = A.adj + (lane < R ? lane : 0);
    const auto measure = [&](int cnt) {
        if (l2) distances<LPV, true, DT, ACC_F64, PB, true>(V, A.d, qs, claimed_ids, cnt, stage);
        else distances<LPV, false, DT, ACC_F64, PB, true>(V, A.d, qs, claimed_ids, cnt, stage);
    };

    if (llog2 > 0)
        for (int i = tid; i < (1 << llog2); i += nthr) lh[i] = 0ull;
    claimed_ids[lane] = A.entry;   // (a pass of the distances reads ids past the last)
    if (tid < 16) un[tid] = 0ull;
    if (tid < MAXW) C->nnew[tid] = C->work[tid] = C->U[tid] = 0;
    if (tid == 0) {
        C->hcount = 1;
        C->nexp = C->flags = C->nslot = C->stop = 0;
        C->mode = llog2 > 0 ? 0 : 1;
    }
    {
        const float *const qrow = A.queries + qi * A.ldq;
        const int nch = A.d >> 2;
        for (int c = tid; c < 4 * LPV; c += nthr)
            reinterpret_cast<float4 *>(qs)[c] =
                c < nch ? *reinterpret_cast<const float4 *>(qrow + 4 * c) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    __syncthreads();
    // the start point: its distance, the list holding only it, and the visited set
    if (w == 0) {
        measure(1);
        __builtin_amdgcn_wave_barrier();
        bool fresh = false;
        uint32_t s0 = 0;
        if (lane == 0) {
            S[0] = entry_of(stage[0], 1u);
            un[0] = 1ull;
            s0 = llog2 > 0 ? visit_claim(lh, llog2, (uint32_t)A.entry, 0u, 0u, &fresh)
                           : visit_claim(gh, glog2, (uint32_t)A.entry, 0u, 0u, &fresh);
        }
        if (llog2 == 0) record_slots(lane == 0, s0, &C->nslot, gslots);
    }
    __syncthreads();

    // Algorithm 2's test: the mean update position against L rho
    const double l_rho = (double)L * A.rho;
    int slen = 1, substeps = 0, gsteps = 0, merges = 0;
    uint32_t epoch = 1;
    int m = A.staged ? 1 : M;
    int32_t pv = -1, pu = -1;   // vertex whose adjacency row is read ahead, and this lane's entry of it
    // ------------------------------------------------------------ one active worker
    // The merge of one local queue into S leaves S equal to the queue: wavefront 0 keeps it in
    // registers (search_queue.h) and writes S when the next worker joins, or at the end.
    if (m == 1) {
        if (w == 0) {
            Queue<NI> Q;
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                Q.k[i] = KEY_EMPTY;
                Q.un[i] = 0ull;
            }
            if (lane == 0) Q.k[0] = key_of(S[0]);
            Q.un[0] = 1ull;
            Q.top = KEY_EMPTY;
            Q.len = 1;
            __builtin_amdgcn_wave_barrier();
            uint64_t worst = L == 1 ? get_key(Q, 0) : KEY_EMPTY;   // the last key of a full queue
            int hcount = 1, nexp = 0, flags = 0, mode = llog2 > 0 ? 0 : 1;
            bool stop = false;
            while (any_unchecked(Q) && !stop) {
                gsteps++;
                int sub_in_step = 0;
                for (;;) {
                    if (substeps >= A.max_substeps) {
                        flags |= SA_QFLAG_MAX_STEPS;
                        stop = true;
                        break;
                    }
                    substeps++;
                    sub_in_step++;
                    nexp++;
                    const int32_t v = take_first(Q.k, Q.un);
                    int32_t u = pu;
                    if (v != pv) u = adj_lane[(int64_t)v * R];
                    // read the row of the next candidate while this step runs
                    {
                        uint64_t ahead[NI];
#pragma unroll
                        for (int i = 0; i < NI; ++i) ahead[i] = Q.un[i];
                        const int32_t a = take_first(Q.k, ahead);
                        pv = a >= 0 ? a : v;
                        pu = adj_lane[(int64_t)pv * R];
                    }
                    if (lane >= R || u < 0 || u >= n) u = -1;   // padding and malformed entries
                    bool fresh = false;
                    uint32_t slot = NO_SLOT;
                    const uint32_t tag = (epoch << 10) | (uint32_t)lane;
                    if (u >= 0) slot = mode ? visit_claim(gh, glog2, (uint32_t)u, tag, epoch, &fresh)
                                            : visit_claim(lh, llog2, (uint32_t)u, tag, epoch, &fresh);
                    if (mode) record_slots(fresh, slot, &C->nslot, gslots);
                    const uint64_t cm = __ballot(fresh);
                    const int nclaim = __popcll(cm);
                    hcount += nclaim;
                    if (fresh) claimed_ids[bits_below(cm)] = u;
                    __builtin_amdgcn_wave_barrier();
                    measure(nclaim);
                    __builtin_amdgcn_wave_barrier();
                    const uint64_t mk = lane < nclaim ? stage[lane] : KEY_EMPTY;
                    __builtin_amdgcn_wave_barrier();
                    const uint64_t sbits = __ballot(mk < worst);
                    int U = L;
                    if (sbits) {
                        // (S, the next S and the published keys follow each other and are idle:
                        // more than 64 NI keys)
                        U = insert_batch<NI, true>(Q, L, mk, sbits, S);
                        if (Q.len == L) worst = get_key(Q, L - 1);
                    }
                    epoch++;
                    // keep the visited set below half (LDS) / three quarters (workspace)
                    const int need = hcount + R;
                    if (mode == 0 && need > (1 << llog2) / 2) {
                        if (need > (3 << glog2) / 4) {
                            flags |= SA_QFLAG_CAPACITY;
                            stop = true;
                            break;
                        }
                        migrate_table(lh, llog2, gh, glog2, gslots, &C->nslot, lane, 64);
                        mode = 1;
                        flags |= SA_QFLAG_SPILLED;
                    } else if (mode == 1 && need > (3 << glog2) / 4) {
                        flags |= SA_QFLAG_CAPACITY;
                        stop = true;
                        break;
                    }
                    bool merge_now;
                    if (A.sync == SA_SYNC_BSP) merge_now = true;
                    else if (A.sync == SA_SYNC_STATIC) merge_now = A.static_I > 0 && sub_in_step >= A.static_I;
                    else merge_now = (double)U >= l_rho;
                    if (!any_unchecked(Q) || merge_now) break;
                }
                merges++;   // S becomes this queue unchanged
                if (M > 1) break;
            }
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                if (64 * i + lane < Q.len)
                    S[64 * i + lane] = entry_of(Q.k[i], __builtin_amdgcn_inverse_ballot_w64(Q.un[i]) ? 1u : 0u);
                if (lane == 0) un[i] = Q.un[i];
            }
            if (lane == 0) {
                C->slen = Q.len;
                C->hcount = hcount;
                C->nexp = nexp;
                C->flags = flags;
                C->mode = mode;
                C->substeps = substeps;
                C->steps = gsteps;   // and merges
                C->epoch = (int32_t)epoch;
                C->stop = stop ? 1 : 0;
            }
        }
        __syncthreads();
        slen = __builtin_amdgcn_readfirstlane(C->slen);
        substeps = __builtin_amdgcn_readfirstlane(C->substeps);
        gsteps = merges = __builtin_amdgcn_readfirstlane(C->steps);
        epoch = (uint32_t)__builtin_amdgcn_readfirstlane(C->epoch);
        m = 2;
        pv = -1;
    }

    // ------------------------------------------------------------ two or more workers
    const bool ended = M < 2 || __builtin_amdgcn_readfirstlane(C->stop) != 0;
    while (!ended) {
        // divide the unchecked entries of S among the m workers: the j-th unchecked entry
        // belongs to worker j mod m
        Worker<NI> W;
        const uint64_t um = lane < nslots ? un[lane] : 0ull;
        const int here = __popcll(um);
        int upto = here;   // unchecked entries up to and including this lane's slot
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) {
            const int v = __shfl_up(upto, o, 64);
            if (lane >= o) upto += v;
        }
        if (__builtin_amdgcn_readlane(upto, 15) == 0) break;
        gsteps++;
        const uint32_t inv = 65536u / (uint32_t)m + 1u;   // r / m = r inv >> 16 for r < 1024, m <= 16
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const uint64_t b = rdlane64(um, i);
            const uint32_t r = (uint32_t)(__builtin_amdgcn_readlane(upto - here, i) + bits_below(b));
            const uint32_t t = r - (r * inv >> 16) * (uint32_t)m;
            W.share[i] = b & __ballot(t == (uint32_t)w);
            if (w >= m) W.share[i] = 0ull;
        }
#pragma unroll
        for (int i = 0; i <= NI; ++i) {
            W.k[i] = KEY_EMPTY;
            W.un[i] = 0ull;
        }
        W.len = 0;
        if (tid < 32) mark[tid] = 0u;
        // (entries that a worker may still add must beat the last of a full S)
        const uint64_t worst = slen == L ? S[L - 1] : ~0ull;
        bool stop = false;
        uint32_t fallen = 0xFFFFFFFFu;   // entries of at least these distance bits have fallen out
        {
            int sub_in_step = 0;
            Pick next = pick_next(W, S, slen, L);
            for (;;) {
                if (substeps >= A.max_substeps) {
                    if (tid == 0) C->flags |= SA_QFLAG_MAX_STEPS;
                    stop = true;
                    break;
                }
                substeps++;
                sub_in_step++;
                const int mode = C->mode;
                const bool has = next.v >= 0;
                const uint32_t tag = (epoch << 10) | ((uint32_t)w << 6) | (uint32_t)lane;
                int32_t u = -1;
                uint32_t slot = NO_SLOT;
                bool fresh = false;
                if (has) {
                    const int32_t v = next.v;
                    if (lane == 0) {
                        // checked from now on
                        if (!next.own) reinterpret_cast<uint32_t *>(S + next.at)[0] = (uint32_t)v << 1;
                        atomicAdd(&C->nexp, 1);
                    }
                    take(W, next);
                    u = pu;
                    if (v != pv) u = adj_lane[(int64_t)v * R];
                    {
                        const Pick a = pick_next(W, S, slen, L);
                        pv = a.v >= 0 ? a.v : v;
                        pu = adj_lane[(int64_t)pv * R];
                    }
                    if (lane >= R || u < 0 || u >= n) u = -1;   // padding and malformed entries
                    if (u >= 0) slot = mode ? visit_claim(gh, glog2, (uint32_t)u, tag, epoch, &fresh)
                                            : visit_claim(lh, llog2, (uint32_t)u, tag, epoch, &fresh);
                }
                __syncthreads();
                int U = L;
                if (has) {
                    bool claimed = false;
                    if (slot != NO_SLOT) {
                        unsigned long long h = mode ? read_slot_global(gh + slot) : lh[slot];
                        claimed = (uint32_t)h == tag;
                    }
                    // the visited count changes only between the two barriers of a local
                    // step, so every wave reads the same value in the decision below
                    const int nfresh = __popcll(__ballot(fresh));
                    if (lane == 0 && nfresh) atomicAdd(&C->hcount, nfresh);
                    if (mode) record_slots(fresh, slot, &C->nslot, gslots);
                    const uint64_t cm = __ballot(claimed);
                    const int nclaim = __popcll(cm);
                    if (claimed) claimed_ids[bits_below(cm)] = u;
                    __builtin_amdgcn_wave_barrier();
                    measure(nclaim);
                    __builtin_amdgcn_wave_barrier();
                    const uint64_t mk = lane < nclaim ? stage[lane] : KEY_EMPTY;
                    __builtin_amdgcn_wave_barrier();
                    uint64_t sbits = __ballot(lane < nclaim && entry_of(mk, 1u) < worst);
                    if (sbits) {
                        // the update position: where the best of them lands in the local queue
                        int at;
                        const uint64_t best = min_key((sbits >> lane) & 1ull ? mk : KEY_EMPTY, &at);
                        U = min(L, own_below(W, best) + count_below(S, slen, nslots, entry_of(best, 1u)));
                        if (U < L) {
                            sbits &= __ballot((uint32_t)(mk >> 32) < fallen);
                            if (W.len + __popcll(sbits) > 64 * (NI + 1)) {
                                // make room: by the distances first, and exactly if entries at one
                                // distance leave too many
                                fallen = fallen_from(W, S, slen, nslots, L);
                                drop_dead<NI, false>(W, S, slen, L, fallen, stage);
                                sbits &= __ballot((uint32_t)(mk >> 32) < fallen);
                                if (W.len + __popcll(sbits) > 64 * (NI + 1))
                                    drop_dead<NI, true>(W, S, slen, L, fallen, stage);
                            }
                            append(W, mk, sbits, true, stage);
                        }
                    }
                    next = pick_next(W, S, slen, L);
                }
                if (lane == 0) {
                    C->U[w] = U;
                    C->work[w] = next.v >= 0;
                }
                epoch++;
                __syncthreads();
                // lane t reads worker t's flag and update position
                const bool any = __ballot(lane < m && C->work[lane & 15] != 0) != 0;
                int sumU = lane < m ? C->U[lane & 15] : 0;
#pragma unroll
                for (int off = 8; off > 0; off >>= 1) sumU += __shfl_xor(sumU, off, 64);
                sumU = __builtin_amdgcn_readfirstlane(sumU);
                bool merge_now;
                if (A.sync == SA_SYNC_STATIC) merge_now = A.static_I > 0 && sub_in_step >= A.static_I;
                else merge_now = (double)sumU / (double)m >= l_rho;
                // keep the visited set below half (LDS) / three quarters (workspace) before
                // the next local step, which adds at most m * R entries
                const int need = __builtin_amdgcn_readfirstlane(C->hcount) + m * R;
                if (mode == 0 && need > (1 << llog2) / 2) {
                    if (need > (3 << glog2) / 4) {
                        if (tid == 0) C->flags |= SA_QFLAG_CAPACITY;
                        stop = true;
                        break;
                    }
                    migrate_table(lh, llog2, gh, glog2, gslots, &C->nslot, tid, nthr);
                    __syncthreads();
                    if (tid == 0) {
                        C->mode = 1;
                        C->flags |= SA_QFLAG_SPILLED;
                    }
                    __syncthreads();
                } else if (mode == 1 && need > (3 << glog2) / 4) {
                    if (tid == 0) C->flags |= SA_QFLAG_CAPACITY;
                    stop = true;
                    break;
                }
                if (!any || merge_now) break;
            }
        }

        // ---- merge
        if (lane == 0) C->nnew[w] = W.len;
        __syncthreads();
        const int mine = lane < M ? C->nnew[lane & 15] : 0;
        int first = mine;   // published before worker `lane`, and its own
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) {
            const int v = __shfl_up(first, o, 64);
            if (lane >= o) first += v;
        }
        const int total_new = __builtin_amdgcn_readlane(first, 15);
        const int own_first = __builtin_amdgcn_readlane(first - mine, w);
        const auto place = [&](uint64_t key, int r, bool unchecked) {
            if (r < L) {
                Sn[r] = entry_of(key, unchecked ? 1u : 0u);
                atomicOr(&mark[r >> 5], 1u << (r & 31));
            }
        };
        if (total_new <= PUBCAP) {
            // all at once: p lanes count for one key
            slots_used<NI + 1>(W.len, [&](auto i) {
                if (64 * i + lane < W.len)
                    pub[own_first + 64 * i + lane] =
                        entry_of(W.k[i], __builtin_amdgcn_inverse_ballot_w64(W.un[i]) ? 1u : 0u);
            });
            __syncthreads();
            int lp = 0;   // log2 p
            while (lp < 4 && (total_new << (lp + 1)) <= nthr) ++lp;
            const int p = 1 << lp;
            for (int i = tid >> lp; i < total_new; i += nthr >> lp) {
                const uint64_t e = pub[i];
                const int part = tid & (p - 1);
                int r = part == 0 ? lower_bound(S, slen, e) : 0;
#pragma unroll 4
                for (int j = part; j < total_new; j += p) r += pub[j] < e ? 1 : 0;
                // sum into the last lane of the group
                if (p > 1) r += (int)row_shr0<1>((uint32_t)r);
                if (p > 2) r += (int)row_shr0<2>((uint32_t)r);
                if (p > 4) r += (int)row_shr0<4>((uint32_t)r);
                if (p > 8) r += (int)row_shr0<8>((uint32_t)r);
                if (part == p - 1) place(key_of(e), r, e & 1ull);
            }
        } else {
            // PUBCAP at a time: every worker counts for its own
            int rk[NI + 1];
#pragma unroll
            for (int i = 0; i <= NI; ++i) rk[i] = 0;
            slots_used<NI + 1>(W.len, [&](auto i) { rk[i] = lower_bound(S, slen, entry_of(W.k[i], 1u)); });
            for (int c0 = 0; c0 < total_new; c0 += PUBCAP) {
                const int cn = min(PUBCAP, total_new - c0);
                if (c0 > 0) __syncthreads();
                slots_used<NI + 1>(W.len, [&](auto i) {
                    const int g = own_first + 64 * i + lane - c0;
                    if (64 * i + lane < W.len && g >= 0 && g < cn) pub[g] = W.k[i];
                });
                __syncthreads();
                slots_used<NI + 1>(W.len, [&](auto i) {
                    const uint64_t key = W.k[i];
                    int below = 0;
                    for (int j = 0; j < cn; ++j) below += pub[j] < key ? 1 : 0;
                    rk[i] += below;
                });
            }
            slots_used<NI + 1>(W.len, [&](auto i) {
                if (64 * i + lane < W.len) place(W.k[i], rk[i], __builtin_amdgcn_inverse_ballot_w64(W.un[i]));
            });
        }
        __syncthreads();
        const int nlen = min(L, slen + total_new);
        for (int s = w; s < nslots; s += M) {
            const uint32_t mw = lane < 32 ? mark[lane] : 0u;
            const uint64_t taken = ((uint64_t)rdlane(mw, 2 * s + 1) << 32) | rdlane(mw, 2 * s);
            int below = lane < 2 * s ? __popc(mw) : 0;   // marks in the slots below
#pragma unroll
            for (int o = 16; o > 0; o >>= 1) below += __shfl_xor(below, o, 64);
            below = __builtin_amdgcn_readfirstlane(below);
            const int P = 64 * s + lane;
            const bool marked = __builtin_amdgcn_inverse_ballot_w64(taken);
            const bool from = !marked && P < nlen;
            const uint64_t e = from ? S[P - below - bits_below(taken)] : 0ull;
            if (from) Sn[P] = e;
            const uint64_t f = marked ? Sn[P] : e;   // (written before the barrier)
            const uint64_t b = __ballot(P < nlen && (f & 1ull));
            if (lane == 0) un[s] = b;
        }
        uint64_t *const t = S;
        S = Sn;
        Sn = t;
        slen = nlen;
        merges++;
        if (A.staged && m < M) m = min(2 * m, M);
        __syncthreads();
        if (stop) break;   // a step limit or a full visited table ends the search after this merge
    }

    if (A.rerank != 0) {
        // hand the first nr entries of the final list to the re-rank kernel
        const int nr = A.rerank < 0 ? slen : min(A.rerank, slen);
        int32_t *const list = rerank_list(gslots, glog2);
        for (int i = tid; i < nr; i += nthr) list[1 + i] = entry_id(S[i]);
        if (tid == 0) list[0] = nr;
    } else {
        for (int i = tid; i < kq; i += nthr) {
            const bool ok = i < slen;
            A.ids[qi * A.ldo + i] = ok ? entry_id(S[i]) : -1;
            A.dists[qi * A.ldo + i] = ok ? key_dist(S[i]) : __builtin_inff();
        }
    }
    // leave the workspace table zero-filled for the next launch
    const int ns = C->nslot;
    for (int i = tid; i < ns; i += nthr) {
        const uint32_t sl = gslots[i];
        gh[sl] = 0ull;
        gslots[i] = 0u;
    }
    if (tid == 0 && A.stats) {
        sa_query_stats st;
        st.global_steps = gsteps;
        st.substeps = substeps;
        st.expansions = C->nexp;
        st.dist_comps = C->hcount;
        st.merges = merges;
        st.flags = C->flags;
        st.t_start = t_start;
        st.t_end = __builtin_amdgcn_s_memrealtime();
        A.stats[qi] = st;
    }
}

// Workgroup b runs job b in workspace region b.  WAVES: wavefronts that a SIMD can hold, which
// bounds the registers (five: up to four workers only, two or three: up to eight); PB: vectors per lane group in
// flight in a gather pass.
template <int LPV, int NI, int DT, int WAVES, int PB>
__global__ void __launch_bounds__(WAVES == 5 ? 256 : WAVES <= 3 ? 512 : 1024) __attribute__((amdgpu_waves_per_eu(WAVES)))
search_multi(KArgs A)
{
    multi_body<LPV, NI, DT, PB>(A, blockIdx.x, blockIdx.x);
}

// Persistent form: each resident workgroup takes jobs from the device counter until none
// is left, every one in its own workspace region (see KArgs::jobctr).
template <int LPV, int NI, int DT>
__global__ void __launch_bounds__(1024) search_multi_loop(KArgs A)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    Ctrl *const C = reinterpret_cast<Ctrl *>(smem + multi_lds(A.L, A.M, LPV, A.llog2).o_ctrl);
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) C->job = atomicAdd(A.jobctr, 1);
        __syncthreads();
        const int job = __builtin_amdgcn_readfirstlane(C->job);
        if (job >= A.njobs) break;
        multi_body<LPV, NI, DT, 1>(A, job, blockIdx.x);
    }
    __syncthreads();
    if (threadIdx.x == 0) release_jobs(A.jobctr);
}

// A kernel of a launch and how many of its queries the device can hold at once.
struct MultiForm {
    const void *k;
    int64_t slots;
};

// Raises the dynamic LDS limit of kernel k to the whole 160 KB, once per kernel and device, not
// on every launch (the latency path launches one query at a time), and asks for its slots.
inline hipError_t multi_form(const void *k, std::atomic<uint64_t> &raised, const KArgs &A, uint32_t lds, MultiForm *f)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = 1ull << (dev & 63);
    if (!(raised.load(std::memory_order_acquire) & bit)) {
        e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        raised.fetch_or(bit, std::memory_order_acq_rel);
    }
    f->k = k;
    // (beyond four wavefronts a workgroup takes as many of each SIMD as of its fullest: at three
    // waves per SIMD a CU holds one workgroup of five, not two)
    return resident_grid(k, A.M <= 4 ? 64 * A.M : (A.M + 3) / 4 * 256, lds, INT32_MAX, &f->slots);
}

// The form of a launch.  Fewer registers let more queries run at once, and make each slower.
//   Up to four workers: three waves per SIMD (at 64 < L <= 128 the compiler stays at that when
// allowed two, and is 1-4% faster), unless the launch takes fewer rounds of the chip at five (at
// L <= 64: four, or five).
// That is so for two workers, who have no LDS table; with more, the table leaves a CU three or
// four queries either way.  200K x 128, adaptive, us at 2 / 3 / 5 waves: two workers, L = 192,
// 1,000 queries 1,192 / 1,164 / 1,220, 2,500 2,398 / 1,833 / 1,519, 10,000 6,696 / 4,912 / 3,928;
// four workers, L = 192, 1,000 queries 955 / 907 / 960, 10,000 7,252 / 5,010 / 5,291.  (Two waves
// whatever the launch had cost full batches of up to four workers a tenth to a third.)
//   Five to eight workers take those registers while all queries are then resident at once, and
// four waves beyond; more workers four waves while resident and eight beyond.  Where the LDS of a
// query (its visited table at large L) leaves room for one workgroup per CU anyway, fewer
// registers gain nothing.  1,000 queries, L = 128: 8 workers 850 (3 waves), 539 (4), 673 (8);
// 16 workers 1,054 (4), 966 (8).
//   Two waves, with eight vectors in flight, only while all queries are resident, at L > 384 or
// d > 256: 33 queries, four workers, L = 768 2,147 (2) against 2,260 (3); 300 of d = 960, L = 64
// 241 against 250.
//   Four waves with two vectors in flight spill five to ten registers at L <= 256 (25 at 512);
// with one none, but eight workers at L = 64 are 9% slower then (704 / 780 us).
template <int LPV, int NI, int DT>
hipError_t launch_multi(const KArgs &A, int64_t nq, hipStream_t s)
{
    static std::atomic<uint64_t> raised[6] = {{0}, {0}, {0}, {0}, {0}, {0}};
    const uint32_t lds = multi_lds(A.L, A.M, LPV, A.llog2).total;
    const int64_t all = nq + A.company;
    const auto form = [&](auto k, int i, MultiForm *f) {
        return multi_form(reinterpret_cast<const void *>(k), raised[i], A, lds, f);
    };
    const auto launch = [&](const MultiForm &f, int64_t grid) {
        KArgs B = A;
        void *args[] = {&B};
        return hipLaunchKernel(f.k, dim3((unsigned)grid), dim3(64 * A.M), args, lds, s);
    };
    constexpr bool TWO = LPV >= 32 || NI >= 8;
    const bool one_a_cu = lds > 80u * 1024u;
    MultiForm f, g;
    hipError_t e;
    if (A.jobctr) {
        e = form(search_multi_loop<LPV, NI, DT>, 0, &f);
        return e == hipSuccess ? launch(f, std::min(nq, f.slots)) : e;
    }
    if constexpr (TWO) {
        if (A.M <= 8) {
            e = form(search_multi<LPV, NI, DT, 2, 8>, 1, &f);
            if (e != hipSuccess) return e;
            if (all <= f.slots || one_a_cu) return launch(f, nq);
        }
    }
    if (A.M <= (TWO ? 4 : 8)) {
        e = form(search_multi<LPV, NI, DT, NI == 2 ? 2 : 3, 4>, 2, &f);
        if (e != hipSuccess) return e;
        if (all <= f.slots || one_a_cu) return launch(f, nq);
    }
    if (A.M <= 4) {
        const auto rounds = [&](const MultiForm &x) { return (all + x.slots - 1) / x.slots; };
        if constexpr (NI == 1) {
            e = form(search_multi<LPV, NI, DT, 4, 2>, 4, &g);
            if (e != hipSuccess) return e;
            if (rounds(g) < rounds(f)) f = g;
        }
        e = form(search_multi<LPV, NI, DT, NI <= 8 ? 5 : 4, 1>, 3, &g);
        if (e != hipSuccess) return e;
        return launch(rounds(g) < rounds(f) ? g : f, nq);
    }
    e = form(search_multi<LPV, NI, DT, 4, 2>, 4, &f);
    if (e != hipSuccess) return e;
    if (A.M <= 8 || all <= f.slots || one_a_cu) return launch(f, nq);
    e = form(search_multi<LPV, NI, DT, 8, 1>, 5, &f);
    return e == hipSuccess ? launch(f, nq) : e;
}

template <int LPV, int DT, bool LARGE>
hipError_t launch_multi_ni(const KArgs &A, int64_t nq, hipStream_t s)
{
    const int ni = (A.L + 63) / 64;
    if constexpr (LARGE) {
        if (ni <= 6) return launch_multi<LPV, 6, DT>(A, nq, s);
        if (ni <= 8) return launch_multi<LPV, 8, DT>(A, nq, s);
        return launch_multi<LPV, 16, DT>(A, nq, s);
    } else {
        if (ni <= 1) return launch_multi<LPV, 1, DT>(A, nq, s);
        if (ni <= 2) return launch_multi<LPV, 2, DT>(A, nq, s);
        return launch_multi<LPV, 4, DT>(A, nq, s);
    }
}

// one instantiation per storage type and size of L (up to 256, and more), each in a file of
// its own (search_multi_*.hip)
template <int DT, bool LARGE>
int launch_multi_dt(const KArgs &A, int64_t nq, hipStream_t s)
{
    hipError_t e;
    switch (lanes_per_vector(A.d)) {
    case 1: e = launch_multi_ni<1, DT, LARGE>(A, nq, s); break;
    case 2: e = launch_multi_ni<2, DT, LARGE>(A, nq, s); break;
    case 4: e = launch_multi_ni<4, DT, LARGE>(A, nq, s); break;
    case 8: e = launch_multi_ni<8, DT, LARGE>(A, nq, s); break;
    case 16: e = launch_multi_ni<16, DT, LARGE>(A, nq, s); break;
    case 32: e = launch_multi_ni<32, DT, LARGE>(A, nq, s); break;
    default: e = launch_multi_ni<64, DT, LARGE>(A, nq, s); break;
    }
    if (e != hipSuccess) return hip_fail(e, "search kernel launch");
    return SA_OK;
}

}  // namespace search_detail
}  // namespace sa
