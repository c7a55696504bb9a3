// Search with one worker (M = 1) and the visited set in the workspace: Algorithm 1, with
// the bookkeeping of Algorithm 3 at T = 1.  With a single worker the merge of Algorithm 3
// leaves the queue as it is, so the schedule (Algorithm 2) only moves the counters of
// global steps and merges.
//
// One 64-lane workgroup per query and no barrier.  Everything is sized for occupancy:
// the fewer registers a query needs, the more queries each SIMD keeps in flight to cover
// the latency of the random reads.
//
// Queue.  NI = ceil(L / 64) slots per lane hold the sorted 64-bit keys (order-preserving
// distance bits, id); entry p sits in slot p / 64 of lane p % 64.  The unchecked entries are
// wave-uniform 64-bit masks, one per slot, so finding the first of them is scalar work.
// The new entries of a step are merged in one pass (see insert_batch).
//
// Visited set.  It starts in LDS: sets of up to three exact tags, which stay.  As long as a
// vertex's set has room, LDS alone tells whether it was visited.  A vertex that finds its
// set full goes to a table in the query's workspace region: open addressing over 32-bit
// entries (id + 1; zero is empty), claimed with compare-and-swap, the first probe of a
// vertex at the line of its id block (see block_slot).  That table is a prefix of the region
// that doubles (rehashing the set) when the visited count passes three quarters of it.  A
// quarter as many sets of recent ids stand in front of it.  When the query ends it clears
// the table in use with whole-line stores, which leaves the region zero for the next launch:
// clearing only the slots it filled would write each of their lines back a second time
// (they are long evicted by then), and listing them would cost writes of its own.
// Every vertex used to be claimed in the table (a filter of recent ids in LDS kept repeats
// away): 2,410 compare-and-swaps per query at L = 192, each a write of 64 B and a round trip
// of its own.  10,000 queries over 1M rows: 2,376 -> 1,852 us (d = 128, two walkers,
// L = 192) and 1,230 -> 993 us (d = 96 bf16, L = 112, re-ranked).
//
// Distances.  LPV lanes share one vector, each lane four float4 chunks (c = g, g + LPV,
// ...), accumulated in double precision (in float32 where the data and the query are
// integers that make every partial sum exact), summed into the group's last lane by DPP
// row shifts and broadcasts, and rounded once to float.  The query row sits in LDS.
#pragma once
#include "search_body.h"
#include "search_queue.h"
#include "search_visited.h"

namespace sa {
namespace single_detail {

using search_detail::ACC_EITHER;
using search_detail::ACC_F32;
using search_detail::ACC_F64;
using search_detail::KArgs;
using search_detail::NO_SLOT;

// LDS of a wavefront besides the visited set: new keys (64, or all slots' keys; one that
// the insert drops what it does not want into, one for alignment), new ids, the query row
template <int LPV>
constexpr uint32_t single_lds_base(int stage = 64)   // stage: keys that the insert exchanges at once
{
    return (stage + 2) * 8 + 64 * 4 + 64 * LPV;
}

// log2 of the sets of the per-query visited set in LDS (one 32-bit word per set) that fits
// whatever the kernel's occupancy: the largest (up to 1024 sets, 4 KB) that keeps a
// wavefront's LDS within 160 KB / 28.  The launcher grows it (up to 2048 sets) where the
// kernel's registers hold fewer wavefronts per CU than that (lds_fill_log2).
template <int LPV>
constexpr int seen_log2()
{
    int l = 10;
    while (l > 6 && single_lds_base<LPV>() + (4u << l) > 160u * 1024u / 28u) --l;
    return l;
}
using search_detail::Queue;
using search_detail::Seen;
using search_detail::any_unchecked;
using search_detail::get_key;
using search_detail::insert_batch;
using search_detail::take_first;
using search_detail::VecSrc;
using search_detail::claim;
using search_detail::claim_rest;
using search_detail::block_slot;
using search_detail::clear_table;
using search_detail::grow_table;
using search_detail::distances;
using search_detail::rerank_list;
using search_detail::bits_below;
using search_detail::rdlane;
using search_detail::rdlane64;

// FEW: the form for launches that leave the chip idle (see launch_few)
template <int LPV, int NI, bool L2, int DT, int ACC, bool FEW>
__device__ __forceinline__ void single_query(const KArgs &A, int64_t qi, uint32_t *tbl)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr int STAGE = FEW ? 64 * NI : 64;
    uint64_t *const nkey = reinterpret_cast<uint64_t *>(smem);    // [STAGE + 2] keys of new vertices
    int32_t *const sid = reinterpret_cast<int32_t *>(nkey + STAGE + 2);   // [64] their ids
    float *const qs = reinterpret_cast<float *>(sid + 64);          // [16 LPV] the query
    // the visited set in LDS: [SEEN] sets and [SEEN / 4] sets of recent ids (see Seen)
    const int SEEN = 1 << A.seen_log2;
    const Seen seen(reinterpret_cast<uint32_t *>(qs + 16 * LPV), A.seen_log2, A.idbits);

    const int lane = __lane_id();
    const int R = A.R, g2 = A.glog2;
    const int L = A.qL ? __builtin_amdgcn_readfirstlane(A.qL[qi]) : A.L;
    const int kq = A.qk ? __builtin_amdgcn_readfirstlane(A.qk[qi]) : A.k;
    const uint64_t t_start = __builtin_amdgcn_s_memrealtime();
    // the second half of the region: scratch while the table grows, and the list handed
    // to the re-rank kernel
    uint32_t *const slots = tbl + (1u << g2);
    // the table in use is the first 2^t2 entries of the region's 2^g2; it doubles when
    // the visited set would pass three quarters of it
    int t2 = A.glog2_init;
    int cap = (3 << t2) / 4;
    const VecSrc V{A.codes, A.scale, A.ldc};
    bool exact32 = false;   // this query's distances are exact in float32

    {
        const int nch = A.d >> 2;
        const float *qrow = A.queries + qi * A.ldq;
        const float lo = (float)A.int_lo, hi = (float)A.int_hi;
        bool outside = false;   // some coordinate is not an integer in [int_lo, int_hi]
        for (int c = lane; c < 4 * LPV; c += 64) {
            const float4 v = c < nch ? *reinterpret_cast<const float4 *>(qrow + 4 * c) : make_float4(0.f, 0.f, 0.f, 0.f);
            reinterpret_cast<float4 *>(qs)[c] = v;
            if (c < nch)
                outside |= !(v.x == rintf(v.x) && v.x >= lo && v.x <= hi) || !(v.y == rintf(v.y) && v.y >= lo && v.y <= hi) ||
                           !(v.z == rintf(v.z) && v.z >= lo && v.z <= hi) || !(v.w == rintf(v.w) && v.w >= lo && v.w <= hi);
        }
        exact32 = __ballot(outside) == 0ull && A.acc_pass > 0;
        // with two passes, each query is searched by exactly one of them
        if (ACC != ACC_EITHER && A.acc_pass >= 0 && (__ballot(outside) == 0ull) != (A.acc_pass == 1)) return;
        sid[lane] = A.entry;
        {   // and recent; 16 bytes at a time (at least 80 words)
            uint4 *const z = reinterpret_cast<uint4 *>(qs + 16 * LPV);
            for (int i = lane; i < (SEEN + SEEN / 4) / 4; i += 64) z[i] = make_uint4(0u, 0u, 0u, 0u);
        }
    }
    __builtin_amdgcn_wave_barrier();

    // one worker: every local step expands one vertex, and every visited vertex has one
    // table slot, so the step count is the expansion count and the slot count is the
    // distance count
    int nslot = 0, substeps = 0, gsteps = 0, merges = 0, flags = 0;
    Queue<NI> Q;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        Q.k[i] = KEY_EMPTY;
        Q.un[i] = 0;
    }
    // dist(P, Q); P goes into the queue and the visited set
    distances<LPV, L2, DT, ACC>(V, A.d, qs, sid, 1, nkey, exact32);
    __builtin_amdgcn_wave_barrier();
    {
        const uint64_t k0 = nkey[0];
        if (lane == 0) Q.k[0] = k0;
        Q.un[0] = 1;
        Q.top = KEY_EMPTY;
        Q.len = 1;
        bool fresh = false;
        if (lane == 0) {
            if (!seen.put_first((uint32_t)A.entry)) (void)claim(tbl, t2, (uint32_t)A.entry, &fresh);
        }
        nslot = 1;
    }
    __builtin_amdgcn_wave_barrier();

    const int max_sub = A.max_substeps;
    const int32_t n = (int32_t)A.n;
    // Two walkers merging after every local step (Top-2, M = 2 with the every-step schedule,
    // R <= 32) also run here: the merge of their two local queues is the queue with both
    // expansions' new vertices inserted, so one queue serves.  Walker 0 expands the first
    // unchecked entry on lanes 0-31, walker 1 the second on lanes 32-63.
    const bool two = A.M == 2;
    // Two vectors per lane group in each pass of the distance loop (one round trip for 16
    // new vertices at d = 128 instead of two) where that pays for its registers, with up to
    // three queue slots per lane: float32 rows accumulated in float32 or wide enough
    // (d > 256) that a pass holds at most two vectors, and bf16 rows up to two slots (at
    // three the registers would cost two waves of seven).  Measured on 1M-row sets, d = 128
    // integer data: +2.3% (two walkers, L = 192) and +2.8% (one, L = 128) at one wave less;
    // d = 960: +2% at L = 64 and 128; d = 96 bf16: +2.8% (two walkers, L = 112, re-ranked);
    // d = 96 float32 in double 1-5% and fp8 1-4% slower.
    // For few queries registers cost nothing: a pass takes 32 vectors (a step of one walker)
    // where eight per lane group hold them.
    constexpr int GATHER_PB = FEW ? (LPV >= 16 ? 8 : (LPV >= 2 ? LPV / 2 : 1)) :
        (DT == SA_BF16 && NI <= 2) || (DT == SA_F32 && NI <= 3 && (ACC == ACC_F32 || LPV >= 32)) ? 2 : 1;
    // Gathers alongside the claims (SPEC) where LDS holds the full 1024 sets, so that few
    // vertices reach the table (with the 128 sets that d = 960 leaves room for, many do and
    // were there already, and each wasted read is a 3.8 KB row: 30-60% slower), and
    // where the five registers it takes cost no wave that pays (not at NI = 7, 8; at NI = 3
    // with float32 accumulation the timed two-walker search went 0.5% slower at 5 waves).
    // Measured on 1M rows: d = 128 one walker +2.5% (L = 128), +2.3% (256), +3.4% (384);
    // d = 96 in double +4% (one walker, L = 128) and +3% (two, L = 192).
    constexpr bool SPEC = FEW || (seen_log2<LPV>() >= 10 && NI != 7 && NI != 8 && !(ACC == ACC_F32 && NI == 3));
    const bool second = two && lane >= 32;
    int m = two && !A.staged ? 2 : 1;   // walkers active in the next step (staged: 1, then 2)
    int nexp = 0;
    // this lane's entry of an adjacency row (R <= 64); lanes past R load entry 0 and drop it
    const int aidx = two ? (lane & 31) : lane;
    const int32_t *const adj_lane = A.adj + (aidx < R ? aidx : 0);
    int32_t pv = -1, pv2 = -1, pu = -1;   // vertices whose rows are prefetched, and this lane's entry
    // Algorithm 2's test U / 1 >= L rho, as a bound on the integer U
    int u_merge;
    {
        const double t = ceil((double)L * A.rho);
        u_merge = !(t <= 2147483647.0) ? 0x7FFFFFFF : (t <= -2147483648.0 ? -0x7FFFFFFF - 1 : (int)t);
    }
    uint64_t worst = KEY_EMPTY;   // the last key of a full queue
    if (L == 1) worst = get_key(Q, 0);
    bool stop = false;
    while (any_unchecked(Q) && !stop) {
        gsteps++;
        int sub_in_step = 0;
        for (;;) {
            if (substeps >= max_sub) {
                flags |= SA_QFLAG_MAX_STEPS;
                stop = true;
                break;
            }
            substeps++;
            sub_in_step++;
            const int32_t v = take_first(Q.k, Q.un);
            const int32_t v2 = m == 2 ? take_first(Q.k, Q.un) : -1;
            nexp += v2 >= 0 ? 2 : 1;
            const int32_t vl = second ? v2 : v;   // the vertex whose row this lane reads
            int32_t u = pu;
            if (vl != (second ? pv2 : pv)) u = adj_lane[(int64_t)(vl >= 0 ? vl : v) * R];
            // prefetch the rows of the next candidates while this step runs
            {
                uint64_t ahead[NI];
#pragma unroll
                for (int i = 0; i < NI; ++i) ahead[i] = Q.un[i];
                const int32_t a1 = take_first(Q.k, ahead);
                pv = a1 >= 0 ? a1 : v;
                if (two) {
                    const int32_t a2 = take_first(Q.k, ahead);
                    pv2 = a2 >= 0 ? a2 : pv;
                }
            }
            pu = adj_lane[(int64_t)(second ? pv2 : pv) * R];
            if (aidx >= R || vl < 0 || u < 0 || u >= n) u = -1;   // idle walker, padding, malformed entries
            bool fresh = false;
            const bool ask = u >= 0 && seen.claim((uint32_t)u, &fresh);   // not settled in LDS
            // The first probe of each claim goes out now.  With SPEC the vectors of every vertex
            // that was not found in LDS are read while it is in flight, and the keys of those
            // found in the table are dropped after.  Without, the claims settle first and only
            // new vertices are read.
            uint32_t old = 0u;
            if (ask) old = atomicCAS(&tbl[block_slot((uint32_t)u, t2)], 0u, (uint32_t)u + 1u);
            bool claimed = false;
            if (!SPEC && ask) (void)claim_rest(tbl, t2, (uint32_t)u, old, &claimed);
            const bool send = fresh || (SPEC ? ask : claimed);   // the vertices whose vectors are read
            const uint64_t am = __ballot(send);
            const int nsend = __popcll(am);
            const int apos = bits_below(am);
            sid[lane] = 0;   // (a pass of the distances reads ids past the last)
            if (send) sid[apos] = u;
            __builtin_amdgcn_wave_barrier();
            distances<LPV, L2, DT, ACC, GATHER_PB, FEW>(V, A.d, qs, sid, nsend, nkey, exact32);
            if (SPEC && ask) (void)claim_rest(tbl, t2, (uint32_t)u, old, &claimed);
            fresh = fresh || claimed;
            nslot += __popcll(__ballot(fresh));
            if (SPEC) {
                __builtin_amdgcn_wave_barrier();
                if (send && !fresh) nkey[apos] = KEY_EMPTY;
            }
            __builtin_amdgcn_wave_barrier();
            const uint64_t mk = lane < nsend ? nkey[lane] : KEY_EMPTY;
            __builtin_amdgcn_wave_barrier();
            // insert the survivors; the update position is the best place one of them takes
            const uint64_t sbits = __ballot(mk < worst);
            int U = L;
            if (sbits) {
                U = insert_batch<NI, FEW>(Q, L, mk, sbits, nkey);
                if (Q.len == L) worst = get_key(Q, L - 1);
            }
            if (nslot + (two ? 2 * R : R) > cap) {
                if (t2 < g2) {
                    // (one doubling suffices: nslot <= cap before, and at most 64 new < cap)
                    ++t2;
                    (void)grow_table(tbl, slots, t2 - 1, t2);
                    cap = (3 << t2) / 4;
                    flags |= SA_QFLAG_SPILLED;
                } else {
                    flags |= SA_QFLAG_CAPACITY;
                    stop = true;
                    break;
                }
            }
            bool merge_now;
            if (A.sync == SA_SYNC_BSP) merge_now = true;
            else if (A.sync == SA_SYNC_STATIC) merge_now = A.static_I > 0 && sub_in_step >= A.static_I;
            else merge_now = U >= u_merge;
            if (!any_unchecked(Q) || merge_now) break;
        }
        merges++;   // the queue is S unchanged
        if (two) m = 2;
    }

    if (A.rerank != 0) {
        // hand the first nr entries of the final list to the re-rank kernel
        const int nr = A.rerank < 0 ? Q.len : min(A.rerank, Q.len);
        int32_t *const list = rerank_list(slots, g2);
#pragma unroll
        for (int i = 0; i < NI; ++i)
            if (64 * i + lane < nr) list[1 + 64 * i + lane] = key_id(Q.k[i]);
        if (lane == 0) list[0] = nr;
    } else {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int p = 64 * i + lane;
            if (p < kq) {
                const bool ok = p < Q.len;
                A.ids[qi * A.ldo + p] = ok ? key_id(Q.k[i]) : -1;
                A.dists[qi * A.ldo + p] = ok ? key_dist(Q.k[i]) : __builtin_inff();
            }
        }
    }
    // leave the workspace zero-filled for the next launch
    clear_table(tbl, t2);
    if (lane == 0 && A.stats) {
        sa_query_stats st;
        st.global_steps = gsteps;
        st.substeps = substeps;
        st.expansions = nexp;
        st.dist_comps = nslot;
        st.merges = merges;
        st.flags = flags;
        st.t_start = t_start;
        st.t_end = __builtin_amdgcn_s_memrealtime();
        A.stats[qi] = st;
    }
}

// Workgroup b runs job b: query order[b] (or b), in workspace region b.  The hardware
// dispatcher hands out workgroups in index order as slots free up, so a batch ordered
// longest first is scheduled longest first.  (A persistent loop over jobs in one
// workgroup was measured: any loop around the search costs 17-36 more VGPRs, about a
// third of the occupancy this latency-bound search lives on.)
template <int LPV, int NI, bool L2, int DT, int ACC>
__global__ void __launch_bounds__(64) search_single(KArgs A)
{
    const int32_t job = blockIdx.x;
    uint32_t *const tbl = reinterpret_cast<uint32_t *>(A.ghash) + ((size_t)job << (A.glog2 + 1));
    single_query<LPV, NI, L2, DT, ACC, false>(A, A.order ? A.order[job] : job, tbl);
}

// Persistent form: each resident workgroup takes jobs from the device counter until none
// is left, every one in its own workspace region (see KArgs::jobctr).
template <int LPV, int NI, bool L2, int DT, int ACC>
__global__ void __launch_bounds__(64) search_single_loop(KArgs A)
{
    uint32_t *const tbl = reinterpret_cast<uint32_t *>(A.ghash) + ((size_t)blockIdx.x << (A.glog2 + 1));
    for (;;) {
        int job = 0;
        if (__lane_id() == 0) job = atomicAdd(A.jobctr, 1);
        job = __builtin_amdgcn_readfirstlane(job);
        if (job >= A.njobs) break;
        // (loads after stores are vector loads: made wave-uniform again, or everything
        // derived from the query index would take vector registers)
        const int32_t qi = A.order ? __builtin_amdgcn_readfirstlane(A.order[job]) : job;
        single_query<LPV, NI, L2, DT, ACC, false>(A, qi, tbl);
    }
    if (__lane_id() == 0) search_detail::release_jobs(A.jobctr);
}

// log2 of the visited set's sets where few queries share a CU: from l (what the kernel's
// registers leave at full occupancy) up to 8192, as far as the LDS of a CU goes round its
// share of the nq queries and until nearly every query's visited set (8 L to 15 L vertices,
// three to a set) fits without going to the workspace table.
inline int seen_log2_for(int64_t nq, uint32_t base, int l, int L)
{
    const int64_t per_cu = (nq + 255) / 256;
    while (l < 13 && (1 << l) < 8 * L && (int64_t)(base + (5u << (l + 1)) + 1024u) * per_cu <= 160 * 1024) ++l;
    return l;
}

template <int LPV, int NI, int DT, int ACC>
hipError_t launch1(const KArgs &A, int64_t nq, hipStream_t s)
{
    constexpr uint32_t base = single_lds_base<LPV>();
    KArgs B = A;
    if (A.jobctr) {
        auto k = A.metric == SA_L2 ? search_single_loop<LPV, NI, true, DT, ACC>
                                   : search_single_loop<LPV, NI, false, DT, ACC>;
        hipError_t e = lds_fill_log2(reinterpret_cast<const void *>(k), 64, base, seen_log2<LPV>(), 11, &B.seen_log2);
        if (e != hipSuccess) return e;
        const uint32_t lds = base + (5u << B.seen_log2);
        int64_t grid = nq;
        e = resident_grid(reinterpret_cast<const void *>(k), 64, lds, nq, &grid);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k, dim3((unsigned)grid), dim3(64), lds, s, B);
        return hipGetLastError();
    }
    auto k = A.metric == SA_L2 ? search_single<LPV, NI, true, DT, ACC> : search_single<LPV, NI, false, DT, ACC>;
    const hipError_t e = lds_fill_log2(reinterpret_cast<const void *>(k), 64, base, seen_log2<LPV>(), 11, &B.seen_log2);
    if (e != hipSuccess) return e;
    B.seen_log2 = seen_log2_for(nq + A.company, base, B.seen_log2, A.L);
    hipLaunchKernelGGL(k, dim3((unsigned)nq), dim3(64), base + (5u << B.seen_log2), s, B);
    return hipGetLastError();
}

template <int LPV, int DT, int ACC>
hipError_t launch1_ni(const KArgs &A, int64_t nq, hipStream_t s)
{
    const int ni = (A.L + 63) / 64;
    if (ni <= 1) return launch1<LPV, 1, DT, ACC>(A, nq, s);
    if (ni <= 2) return launch1<LPV, 2, DT, ACC>(A, nq, s);
    if (ni <= 3) return launch1<LPV, 3, DT, ACC>(A, nq, s);
    if (ni <= 4) return launch1<LPV, 4, DT, ACC>(A, nq, s);
    if (ni <= 5) return launch1<LPV, 5, DT, ACC>(A, nq, s);
    if (ni <= 6) return launch1<LPV, 6, DT, ACC>(A, nq, s);
    if (ni <= 7) return launch1<LPV, 7, DT, ACC>(A, nq, s);
    if (ni <= 8) return launch1<LPV, 8, DT, ACC>(A, nq, s);
    return launch1<LPV, 16, DT, ACC>(A, nq, s);
}

// one instantiation per storage type, each in a file of its own (search_single_*.hip)
// float32 accumulation is compiled for float32 storage up to d = 256 (integer data such
// as 8-bit descriptors); the launcher asks for it only there
template <int LPV, int DT>
hipError_t launch_lpv(const KArgs &A, int64_t nq, hipStream_t s)
{
    if constexpr (DT == SA_F32 && LPV <= 16)
        if (A.acc_pass == 1) return launch1_ni<LPV, DT, ACC_F32>(A, nq, s);
    return launch1_ni<LPV, DT, ACC_F64>(A, nq, s);
}

template <int DT>
int launch_dt(const KArgs &A, int64_t nq, hipStream_t s)
{
    hipError_t e;
    switch (search_detail::lanes_per_vector(A.d)) {
    case 1: e = launch_lpv<1, DT>(A, nq, s); break;
    case 2: e = launch_lpv<2, DT>(A, nq, s); break;
    case 4: e = launch_lpv<4, DT>(A, nq, s); break;
    case 8: e = launch_lpv<8, DT>(A, nq, s); break;
    case 16: e = launch_lpv<16, DT>(A, nq, s); break;
    case 32: e = launch_lpv<32, DT>(A, nq, s); break;
    default: e = launch_lpv<64, DT>(A, nq, s); break;
    }
    if (e != hipSuccess) return hip_fail(e, "search kernel launch");
    return SA_OK;
}

// The form for launches of so few queries that all are resident at once whatever their
// registers: up to eight vectors per lane group in flight, and one launch for both
// arithmetics of integer data.
template <int LPV, int NI, bool L2, int DT>
__global__ void __launch_bounds__(64) search_few(KArgs A)
{
    const int32_t job = blockIdx.x;
    uint32_t *const tbl = reinterpret_cast<uint32_t *>(A.ghash) + ((size_t)job << (A.glog2 + 1));
    constexpr int ACC = DT == SA_F32 && LPV <= 16 ? ACC_EITHER : ACC_F64;
    single_query<LPV, NI, L2, DT, ACC, true>(A, A.order ? A.order[job] : job, tbl);
}

template <int LPV, int NI, int DT>
hipError_t launch_few(const KArgs &A, int64_t nq, hipStream_t s, bool *taken)
{
    constexpr uint32_t base = single_lds_base<LPV>(64 * NI);
    auto k = A.metric == SA_L2 ? search_few<LPV, NI, true, DT> : search_few<LPV, NI, false, DT>;
    KArgs B = A;
    const int64_t all = nq + A.company;
    B.seen_log2 = seen_log2_for(all, base, seen_log2<LPV>(), A.L);
    int64_t grid = 0;
    const hipError_t e = resident_grid(reinterpret_cast<const void *>(k), 64, base + (5u << B.seen_log2), all, &grid);
    if (e != hipSuccess) return e;
    *taken = grid >= all;
    if (!*taken) return hipSuccess;
    hipLaunchKernelGGL(k, dim3((unsigned)nq), dim3(64), base + (5u << B.seen_log2), s, B);
    return hipGetLastError();
}

template <int LPV, int DT>
hipError_t launch_few_ni(const KArgs &A, int64_t nq, hipStream_t s, bool *taken)
{
    const int ni = (A.L + 63) / 64;
    if (ni <= 1) return launch_few<LPV, 1, DT>(A, nq, s, taken);
    if (ni <= 2) return launch_few<LPV, 2, DT>(A, nq, s, taken);
    if (ni <= 3) return launch_few<LPV, 3, DT>(A, nq, s, taken);
    if (ni <= 4) return launch_few<LPV, 4, DT>(A, nq, s, taken);
    if (ni <= 6) return launch_few<LPV, 6, DT>(A, nq, s, taken);
    if (ni <= 8) return launch_few<LPV, 8, DT>(A, nq, s, taken);
    return launch_few<LPV, 16, DT>(A, nq, s, taken);
}

template <int DT>
int launch_few_dt(const KArgs &A, int64_t nq, hipStream_t s, bool *taken)
{
    hipError_t e;
    *taken = false;
    switch (search_detail::lanes_per_vector(A.d)) {
    case 1: e = launch_few_ni<1, DT>(A, nq, s, taken); break;
    case 2: e = launch_few_ni<2, DT>(A, nq, s, taken); break;
    case 4: e = launch_few_ni<4, DT>(A, nq, s, taken); break;
    case 8: e = launch_few_ni<8, DT>(A, nq, s, taken); break;
    case 16: e = launch_few_ni<16, DT>(A, nq, s, taken); break;
    case 32: e = launch_few_ni<32, DT>(A, nq, s, taken); break;
    default: e = launch_few_ni<64, DT>(A, nq, s, taken); break;
    }
    if (e != hipSuccess) return hip_fail(e, "search kernel launch");
    return SA_OK;
}

}  // namespace single_detail
}  // namespace sa
