// Search with several workers that merge after every local step (the "bsp" schedule:
// Top-M, Sec. 4.1 of the paper, staged as in Sec. 4.2): the case of Algorithm 3 in which the
// local queues need not exist.  A worker's queue is S for one expansion, so a global step is:
// the first m unchecked entries of S are expanded, one per wavefront; their new neighbours'
// distances are computed; S becomes the best L of S and these.  Neither the worker that
// claims a vertex nor a local queue that overflows changes that (what a local queue drops
// has L better keys before it), and the update positions are not read.
//
// One workgroup of M wavefronts runs one query.  S is a sorted array in LDS, in two copies;
// its entries are keys with the id moved up by one bit and the unchecked flag below it, which
// leaves their order.  A step, with a barrier after each part:
//   1. wavefront t picks the t-th unchecked entry from the slots' masks, reads its row, and
//      claims the neighbours (search_visited.h); new ones are appended to one list
//   2. the wavefronts share out the list and compute the distances; those that beat the last
//      key of a full S are appended to the list of new keys
//   3. each new key is ranked among S and the new keys by counting, a group of lanes per key;
//      it is written to its place in the next S, which is marked in a bit mask
//   4. the other places are filled from S in order, and the slots' unchecked masks built
// Few instructions and four barriers a step; bound by the row and the vectors, two dependent
// round trips to memory.  The general kernel (search_multi.h), which this replaced for the
// schedule, inserted into every local queue, one key after the other, and ranked each against
// all other queues behind eight barriers.  Over 1M x 128, one query with 16 workers, L = 176:
// 291 -> 102 us; over 200K x 128, 1,000 queries with 4 workers, L = 192: 842 -> 237 us; L = 768,
// 16 workers: 1,157 -> 193 us.
#include "search_body.h"
#include "search_visited.h"

#include <algorithm>
#include <atomic>

namespace sa {
namespace search_detail {
namespace {

struct BspLds {
    uint32_t o_key, o_ids, o_out, o_q, o_mark, o_un, o_ctrl, o_seen, total;   // o_key: S, S', new keys
};

struct BspCtrl {
    int32_t nlist[2], nnew[2];   // by parity of the step: vertices to measure, new keys
    int32_t used;   // some claim went to the workspace table
    int32_t job;
};

__host__ __device__ inline BspLds bsp_lds(int L, int M, int lpv, int seen_log2)
{
    BspLds Y;
    const uint32_t Lp = (uint32_t)(L + 63) / 64 * 64;
    uint32_t o = 0;
    Y.o_key = o; o += 8u * (2u * Lp + 64u * M);
    Y.o_out = o; o += 8u * 64u * M;
    Y.o_un = o; o += 8u * 16u;
    Y.o_ids = o; o += 4u * 64u * (M + 1);   // (a pass of the last wavefront reads past the list)
    Y.o_mark = o; o += 4u * 32u * 2u;
    Y.o_ctrl = o; o += 32u;
    Y.o_q = o; o += 64u * (uint32_t)lpv;
    Y.o_seen = o; o += 5u << seen_log2;
    Y.total = o;
    return Y;
}

// the r-th (from 0) set bit of the wave-uniform m, which has more than r
__device__ __forceinline__ int nth_bit(uint64_t m, int r)
{
    const bool set = __builtin_amdgcn_inverse_ballot_w64(m);
    return __builtin_ctzll(__ballot(set && bits_below(m) == r));
}

template <int LPV, bool L2, int DT>
__device__ __forceinline__ void bsp_body(const KArgs &A, int64_t job, int64_t region)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    // (a wavefront takes some ten of a step's vectors)
    constexpr int PB = LPV >= 32 ? 4 : 2;
    constexpr int ACC = DT == SA_F32 && LPV <= 16 ? ACC_EITHER : ACC_F64;
    const int tid = threadIdx.x, lane = __lane_id(), nthr = blockDim.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t qi = A.order ? __builtin_amdgcn_readfirstlane(A.order[job]) : job;
    const int L = A.qL ? __builtin_amdgcn_readfirstlane(A.qL[qi]) : A.L, M = A.M, R = A.R;
    const int kq = A.qk ? __builtin_amdgcn_readfirstlane(A.qk[qi]) : A.k;
    const int nslots = (L + 63) >> 6;
    const BspLds Y = bsp_lds(A.L, M, LPV, A.seen_log2);
    uint64_t *S = reinterpret_cast<uint64_t *>(smem + Y.o_key);
    uint64_t *Sn = S + (A.L + 63) / 64 * 64;
    uint64_t *const nk = Sn + (A.L + 63) / 64 * 64;                               // [64 M] new keys
    uint64_t *const out = reinterpret_cast<uint64_t *>(smem + Y.o_out) + 64 * w;   // [64]
    uint64_t *const un = reinterpret_cast<uint64_t *>(smem + Y.o_un);              // [16] unchecked entries of S
    int32_t *const ids = reinterpret_cast<int32_t *>(smem + Y.o_ids);              // [64 (M + 1)]
    uint32_t *const marks = reinterpret_cast<uint32_t *>(smem + Y.o_mark);         // [2][32], by parity
    BspCtrl *const C = reinterpret_cast<BspCtrl *>(smem + Y.o_ctrl);
    float *const qs = reinterpret_cast<float *>(smem + Y.o_q);
    const Seen seen(reinterpret_cast<uint32_t *>(smem + Y.o_seen), A.seen_log2, A.idbits);
    unsigned char *const ws = reinterpret_cast<unsigned char *>(A.ghash) + ((size_t)region << (A.glog2 + 4));
    uint32_t *const tbl = reinterpret_cast<uint32_t *>(ws);   // 2^glog2 entries, if the sets overflow
    const VecSrc V{A.codes, A.scale, A.ldc};
    const uint64_t t_start = __builtin_amdgcn_s_memrealtime();
    const int32_t n = (int32_t)A.n;
    const int32_t *const adj_lane = A.adj + (lane < R ? lane : 0);

    for (int i = tid; i < (5 << A.seen_log2) / 16; i += nthr)
        reinterpret_cast<uint4 *>(smem + Y.o_seen)[i] = make_uint4(0u, 0u, 0u, 0u);
    for (int i = tid; i < 64 * (M + 1); i += nthr) ids[i] = A.entry;
    if (tid < 64) marks[tid] = 0u;
    if (tid < 16) un[tid] = 0ull;
    if (tid < 2) C->nlist[tid] = C->nnew[tid] = 0;
    if (tid == 0) C->used = 0;
    bool exact32 = false;   // this query's distances are exact in float32
    {
        const int nch = A.d >> 2;
        const float *const qrow = A.queries + qi * A.ldq;
        const float lo = (float)A.int_lo, hi = (float)A.int_hi;
        bool outside = false;
        // (every wavefront reads and writes the whole row: the flag is then known to all)
        for (int c = lane; c < 4 * LPV; c += 64) {
            const float4 v = c < nch ? *reinterpret_cast<const float4 *>(qrow + 4 * c) : make_float4(0.f, 0.f, 0.f, 0.f);
            reinterpret_cast<float4 *>(qs)[c] = v;
            if (c < nch)
                outside |= !(v.x == rintf(v.x) && v.x >= lo && v.x <= hi) || !(v.y == rintf(v.y) && v.y >= lo && v.y <= hi) ||
                           !(v.z == rintf(v.z) && v.z >= lo && v.z <= hi) || !(v.w == rintf(v.w) && v.w >= lo && v.w <= hi);
        }
        exact32 = __ballot(outside) == 0ull && A.acc_pass > 0;
    }
    __syncthreads();
    if (w == 0) {
        // the start point: its distance, the list holding only it, and the visited set
        distances<LPV, L2, DT, ACC>(V, A.d, qs, ids, 1, out, exact32);
        __builtin_amdgcn_wave_barrier();
        if (lane == 0) {
            S[0] = entry_of(out[0], 1u);
            un[0] = 1ull;
            if (!seen.put_first((uint32_t)A.entry)) {
                bool fresh;
                (void)claim(tbl, A.glog2, (uint32_t)A.entry, &fresh);
                C->used = 1;
            }
        }
    }
    __syncthreads();

    // Every wavefront keeps the same counts.  The visited set's bounds are those of the general
    // kernel's tables, so that a search spills and stops where it did there.  The table always
    // has room for what they allow: glog2 >= llog2 (the launcher sees to it), so half of 2^llog2
    // is at most half of it.
    int slen = 1, hcount = 1, steps = 0, nexp = 0, flags = 0;
    bool spilled = A.llog2 == 0, stop = false;
    int m = A.staged ? 1 : M;
    while (!stop) {
        // ---- 1. the first m unchecked entries, one per wavefront
        const uint64_t um = lane < nslots ? un[lane] : 0ull;
        int upto = __popcll(um);   // unchecked entries up to and including this lane's slot
        const int here = upto;
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) {
            const int v = __shfl_up(upto, o, 64);
            if (lane >= o) upto += v;
        }
        const int total = __builtin_amdgcn_readlane(upto, 15);
        if (total == 0) break;
        const int active = min(m, total);
        const auto find = [&](int r) {   // position of the r-th unchecked entry
            const int s = __builtin_ctzll(__ballot(upto > r));
            return 64 * s + nth_bit(rdlane64(um, s), r - __builtin_amdgcn_readlane(upto - here, s));
        };
        const int par = steps & 1;
        if (steps >= A.max_substeps) {
            flags |= SA_QFLAG_MAX_STEPS;
            ++steps;       // (counted as a global step and a merge, not as a local step)
            nexp |= 1 << 30;
            break;
        }
        ++steps;
        const int last = find(active - 1);   // every unchecked entry up to here is expanded
        nexp += active;
        bool fresh = false;
        int32_t u = -1;
        if (w < active) {
            const int32_t v = entry_id(S[find(w)]);
            u = adj_lane[(int64_t)v * R];
            if (lane >= R || u < 0 || u >= n) u = -1;   // padding and malformed entries
            if (u >= 0 && seen.claim((uint32_t)u, &fresh)) {
                (void)claim(tbl, A.glog2, (uint32_t)u, &fresh);
                C->used = 1;
            }
            const uint64_t fm = __ballot(fresh);
            int base = 0;
            if (lane == 0 && fm) base = atomicAdd(&C->nlist[par], __popcll(fm));
            base = __builtin_amdgcn_readfirstlane(base);
            if (fresh) ids[base + bits_below(fm)] = u;
        }
        if (tid < 32) marks[32 * (par ^ 1) + tid] = 0u;
        if (tid == 0) C->nnew[par ^ 1] = 0;
        __syncthreads();

        // ---- 2. distances of the new vertices
        const int nlist = __builtin_amdgcn_readfirstlane(C->nlist[par]);
        hcount += nlist;
        const uint64_t worst = slen == L ? S[L - 1] : ~0ull;
        {
            const int share = (nlist + M - 1) / M;   // at most 64
            const int i0 = w * share, cnt = min(share, nlist - i0);
            if (cnt > 0) {
                distances<LPV, L2, DT, ACC, PB, true>(V, A.d, qs, ids + i0, cnt, out, exact32);
                __builtin_amdgcn_wave_barrier();
                const uint64_t e = lane < cnt ? entry_of(out[lane], 1u) : ~0ull;
                const bool in = e < worst;
                const uint64_t im = __ballot(in);
                int base = 0;
                if (lane == 0 && im) base = atomicAdd(&C->nnew[par], __popcll(im));
                base = __builtin_amdgcn_readfirstlane(base);
                if (in) nk[base + bits_below(im)] = e;
            }
        }
        if (tid == 0) C->nlist[par ^ 1] = 0;
        __syncthreads();

        // ---- 3. ranks of the new keys: p lanes count for one key
        const int nnew = __builtin_amdgcn_readfirstlane(C->nnew[par]);
        uint32_t *const mark = marks + 32 * par;
        int lp = 0;   // log2 p
        while (lp < 4 && (nnew << (lp + 1)) <= nthr) ++lp;
        const int p = 1 << lp;
        for (int i = tid >> lp; i < nnew; i += nthr >> lp) {
            const uint64_t e = nk[i];
            const int part = tid & (p - 1);
            int r = 0;
            // (a search of S takes about ten round trips through LDS, a count four instructions
            // per entry)
            if (slen > 32 * p) {
                if (part == 0) r = lower_bound(S, slen, e);
            } else {
#pragma unroll 4
                for (int j = part; j < slen; j += p) r += S[j] < e ? 1 : 0;
            }
#pragma unroll 4
            for (int j = part; j < nnew; j += p) r += nk[j] < e ? 1 : 0;
            // sum into the last lane of the group
            if (p > 1) r += (int)row_shr0<1>((uint32_t)r);
            if (p > 2) r += (int)row_shr0<2>((uint32_t)r);
            if (p > 4) r += (int)row_shr0<4>((uint32_t)r);
            if (p > 8) r += (int)row_shr0<8>((uint32_t)r);
            if (part == p - 1 && r < L) {
                Sn[r] = e;
                atomicOr(&mark[r >> 5], 1u << (r & 31));
            }
        }
        __syncthreads();

        // ---- 4. the other places, in order, from S
        const int nlen = min(L, slen + nnew);
        for (int s = w; s < nslots; s += M) {
            const uint32_t mw = lane < 32 ? mark[lane] : 0u;
            const uint64_t own = ((uint64_t)rdlane(mw, 2 * s + 1) << 32) | rdlane(mw, 2 * s);
            int below = lane < 2 * s ? __popc(mw) : 0;   // marks in the slots below
#pragma unroll
            for (int o = 16; o > 0; o >>= 1) below += __shfl_xor(below, o, 64);
            below = __builtin_amdgcn_readfirstlane(below);
            const int P = 64 * s + lane;
            const bool marked = __builtin_amdgcn_inverse_ballot_w64(own);
            const int j = P - below - bits_below(own);
            const bool from = !marked && P < nlen;
            uint64_t e = S[from ? j : 0];
            if (j <= last) e &= ~1ull;   // expanded in this step, or before
            if (from) Sn[P] = e;
            const uint64_t b = __ballot(P < nlen && (marked || (e & 1ull)));
            if (lane == 0) un[s] = b;
        }
        uint64_t *const t = S;
        S = Sn;
        Sn = t;
        slen = nlen;
        // keep the visited set below half (LDS) / three quarters (workspace) before the next
        // step, which adds at most m R entries
        const int need = hcount + m * R;
        if (!spilled && need > (1 << A.llog2) / 2) {
            if (need > (3 << A.glog2) / 4) {
                flags |= SA_QFLAG_CAPACITY;
                stop = true;
            } else {
                spilled = true;
                flags |= SA_QFLAG_SPILLED;
            }
        } else if (spilled && need > (3 << A.glog2) / 4) {
            flags |= SA_QFLAG_CAPACITY;
            stop = true;
        }
        if (A.staged && m < M) m = min(2 * m, M);
        __syncthreads();
    }

    if (A.rerank != 0) {
        // hand the first nr entries of the final list to the re-rank kernel
        const int nr = A.rerank < 0 ? slen : min(A.rerank, slen);
        int32_t *const list = rerank_list(reinterpret_cast<uint32_t *>(ws + ((size_t)8 << A.glog2)), A.glog2);
        for (int i = tid; i < nr; i += nthr) list[1 + i] = entry_id(S[i]);
        if (tid == 0) list[0] = nr;
    } else {
        for (int i = tid; i < kq; i += nthr) {
            const bool ok = i < slen;
            A.ids[qi * A.ldo + i] = ok ? entry_id(S[i]) : -1;
            A.dists[qi * A.ldo + i] = ok ? key_dist(S[i]) : __builtin_inff();
        }
    }
    // leave the workspace zero-filled for the next launch
    if (C->used) {   // (set before the last barrier)
        uint4 *const z = reinterpret_cast<uint4 *>(tbl);
        for (int i = tid; i < (1 << (A.glog2 - 2)); i += nthr) z[i] = make_uint4(0u, 0u, 0u, 0u);
    }
    if (tid == 0 && A.stats) {
        const int cut = nexp >> 30;   // the search ended at its step limit
        sa_query_stats st;
        st.global_steps = steps;
        st.substeps = steps - cut;
        st.expansions = nexp & ((1 << 30) - 1);
        st.dist_comps = hcount;
        st.merges = steps;
        st.flags = flags;
        st.t_start = t_start;
        st.t_end = __builtin_amdgcn_s_memrealtime();
        A.stats[qi] = st;
    }
}

template <int LPV, bool L2, int DT>
__global__ void __launch_bounds__(1024) search_bsp(KArgs A)
{
    bsp_body<LPV, L2, DT>(A, blockIdx.x, blockIdx.x);
}

// Persistent form: each resident workgroup takes jobs from the device counter until none
// is left, every one in its own workspace region (see KArgs::jobctr).
template <int LPV, bool L2, int DT>
__global__ void __launch_bounds__(1024) search_bsp_loop(KArgs A)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    BspCtrl *const C = reinterpret_cast<BspCtrl *>(smem + bsp_lds(A.L, A.M, LPV, A.seen_log2).o_ctrl);
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) C->job = atomicAdd(A.jobctr, 1);
        __syncthreads();
        const int job = __builtin_amdgcn_readfirstlane(C->job);
        if (job >= A.njobs) break;
        bsp_body<LPV, L2, DT>(A, job, blockIdx.x);
    }
    __syncthreads();
    if (threadIdx.x == 0) release_jobs(A.jobctr);
}

template <int LPV, int DT>
hipError_t launch_bsp_one(const KArgs &A, int64_t nq, hipStream_t s)
{
    const void *const k =
        A.jobctr ? (A.metric == SA_L2 ? reinterpret_cast<const void *>(search_bsp_loop<LPV, true, DT>)
                                      : reinterpret_cast<const void *>(search_bsp_loop<LPV, false, DT>))
                 : (A.metric == SA_L2 ? reinterpret_cast<const void *>(search_bsp<LPV, true, DT>)
                                      : reinterpret_cast<const void *>(search_bsp<LPV, false, DT>));
    // the dynamic LDS limit is raised to the whole 160 KB once per kernel and device, not on
    // every launch (the latency path launches one query at a time)
    static std::atomic<uint64_t> raised[4] = {{0}, {0}, {0}, {0}};
    std::atomic<uint64_t> &done = raised[(A.jobctr ? 2 : 0) + (A.metric == SA_L2 ? 1 : 0)];
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = 1ull << (dev & 63);
    if (!(done.load(std::memory_order_acquire) & bit)) {
        e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        done.fetch_or(bit, std::memory_order_acq_rel);
    }
    // Sets for some 24 L visited vertices (three to a set; sixteen workers explore more than
    // one), as far as the LDS goes round the queries of a CU: its share of the launch, at most
    // the workgroups that 16 wavefronts make
    KArgs B = A;
    const int64_t per_cu = std::max<int64_t>(1, std::min<int64_t>((nq + A.company + 255) / 256, 16 / A.M));
    B.seen_log2 = 8;
    while (B.seen_log2 < 13 && (1 << B.seen_log2) < 8 * A.L &&
           (int64_t)bsp_lds(A.L, A.M, LPV, B.seen_log2 + 1).total * per_cu <= 156 * 1024)
        ++B.seen_log2;
    const uint32_t lds = bsp_lds(A.L, A.M, LPV, B.seen_log2).total;
    int64_t grid = nq;
    if (A.jobctr) {
        e = resident_grid(k, 64 * A.M, lds, nq, &grid);
        if (e != hipSuccess) return e;
    }
    void *args[] = {&B};
    return hipLaunchKernel(k, dim3((unsigned)grid), dim3(64 * A.M), args, lds, s);
}

template <int DT>
hipError_t launch_bsp_dt(const KArgs &A, int64_t nq, hipStream_t s)
{
    switch (lanes_per_vector(A.d)) {
    case 1: return launch_bsp_one<1, DT>(A, nq, s);
    case 2: return launch_bsp_one<2, DT>(A, nq, s);
    case 4: return launch_bsp_one<4, DT>(A, nq, s);
    case 8: return launch_bsp_one<8, DT>(A, nq, s);
    case 16: return launch_bsp_one<16, DT>(A, nq, s);
    case 32: return launch_bsp_one<32, DT>(A, nq, s);
    default: return launch_bsp_one<64, DT>(A, nq, s);
    }
}

}  // namespace
}  // namespace search_detail

int launch_search_bsp(const search_detail::KArgs &A, int dtype, int64_t nq, hipStream_t s)
{
    const hipError_t e = dtype == SA_BF16       ? search_detail::launch_bsp_dt<SA_BF16>(A, nq, s)
                         : dtype == SA_FP8E4M3 ? search_detail::launch_bsp_dt<SA_FP8E4M3>(A, nq, s)
                                               : search_detail::launch_bsp_dt<SA_F32>(A, nq, s);
    return e == hipSuccess ? SA_OK : hip_fail(e, "search kernel launch");
}

}  // namespace sa
