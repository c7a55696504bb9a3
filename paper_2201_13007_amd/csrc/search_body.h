// What the search kernels share (Speed-ANN, arXiv 2201.13007, Algorithm 3 with CheckMetrics of
// Algorithm 2; Algorithm 1 when there is one worker), for gfx950: the arguments, cross-lane
// helpers and the distances.
//
//   search_single.h   one worker, and two that merge after every step, in one wavefront
//   search_bsp.hip    several workers that merge after every step
//   search_multi.h    every other case
//
// Distances: LPV lanes share one vector, each lane four float4 chunks, accumulated in double
// precision (or exactly in float32 for integer data), summed by DPP row shifts and rounded
// once to float; the query sits in LDS.
#pragma once
#include "sa_internal.h"

#include <type_traits>

namespace sa {
namespace search_detail {

constexpr uint32_t NO_SLOT = 0xFFFFFFFFu;

struct KArgs {
    const void *codes;           // stored vectors: rows of ldc elements of the index's dtype
    const float *scale;          // fp8: one scale per vector
    int64_t ldc;
    const float *vec32;          // float32 vectors for the re-rank
    int64_t ld32;
    int32_t rerank;
    const int32_t *adj;
    const float *queries;
    int64_t ldq;
    int32_t *ids;
    float *dists;
    sa_query_stats *stats;
    unsigned long long *ghash;   // per query: 2^glog2 table entries, then 2^glog2 slot indices
    int64_t n;
    int32_t d, metric, R, entry, k, L, M, sync, static_I, staged, max_substeps;
    double rho;
    int32_t glog2, llog2;        // llog2 == 0: no LDS table
    int32_t glog2_init;          // single worker: log2 of the table a query starts in (<= glog2)
    // single worker over integer-valued float32 vectors in [int_lo, int_hi] (see
    // index_integer_range): pass 1 takes the queries that are integers in that range and
    // accumulates in float32, pass 0 takes the others; -1: one pass takes every query, in
    // double; 2: one pass takes every query, each in the arithmetic it allows
    int32_t int_lo, int_hi, acc_pass;
    int32_t idbits;              // vertex ids fit in idbits bits (2^idbits >= n)
    int32_t seen_log2;           // single-worker kernel: log2 of the seen filter's sets (set by its launcher)
    // batches: per-query L and k (null: L and k above) and the query each workgroup
    // runs (null: workgroup b runs query b)
    const int32_t *qL, *qk, *order;
    int64_t ldo;                 // row stride of ids and dists
    // persistent form (null: one workgroup per job): jobctr[0] hands out the jobs 0 ..
    // njobs - 1, jobctr[1] counts the workgroups that found none left; both are zero
    // before a launch and the last workgroup sets them back to zero
    int32_t *jobctr;
    int32_t njobs;
    int64_t company;             // host: queries of other launches on the device (see SearchLaunch)
};

// Persistent form, end of a workgroup (one thread): the last one to finish puts the job
// counters back to zero for the next launch.
__device__ __forceinline__ void release_jobs(int32_t *ctr)
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    if (atomicAdd(ctr + 1, 1) == (int)gridDim.x - 1) {
        atomicExch(ctr, 0);
        atomicExch(ctr + 1, 0);
    }
}

// set bits of the wave-uniform m in the lanes below this one
__device__ __forceinline__ int bits_below(uint64_t m)
{
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

__device__ __forceinline__ uint32_t rdlane(uint32_t v, int l) { return (uint32_t)__builtin_amdgcn_readlane((int)v, l); }
__device__ __forceinline__ uint64_t rdlane64(uint64_t v, int l)
{
    return ((uint64_t)rdlane((uint32_t)(v >> 32), l) << 32) | rdlane((uint32_t)v, l);
}

// lower_bound: number of entries of the sorted array a[0..n) smaller than key
__device__ __forceinline__ int lower_bound(const uint64_t *a, int n, uint64_t key)
{
    int lo = 0, hi = n;
    while (lo < hi) {
        int mid = (lo + hi) >> 1;
        if (a[mid] < key) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// ---------------------------------------------------------------- cross-lane helpers

constexpr int DPP_ROW_SHR = 0x110;     // + n: row_shr:n
constexpr int DPP_ROW_BCAST15 = 0x142;
constexpr int DPP_ROW_BCAST31 = 0x143;

// lanes whose DPP source is invalid (outside the row or the enabled rows) keep `old`
template <int CTRL, int ROWMASK = 0xF>
__device__ __forceinline__ uint32_t dpp32(uint32_t v, uint32_t old)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)v, CTRL, ROWMASK, 0xF, false);
}

// v of the lane N below in its row of 16, zero in the first N lanes (in a form that the
// compiler folds into the instruction that uses it)
template <int N>
__device__ __forceinline__ uint32_t row_shr0(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, DPP_ROW_SHR + N, 0xF, 0xF, true);
}

template <int CTRL, int ROWMASK = 0xF>
__device__ __forceinline__ double dpp_f64(double v)
{
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = dpp32<CTRL, ROWMASK>((uint32_t)b, 0u);
    const uint32_t hi = dpp32<CTRL, ROWMASK>((uint32_t)(b >> 32), 0u);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// sum of each group of LPV lanes, left in the group's last lane
template <int LPV>
__device__ __forceinline__ double group_sum(double v)
{
    if constexpr (LPV >= 2) v += dpp_f64<DPP_ROW_SHR + 1>(v);
    if constexpr (LPV >= 4) v += dpp_f64<DPP_ROW_SHR + 2>(v);
    if constexpr (LPV >= 8) v += dpp_f64<DPP_ROW_SHR + 4>(v);
    if constexpr (LPV >= 16) v += dpp_f64<DPP_ROW_SHR + 8>(v);
    if constexpr (LPV >= 32) v += dpp_f64<DPP_ROW_BCAST15, 0xA>(v);
    if constexpr (LPV >= 64) v += dpp_f64<DPP_ROW_BCAST31, 0xC>(v);
    return v;
}

// the same sums in float32
template <int LPV>
__device__ __forceinline__ float group_sum_f32(float v)
{
    if constexpr (LPV >= 2) v += __uint_as_float(row_shr0<1>(__float_as_uint(v)));
    if constexpr (LPV >= 4) v += __uint_as_float(row_shr0<2>(__float_as_uint(v)));
    if constexpr (LPV >= 8) v += __uint_as_float(row_shr0<4>(__float_as_uint(v)));
    if constexpr (LPV >= 16) v += __uint_as_float(row_shr0<8>(__float_as_uint(v)));
    if constexpr (LPV >= 32) v += __uint_as_float(dpp32<DPP_ROW_BCAST15, 0xA>(__float_as_uint(v), 0u));
    if constexpr (LPV >= 64) v += __uint_as_float(dpp32<DPP_ROW_BCAST31, 0xC>(__float_as_uint(v), 0u));
    return v;
}

// The smallest key among the lanes and a lane that holds it.
__device__ __forceinline__ uint64_t min_key(uint64_t k, int *at)
{
    const auto wave_min = [](uint32_t v) {
        v = min(v, dpp32<DPP_ROW_SHR + 1>(v, v));
        v = min(v, dpp32<DPP_ROW_SHR + 2>(v, v));
        v = min(v, dpp32<DPP_ROW_SHR + 4>(v, v));
        v = min(v, dpp32<DPP_ROW_SHR + 8>(v, v));
        v = min(v, dpp32<DPP_ROW_BCAST15, 0xA>(v, v));
        v = min(v, dpp32<DPP_ROW_BCAST31, 0xC>(v, v));
        return rdlane(v, 63);
    };
    const uint32_t hi = wave_min((uint32_t)(k >> 32));
    uint64_t b = __ballot((uint32_t)(k >> 32) == hi);
    if (b & (b - 1ull)) {
        const uint32_t lo = wave_min((b >> __lane_id()) & 1ull ? (uint32_t)k : 0xFFFFFFFFu);
        b &= __ballot((uint32_t)k == lo);
    }
    *at = __builtin_ctzll(b);
    return rdlane64(k, *at);
}

// lanes per vector: the smallest power of two that leaves at most four float4 chunks per
// lane (d <= 1024)
__host__ __device__ inline int lanes_per_vector(int d)
{
    const int nch = d / 4;
    int lpv = 1;
    while (lpv < 64 && 4 * lpv < nch) lpv *= 2;
    return lpv;
}

// Where a kernel reads vectors: rows of ld elements of storage type DT (sa_dtype).
struct VecSrc {
    const void *p;
    const float *scale;   // SA_FP8E4M3 only
    int64_t ld;
};

// Four coordinates of a row as stored: this raw form is what stays in registers while the
// loads are in flight, and is decoded where the distance uses it.
template <int DT> struct Raw4T { using type = uint32_t; };
template <> struct Raw4T<SA_F32> { using type = float4; };
template <> struct Raw4T<SA_BF16> { using type = uint2; };
template <int DT> using Raw4 = typename Raw4T<DT>::type;

// How distances are accumulated: in double, in float32 (only where every partial sum is an
// integer below 2^24, so that the float32 sum is exact and equals the double one), or either
// by a flag of the query.
enum { ACC_F64 = 0, ACC_F32 = 1, ACC_EITHER = 2 };

// Partial sums of one pass (see distances), summed over each lane group and written as keys.
template <typename Acc, int LPV, bool L2, int DT, int PB>
__device__ __forceinline__ void pass_keys(int nch, const float *qs, const Raw4<DT> (&x)[PB][4], const float (&sc)[PB],
                                          const int32_t (&id)[PB], uint64_t *out)
{
    constexpr int VPW = 64 / LPV;
    constexpr int SURE = LPV == 1 ? 1 : 2;          // chunks inside the row for every lane
    constexpr bool F32 = std::is_same<Acc, float>::value;
    const int lane = __lane_id(), grp = lane / LPV, g = lane % LPV;
    Acc acc[PB];
#pragma unroll
    for (int pp = 0; pp < PB; ++pp) acc[pp] = 0;
    float4 an = reinterpret_cast<const float4 *>(qs)[g];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const bool in = i < SURE || g + LPV * i < nch;
        const float4 a = an;
        if (i < 3) an = reinterpret_cast<const float4 *>(qs)[g + LPV * (i + 1)];
        __builtin_amdgcn_sched_barrier(0);
        const Acc ax = (Acc)a.x, ay = (Acc)a.y, az = (Acc)a.z, aw = (Acc)a.w;
#pragma unroll
        for (int pp = 0; pp < PB; ++pp) {
            // codes outside the row are taken as code 0, which is 0.0 in every storage type
            float bx, by, bz, bw;
            if constexpr (DT == SA_F32) {
                bx = in ? x[pp][i].x : 0.f; by = in ? x[pp][i].y : 0.f;
                bz = in ? x[pp][i].z : 0.f; bw = in ? x[pp][i].w : 0.f;
            } else if constexpr (DT == SA_BF16) {
                const uint32_t lo = in ? x[pp][i].x : 0u, hi = in ? x[pp][i].y : 0u;
                bx = __uint_as_float(lo << 16); by = __uint_as_float(lo & 0xFFFF0000u);
                bz = __uint_as_float(hi << 16); bw = __uint_as_float(hi & 0xFFFF0000u);
            } else {
                // e4m3 -> f16 bit pattern, two codes at a time: same mantissa bits,
                // exponent bias 15 instead of 7, so every value, subnormals included,
                // comes out 2^-8 too small; 2^8 joins the scale, and s * 2^8 * v rounds
                // once like s * value.  (The hardware fp8 conversion gives the same
                // values for every code that is written, but not for codes 0x7F / 0xFF,
                // NaN in e4m3, which decode as 480 / -480 here.)
                typedef _Float16 half2v __attribute__((ext_vector_type(2)));
                const uint32_t w = in ? x[pp][i] : 0u, w1 = w >> 8;
                const uint32_t h02 = ((w & 0x007F007Fu) << 7) | ((w & 0x00800080u) << 8);
                const uint32_t h13 = ((w1 & 0x007F007Fu) << 7) | ((w1 & 0x00800080u) << 8);
                const half2v e02 = __builtin_bit_cast(half2v, h02), e13 = __builtin_bit_cast(half2v, h13);
                const float s8 = sc[pp] * 256.f;
                bx = s8 * (float)e02.x;
                by = s8 * (float)e13.x;
                bz = s8 * (float)e02.y;
                bw = s8 * (float)e13.y;
            }
            Acc s = acc[pp];
            if constexpr (L2) {
                const Acc t0 = ax - (Acc)bx, t1 = ay - (Acc)by, t2 = az - (Acc)bz, t3 = aw - (Acc)bw;
                if constexpr (F32) {
                    s = __builtin_fmaf(t0, t0, s); s = __builtin_fmaf(t1, t1, s);
                    s = __builtin_fmaf(t2, t2, s); s = __builtin_fmaf(t3, t3, s);
                } else {
                    s += t0 * t0; s += t1 * t1; s += t2 * t2; s += t3 * t3;
                }
            } else if constexpr (F32) {
                s = __builtin_fmaf(ax, bx, s); s = __builtin_fmaf(ay, by, s);
                s = __builtin_fmaf(az, bz, s); s = __builtin_fmaf(aw, bw, s);
            } else {
                s = __builtin_fma(ax, (Acc)bx, s); s = __builtin_fma(ay, (Acc)by, s);
                s = __builtin_fma(az, (Acc)bz, s); s = __builtin_fma(aw, (Acc)bw, s);
            }
            acc[pp] = s;
        }
    }
#pragma unroll
    for (int pp = 0; pp < PB; ++pp) {
        Acc s = acc[pp];
        if constexpr (F32) s = group_sum_f32<LPV>(s);
        else s = group_sum<LPV>(s);
        if (g == LPV - 1) out[pp * VPW + grp] = make_key(L2 ? (float)s : (float)(-s), id[pp]);
    }
}

// Keys of the vectors ids[0..n) (n <= 64) to out[0..n), 64 / LPV vectors per pass; qs is
// the query, zero padded to 16 LPV floats.  ids[n..64) must be rows of the index too (any;
// a pass reads them with the rest), and out[n..64) is overwritten.  The loads are issued
// unconditionally, from clamped addresses, and the empty asm keeps them there: a load that
// the compiler moves under a lane condition gets a wait of its own, which turns one memory
// round trip into two.  (Written as a pass loop over arrays: the same steps as a per-vector
// helper cost some twenty more registers.)
// PB: vectors per lane group in one pass (PB 64 / LPV a pass, each pass one memory round
// trip; each more in flight costs sixteen registers at d = 128).  With HALVES a last pass that
// needs half of them or fewer takes the half (9 registers at PB = 2, d = 128).
//
// The searches issue instructions for a quarter (many queries) to half (few) of a wave's
// life, so a pass is kept short: the query is read and converted once for all of its
// vectors, products that are exact (inner products of float32 in double, everything with
// float32 sums) go through one fused multiply-add, and only a lane's third and fourth chunk are
// masked, the ones that can lie past the row's end (LPV is the smallest power of two with
// 4 LPV >= chunks).
template <int LPV, bool L2, int DT, int ACC = ACC_F64, int PBMAX = 1, bool HALVES = false>
__device__ __forceinline__ void distances(const VecSrc &V, int d, const float *qs, const int32_t *ids, int n,
                                          uint64_t *out, bool exact32 = false)
{
    constexpr int VPW = 64 / LPV;
    constexpr int PB = PBMAX < LPV ? PBMAX : LPV;   // VPW PB <= 64
    constexpr int SURE = LPV == 1 ? 1 : 2;
    constexpr int CB = sizeof(Raw4<DT>);            // bytes of a chunk
    const int lane = __lane_id(), grp = lane / LPV, g = lane % LPV;
    const int nch = d >> 2;
    const uint64_t stride = (uint64_t)V.ld * (CB / 4);
    const char *const lane_base = static_cast<const char *>(V.p) + g * CB;
    for (int p0 = 0; p0 < n; p0 += VPW * PB) {
        if constexpr (HALVES && PB > 1)
            if (n - p0 <= VPW * PB / 2) {
                distances<LPV, L2, DT, ACC, PB / 2, true>(V, d, qs, ids + p0, n - p0, out + p0, exact32);
                return;
            }
        Raw4<DT> x[PB][4];
        float sc[PB];
        int32_t id[PB];
#pragma unroll
        for (int pp = 0; pp < PB; ++pp) {
            id[pp] = ids[p0 + pp * VPW + grp];
            const char *const row = lane_base + (uint64_t)(uint32_t)id[pp] * stride;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                x[pp][i] = *reinterpret_cast<const Raw4<DT> *>(
                    row + (i < SURE || g + LPV * i < nch ? LPV * i * CB : 0));
            sc[pp] = DT == SA_FP8E4M3 ? V.scale[id[pp]] : 1.f;
        }
        asm volatile("" ::: "memory");
        if constexpr (ACC == ACC_F32) pass_keys<float, LPV, L2, DT, PB>(nch, qs, x, sc, id, out + p0);
        else if constexpr (ACC == ACC_F64) pass_keys<double, LPV, L2, DT, PB>(nch, qs, x, sc, id, out + p0);
        else if (exact32) pass_keys<float, LPV, L2, DT, PB>(nch, qs, x, sc, id, out + p0);
        else pass_keys<double, LPV, L2, DT, PB>(nch, qs, x, sc, id, out + p0);
    }
}

// Where a query leaves its final list for the re-rank: the last 1025 entries of its slot
// list (a count, then up to 1024 ids).  Slots stop at three quarters of a table of at
// least 4096, so the search never writes there; the re-rank zeroes it again.
__device__ __forceinline__ int32_t *rerank_list(uint32_t *slots, int glog2)
{
    return reinterpret_cast<int32_t *>(slots + (1u << glog2) - 1025u);
}

// The kernels of several workers keep S as a sorted array of entries: keys with the id moved
// up by one bit and the unchecked flag below it, which leaves their order.
__device__ __forceinline__ uint64_t entry_of(uint64_t key, uint32_t unchecked)
{
    return (key & 0xFFFFFFFF00000000ull) | ((uint32_t)key << 1) | unchecked;
}
__device__ __forceinline__ int32_t entry_id(uint64_t e) { return (int32_t)((uint32_t)e >> 1); }
__device__ __forceinline__ uint64_t key_of(uint64_t e) { return (e & 0xFFFFFFFF00000000ull) | ((uint32_t)e >> 1); }

}  // namespace search_detail

int launch_rerank(const float *vec32, int64_t ld32, const float *queries, int64_t ldq, int64_t nq, int32_t d,
                  int32_t metric, int32_t k, int32_t L, void *ws, int64_t stride, int64_t list_off, int32_t *ids,
                  float *dists, const int32_t *order, const int32_t *qk, int64_t ldo, hipStream_t s);
int launch_search_single_f32(const search_detail::KArgs &A, int64_t nq, hipStream_t s);
int launch_search_single_bf16(const search_detail::KArgs &A, int64_t nq, hipStream_t s);
int launch_search_single_fp8(const search_detail::KArgs &A, int64_t nq, hipStream_t s);
// the forms for few queries; *taken tells whether the launch suits them (and was made)
int launch_search_few_f32(const search_detail::KArgs &A, int64_t nq, hipStream_t s, bool *taken);
int launch_search_few_bf16(const search_detail::KArgs &A, int64_t nq, hipStream_t s, bool *taken);
int launch_search_few_fp8(const search_detail::KArgs &A, int64_t nq, hipStream_t s, bool *taken);
int launch_search_bsp(const search_detail::KArgs &A, int dtype, int64_t nq, hipStream_t s);
int launch_search_multi_f32(const search_detail::KArgs &A, int64_t nq, hipStream_t s);
int launch_search_multi_large_f32(const search_detail::KArgs &A, int64_t nq, hipStream_t s);
int launch_search_multi_bf16(const search_detail::KArgs &A, int64_t nq, hipStream_t s);
int launch_search_multi_large_bf16(const search_detail::KArgs &A, int64_t nq, hipStream_t s);
int launch_search_multi_fp8(const search_detail::KArgs &A, int64_t nq, hipStream_t s);
int launch_search_multi_large_fp8(const search_detail::KArgs &A, int64_t nq, hipStream_t s);

}  // namespace sa
