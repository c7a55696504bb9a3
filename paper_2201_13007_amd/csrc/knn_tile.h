// Matrix-core kNN: the tile layout, the product-and-filter kernel and the selection
// kernel shared by the integer and the float form (knn_mfma.hip says why each is exact).
//
// The base is processed in stages.  Stage 0 computes all distances to a first sample of
// 256 to 1024 rows; after every stage a selection keeps each query's kt smallest keys, and the
// kt-th of them bounds what a later row has to beat.  A later stage is a plain matrix
// product whose results are compared with that bound in registers: only the few that pass
// (about kt per doubling of the rows seen) are appended to a buffer, so the product loop
// holds no list, no sort and one barrier per tile, and the base can be split over as many
// workgroups as the device holds however few the queries are.  (Keeping sorted lists
// inside the product kernel, one workgroup per 64 queries for the whole base, took 17.4 ms
// for 10,000 queries over 1M x 128 integer rows: 157 workgroups on 256 CUs, a barrier and
// a flush test every tile.)
//
// Rows are dealt to tiles so that every tile, and every run of tiles, samples the whole
// base: position 64 t + o holds row o * ntile + tab[t], tab a golden-ratio permutation.
// A stage's threshold then fits the rows of the next one however the base is ordered.
// Where it does not all the same, a buffer overflows, which is counted, and that query is
// answered by the scan instead.
//
// Layout.  Base and query copies are stored in the operand order of
// v_mfma_f32_16x16x32_bf16: blocks of 16 rows, within a block [part][k-step][lane] 16-byte
// pieces (lane l: row l % 16, dimensions 8 (l / 16) .. + 7 of the k-step), so a wavefront
// moves a 1 KB operand with one coalesced load, straight into LDS, and reads it back
// without bank conflicts.
#pragma once
#include "knn_select.h"

#include <climits>

namespace sa {
namespace knn_tile {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;

constexpr int TROWS = 64;       // base rows per tile
constexpr int SELCAP = 2048;    // keys a selection can hold
constexpr int MAX_SPLITS = 1024;

// How a product becomes the value v the filter compares:
//   FLOAT   v = fma(s, q.x, |x|^2), the approximate distance less |q|^2
//   INT     queries stored times -2 (or -1): v = acc + |x|^2, rounded once from the exact
//           integer (a sum of even integers is exact to 2^25, and 2 * 256 * 255^2 is below)
//   FOLDED  the same with |x|^2 + 2 |q| |x| < 2^24: the accumulators start at |x|^2, every
//           partial sum is still an exact integer, so v is the accumulator itself and the
//           filter one comparison per product (at 10,000 x 1M x 128 the last stage had 4.4
//           vector instructions per matrix instruction without it, and the matrix cores
//           were busy half the time)
enum Form { FLOAT = 0, INT = 1, FOLDED = 2 };

struct TileArgs {
    const unsigned char *xt;   // base blocks
    const float *xn;           // per position: |x|^2 (0 for the inner product), +inf for padding
    const int32_t *tab;        // tile -> its row offset
    const unsigned char *qt;   // query blocks of this call's queries
    const void *qn;            // their |q|^2 (int32 for integer data, else float)
    int64_t n, q0;             // q0: index of the first query in the caller's array
    int32_t nq, ntile, t0, t1, splits, qtiles, nks;
    float s;                   // -2 (squared l2) or -1 (inner product)
    int32_t dense, exclude_self, capseg;
    const uint64_t *thr;       // per query: keys below it pass (KEY_EMPTY: all, 0: none)
    uint64_t *buf;             // passing keys: [query][split][capseg], or [query][rows] when dense
    int32_t *cnt;              // [query][split] keys that passed (may exceed capseg)
};

// Workgroup -> (split, query tile).  Workgroups go to the 8 XCDs round robin; each XCD gets
// a contiguous run of splits with all their query tiles, so the tiles of a split are read
// into one L2 by workgroups that run at the same time.
__device__ __forceinline__ bool tile_job(const TileArgs &A, int &split, int &qtile)
{
    const int total = A.splits * A.qtiles, per = (total + 7) / 8;
    const int j = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per || j >= total) return false;
    split = j / A.qtiles;
    qtile = j - split * A.qtiles;
    return true;
}

// 1 KB from global memory to LDS: lane l's 16 bytes go to dst + 16 l
__device__ __forceinline__ void load_1k(const unsigned char *src, unsigned char *dst)
{
    __builtin_amdgcn_global_load_lds(
        (const __attribute__((address_space(1))) void *)(src + 16 * __lane_id()),
        (__attribute__((address_space(3))) void *)dst, 16, 0, 0);
}

__device__ __forceinline__ void load_256b(const float *src, unsigned char *dst)
{
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src + __lane_id()),
                                     (__attribute__((address_space(3))) void *)dst, 4, 0, 0);
}

__device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// The largest float (rounded as the products are) a passing product may have.  Integer
// data: distances are roundings of integers, so the float of key thr is integral; below
// 2^24 it is exact, above it one unit in the last place covers every integer that rounds
// down onto it; u <= B implies round(u) <= round(B).
template <int FORM>
__device__ __forceinline__ float filter_bound(uint64_t thr, int32_t qnorm)
{
    if (thr == 0) return -__builtin_inff();
    if (thr == KEY_EMPTY) return __builtin_inff();
    const float f = key_dist(thr);
    if constexpr (FORM == FLOAT) return f;
    int64_t t = (int64_t)f;
    const float a = fabsf(f);
    if (a >= 16777216.f) t += int64_t(1) << ((int)((__float_as_uint(a) >> 23) & 0xFF) - 127 - 23);
    return (float)(t - qnorm);
}

template <int FORM>
__device__ __forceinline__ float filter_value(float s, float acc, float nx)
{
    return FORM == FOLDED ? acc : __builtin_fmaf(s, acc, nx);
}

// The results of one 16-row block against four query blocks: lane l holds rows 4 (l / 16)
// + r (norms nx) for the queries 16 qb + l % 16.  The few that pass the bounds are taken
// one per lane and turn in a loop of their own: unrolled over the sixteen, the compiler
// keeps their buffer addresses in registers across the product loop (236 registers
// instead of 128 at d = 128, two wavefronts per SIMD instead of four).  slot0: this
// lane's place, for qb = 0, in the workgroup's counters, thresholds and norms; o0: offset
// of row r = 0 in tile t, whose row offset is trow.
template <int FORM>
__device__ __forceinline__ void filter_append(const TileArgs &A, int split, int qfirst, int slot0, int32_t t, int32_t trow,
                                              int o0, const f32x4 (&acc)[4], const f32x4 &nx, const float (&bq)[4],
                                              int *cnt, const uint64_t *thr, const int32_t *qn)
{
    bool any = A.dense != 0;
#pragma unroll
    for (int qb = 0; qb < 4; ++qb)
#pragma unroll
        for (int r = 0; r < 4; ++r) any |= filter_value<FORM>(A.s, acc[qb][r], nx[r]) <= bq[qb];
    if (!__ballot(any)) return;
    uint32_t mask = 0;
#pragma unroll
    for (int qb = 0; qb < 4; ++qb)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            mask |= A.dense || filter_value<FORM>(A.s, acc[qb][r], nx[r]) <= bq[qb] ? 1u << (4 * qb + r) : 0u;
    while (mask) {
        const int i = __builtin_ctz(mask), qb = i >> 2, r = i & 3;
        mask &= mask - 1;
        float v = acc[0][0];
#pragma unroll
        for (int c = 1; c < 16; ++c) v = i == c ? acc[c >> 2][c & 3] : v;
        const float nv = r == 0 ? nx[0] : r == 1 ? nx[1] : r == 2 ? nx[2] : nx[3];
        const int slot = slot0 + 16 * qb, ql = qfirst + slot, o = o0 + r;
        if (ql >= A.nq) continue;
        const int64_t id = (int64_t)o * A.ntile + trow;
        const bool valid = id < A.n && !(A.exclude_self && id == A.q0 + ql);
        uint64_t key = KEY_EMPTY;
        if (valid) {
            if constexpr (FORM == FLOAT) key = make_key(__builtin_fmaf(A.s, v, nv), (int32_t)id);
            else key = make_key((float)(qn[slot] + (FORM == FOLDED ? (int)v : (int)nv + (int)A.s * (int)v)), (int32_t)id);
        }
        if (A.dense) {
            A.buf[(int64_t)ql * ((A.t1 - A.t0) * TROWS) + (t - A.t0) * TROWS + o] = key;
        } else if (key < thr[slot]) {
            const int pos = atomicAdd(&cnt[slot], 1);
            if (pos < A.capseg) A.buf[((int64_t)ql * A.splits + split) * A.capseg + pos] = key;
        }
    }
}

// Queries in registers.  Four wavefronts; WQ of them hold 64 queries each and the others
// repeat those queries on other rows of the tile (WQ = 4 for many queries, 1 for at most
// 64).  Base tiles of 64 rows stream through two LDS buffers, the next one in flight while
// the current one multiplies.  NP parts per coordinate: 1 (bf16 holds it), or 2 (hi and
// lo; three products hi.hi + lo.hi + hi.lo).
template <int KS, int NP, int WQ, int FORM>
__global__ void __launch_bounds__(256, KS * NP <= 4 ? 4 : 2) knn_tile_kernel(TileArgs A)
{
    constexpr int TILE = 4 * KS * NP * 1024, STAGE = TILE + 256;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    uint64_t *const thr = reinterpret_cast<uint64_t *>(smem + 2 * STAGE);   // [64 WQ]
    int *const cnt = reinterpret_cast<int *>(thr + 64 * WQ);                 // [64 WQ]
    int32_t *const qns = cnt + 64 * WQ;                                      // [64 WQ]
    int split, qtile;
    if (!tile_job(A, split, qtile)) return;
    const int tid = threadIdx.x, lane = __lane_id();
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wq = w % WQ, wr = w / WQ;
    const int qfirst = qtile * 64 * WQ;
    for (int i = tid; i < 64 * WQ; i += 256) {
        const int q = qfirst + i;
        cnt[i] = 0;
        thr[i] = q < A.nq ? A.thr[q] : 0ull;
        qns[i] = FORM != FLOAT && q < A.nq ? static_cast<const int32_t *>(A.qn)[q] : 0;
    }
    bf16x8 q[4][NP][KS];
    {
        const unsigned char *p = A.qt + (int64_t)(qfirst / 16 + 4 * wq) * (NP * KS * 1024) + 16 * lane;
#pragma unroll
        for (int qb = 0; qb < 4; ++qb)
#pragma unroll
            for (int pt = 0; pt < NP; ++pt)
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
                    q[qb][pt][ks] = *reinterpret_cast<const bf16x8 *>(p + ((qb * NP + pt) * KS + ks) * 1024);
    }
    __syncthreads();
    float bq[4];
#pragma unroll
    for (int qb = 0; qb < 4; ++qb) {
        const int i = 64 * wq + 16 * qb + (lane & 15);
        bq[qb] = filter_bound<FORM>(thr[i], qns[i]);
    }
    const int ntl = A.t1 - A.t0;
    const int ta = A.t0 + (int)((int64_t)ntl * split / A.splits), tb = A.t0 + (int)((int64_t)ntl * (split + 1) / A.splits);
    auto fetch = [&](int t, int b) {
        const unsigned char *src = A.xt + (int64_t)t * TILE;
        unsigned char *dst = smem + b * STAGE;
#pragma unroll
        for (int c = 0; c < KS * NP; ++c) load_1k(src + (4 * c + w) * 1024, dst + (4 * c + w) * 1024);
        if (w == 0) load_256b(A.xn + (int64_t)t * TROWS, dst + TILE);
    };
    if (ta < tb) fetch(ta, 0);
    wait_loads();
    __syncthreads();
    for (int t = ta; t < tb; ++t) {
        const int b = (t - ta) & 1;
        if (t + 1 < tb) fetch(t + 1, b ^ 1);
        const unsigned char *tile = smem + b * STAGE;
        const int32_t trow = A.tab[t];
#pragma unroll 1
        for (int rr = 0; rr < WQ; ++rr) {
            const int rb = WQ == 4 ? rr : wr * WQ + rr;
            const f32x4 nx = *reinterpret_cast<const f32x4 *>(tile + TILE + (rb * 16 + 4 * (lane >> 4)) * 4);
            f32x4 acc[4];
#pragma unroll
            for (int qb = 0; qb < 4; ++qb) acc[qb] = FORM == FOLDED ? nx : f32x4{0.f, 0.f, 0.f, 0.f};
            const unsigned char *xp = tile + rb * (NP * KS * 1024) + 16 * lane;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const bf16x8 xh = *reinterpret_cast<const bf16x8 *>(xp + ks * 1024);
#pragma unroll
                for (int qb = 0; qb < 4; ++qb)
                    acc[qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xh, q[qb][0][ks], acc[qb], 0, 0, 0);
                if constexpr (NP == 2) {
                    const bf16x8 xl = *reinterpret_cast<const bf16x8 *>(xp + (KS + ks) * 1024);
#pragma unroll
                    for (int qb = 0; qb < 4; ++qb)
                        acc[qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xl, q[qb][0][ks], acc[qb], 0, 0, 0);
#pragma unroll
                    for (int qb = 0; qb < 4; ++qb)
                        acc[qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xh, q[qb][1][ks], acc[qb], 0, 0, 0);
                }
            }
            filter_append<FORM>(A, split, qfirst, 64 * wq + (lane & 15), t, trow, rb * 16 + 4 * (lane >> 4), acc, nx, bq, cnt,
                               thr, qns);
        }
        wait_loads();      // the next tile is in LDS before any wavefront passes the barrier
        __syncthreads();
    }
    if (!A.dense)
        for (int i = tid; i < 64 * WQ; i += 256)
            if (qfirst + i < A.nq) A.cnt[(int64_t)(qfirst + i) * A.splits + split] = cnt[i];
}

// Queries too wide for registers (two parts, d > 128): a workgroup multiplies 128 rows by
// 128 queries, 64 x 64 per wavefront (64 accumulator registers), and both operands of each
// 32-dimension step go through two LDS buffers of 32 KB, the next step in flight while the
// current one multiplies: 48 matrix instructions per wavefront against 16 LDS reads of
// 1 KB, two workgroups per CU.
__global__ void __launch_bounds__(256, 2) knn_tile_wide_kernel(TileArgs A)
{
    constexpr int NP = 2, QN = 128, STEP = 32 * 1024;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    uint64_t *const thr = reinterpret_cast<uint64_t *>(smem + 2 * STEP);   // [128]
    int *const cnt = reinterpret_cast<int *>(thr + QN);                     // [128]
    int split, qtile;
    if (!tile_job(A, split, qtile)) return;
    const int tid = threadIdx.x, lane = __lane_id();
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wq = w & 1, wb = w >> 1;
    const int qfirst = qtile * QN, nks = A.nks;
    const int64_t blk = (int64_t)NP * nks * 1024;   // bytes of a 16-row block
    for (int i = tid; i < QN; i += 256) {
        cnt[i] = 0;
        thr[i] = qfirst + i < A.nq ? A.thr[qfirst + i] : 0ull;
    }
    __syncthreads();
    float bq[4];
#pragma unroll
    for (int qb = 0; qb < 4; ++qb) bq[qb] = filter_bound<FLOAT>(thr[64 * wq + 16 * qb + (lane & 15)], 0);
    // tile pairs [ta, tb) of this split; stages begin and end at even tiles
    const int npair = (A.t1 - A.t0) / 2;
    const int ta = A.t0 / 2 + (int)((int64_t)npair * split / A.splits);
    const int tb = A.t0 / 2 + (int)((int64_t)npair * (split + 1) / A.splits);
    const unsigned char *const qsrc = A.qt + (int64_t)(qfirst / 16) * blk;
    // step buffer: 16 pieces of the rows ([block][part]), then 16 of the queries
    auto fetch = [&](int pr, int ks, int b) {
        const unsigned char *xsrc = A.xt + (int64_t)pr * 8 * blk;
        unsigned char *dst = smem + b * STEP;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int pc = 4 * c + w;   // piece: block pc / 2, part pc % 2
            const int64_t off = (pc >> 1) * blk + ((int64_t)(pc & 1) * nks + ks) * 1024;
            load_1k(xsrc + off, dst + pc * 1024);
            load_1k(qsrc + off, dst + (16 + pc) * 1024);
        }
    };
    f32x4 acc[4][4];   // [row block][query block]
#pragma unroll
    for (int rb = 0; rb < 4; ++rb)
#pragma unroll
        for (int qb = 0; qb < 4; ++qb) acc[rb][qb] = f32x4{0.f, 0.f, 0.f, 0.f};
    int pr = ta, ks = 0, b = 0;
    if (ta < tb) fetch(pr, 0, 0);
    wait_loads();
    __syncthreads();
    while (pr < tb) {
        const int ksn = ks + 1 < nks ? ks + 1 : 0, prn = ksn ? pr : pr + 1;
        if (prn < tb) fetch(prn, ksn, b ^ 1);
        const unsigned char *const xs = smem + b * STEP + wb * 8 * 1024 + 16 * lane;
        const unsigned char *const qs_ = smem + b * STEP + (16 + wq * 8) * 1024 + 16 * lane;
        bf16x8 qh[4], ql[4];
#pragma unroll
        for (int qb = 0; qb < 4; ++qb) {
            qh[qb] = *reinterpret_cast<const bf16x8 *>(qs_ + (2 * qb) * 1024);
            ql[qb] = *reinterpret_cast<const bf16x8 *>(qs_ + (2 * qb + 1) * 1024);
        }
#pragma unroll
        for (int rb = 0; rb < 4; ++rb) {
            const bf16x8 xh = *reinterpret_cast<const bf16x8 *>(xs + (2 * rb) * 1024);
            const bf16x8 xl = *reinterpret_cast<const bf16x8 *>(xs + (2 * rb + 1) * 1024);
#pragma unroll
            for (int qb = 0; qb < 4; ++qb) acc[rb][qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xh, qh[qb], acc[rb][qb], 0, 0, 0);
#pragma unroll
            for (int qb = 0; qb < 4; ++qb) acc[rb][qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xl, qh[qb], acc[rb][qb], 0, 0, 0);
#pragma unroll
            for (int qb = 0; qb < 4; ++qb) acc[rb][qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xh, ql[qb], acc[rb][qb], 0, 0, 0);
        }
        if (ksn == 0) {
            const int t = 2 * pr + wb;
            const int32_t trow = A.tab[t];
#pragma unroll
            for (int rb = 0; rb < 4; ++rb) {
                const f32x4 nx = *reinterpret_cast<const f32x4 *>(A.xn + (int64_t)t * TROWS + rb * 16 + 4 * (lane >> 4));
                filter_append<FLOAT>(A, split, qfirst, 64 * wq + (lane & 15), t, trow, rb * 16 + 4 * (lane >> 4), acc[rb],
                                     nx, bq, cnt, thr, nullptr);
#pragma unroll
                for (int qb = 0; qb < 4; ++qb) acc[rb][qb] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
        }
        wait_loads();
        __syncthreads();
        pr = prn;
        ks = ksn;
        b ^= 1;
    }
    if (!A.dense)
        for (int i = tid; i < QN; i += 256)
            if (qfirst + i < A.nq) A.cnt[(int64_t)(qfirst + i) * A.splits + split] = cnt[i];
}

struct SelArgs {
    const uint64_t *buf;
    const int32_t *cnt;
    int32_t splits, capseg, dense_rows;   // dense_rows > 0: that many keys per query, no counters
    int32_t kt, nq, first;                // first: no list yet
    int32_t cap;                          // a selection by one wavefront sorts at most so many keys (a power of two >= kt)
    uint64_t *list;                       // [query][kt] smallest keys so far, sorted (KEY_EMPTY past the end)
    uint64_t *thr;
    int32_t *over;                        // per query: a buffer overflowed
    // last stage of the integer form (ids null otherwise): the first k keys are the results of
    // query q0 + q; queries whose buffers overflowed are listed for the scan instead
    int32_t *ids;
    float *dists;
    int64_t q0;
    int32_t k;
    int32_t *failed, *failed_list;
};

__device__ __forceinline__ void put_result(const SelArgs &S, int64_t q, int i, uint64_t key)
{
    if (!S.ids || i >= S.k) return;
    const bool ok = key != KEY_EMPTY;
    S.ids[(S.q0 + q) * S.k + i] = ok ? key_id(key) : -1;
    S.dists[(S.q0 + q) * S.k + i] = ok ? key_dist(key) : __builtin_inff();
}

// one lane: the query's buffer overflowed
__device__ __forceinline__ void give_up(const SelArgs &S, int64_t q)
{
    S.over[q] = 1;
    S.thr[q] = 0ull;   // (answered elsewhere: nothing more passes for this query)
    if (S.ids) S.failed_list[atomicAdd(S.failed, 1)] = (int32_t)(S.q0 + q);
}

// sorts the P (a power of two) keys of LDS array a, ascending, with the whole workgroup
__device__ __forceinline__ void sort_lds(uint64_t *a, int P)
{
    for (int k = 2; k <= P; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            __syncthreads();
            for (int i = threadIdx.x; i < P / 2; i += blockDim.x) {
                const int lo = ((i & ~(j - 1)) << 1) | (i & (j - 1)), hi = lo | j;
                const uint64_t x = a[lo], y = a[hi];
                if ((x > y) == ((lo & k) == 0)) {
                    a[lo] = y;
                    a[hi] = x;
                }
            }
        }
    __syncthreads();
}

// the same with one wavefront (the arrays of several in one workgroup)
__device__ __forceinline__ void sort_lds_wave(uint64_t *a, int P)
{
    const int lane = __lane_id();
    for (int k = 2; k <= P; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            for (int i = lane; i < P / 2; i += 64) {
                const int lo = ((i & ~(j - 1)) << 1) | (i & (j - 1)), hi = lo | j;
                const uint64_t x = a[lo], y = a[hi];
                if ((x > y) == ((lo & k) == 0)) {
                    a[lo] = y;
                    a[hi] = x;
                }
            }
        }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// knn_select_kernel with one wavefront per query, four queries per workgroup: at most 256
// segments and 64 NK keys, held in registers.  The kt smallest are first cut out by
// bisection on the key (counts by ballot, no memory; it stops when kt to S.cap keys are
// left, which a dozen steps reach) and only those are sorted in LDS (dynamic: 4 cap
// keys).  Sorting every key with a workgroup was bound by LDS: 50 us for 2,000 queries of
// 1,024 keys, 62 us for 10,000 of 120.
template <int NK>
__global__ void __launch_bounds__(256) knn_select_wave_kernel(SelArgs S)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ int pre_all[4][256];
    const int lane = __lane_id(), w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t q = (int64_t)blockIdx.x * 4 + w;
    if (q >= S.nq) return;
    uint64_t *const a = reinterpret_cast<uint64_t *>(smem) + (size_t)w * S.cap;
    int *const pre = pre_all[w];
    uint64_t key[NK];
    if (S.dense_rows > 0) {
#pragma unroll
        for (int j = 0; j < NK; ++j)
            key[j] = 64 * j + lane < S.dense_rows ? S.buf[q * S.dense_rows + 64 * j + lane] : KEY_EMPTY;
    } else {
        int c[4], sum = 0;
        bool over = false;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            c[j] = 4 * lane + j < S.splits ? S.cnt[q * S.splits + 4 * lane + j] : 0;
            over |= c[j] > S.capseg;
            sum += c[j];
        }
        int inc = sum;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int v = __shfl_up(inc, off, 64);
            if (lane >= off) inc += v;
        }
        const int total = __builtin_amdgcn_readlane(inc, 63);
        if (__ballot(over) != 0 || total + S.kt > 64 * NK || (!S.first && S.over[q])) {
            if (lane == 0) give_up(S, q);
            return;
        }
        int base = inc - sum;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            pre[4 * lane + j] = base;
            base += c[j];
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int j = 0; j < NK; ++j) {
            const int i = 64 * j + lane;
            key[j] = KEY_EMPTY;
            if (i < total) {
                int lo = 0, hi = S.splits - 1;   // the last segment whose prefix is <= i
                while (lo < hi) {
                    const int mid = (lo + hi + 1) >> 1;
                    if (pre[mid] <= i) lo = mid;
                    else hi = mid - 1;
                }
                key[j] = S.buf[(q * S.splits + lo) * S.capseg + (i - pre[lo])];
            } else if (i < total + S.kt) {
                key[j] = S.list[q * S.kt + i - total];
            }
        }
    }
    uint64_t mn = KEY_EMPTY, mx = 0;   // smallest key, largest but KEY_EMPTY
    int have = 0;
#pragma unroll
    for (int j = 0; j < NK; ++j) {
        mn = key[j] < mn ? key[j] : mn;
        if (key[j] != KEY_EMPTY && key[j] > mx) mx = key[j];
        have += __popcll(__ballot(key[j] != KEY_EMPTY));
    }
    uint64_t cut = KEY_EMPTY - 1;   // keys up to here are kept
    if (have > S.cap) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            const uint64_t u = (uint64_t)__shfl_xor((unsigned long long)mn, off, 64), v = (uint64_t)__shfl_xor((unsigned long long)mx, off, 64);
            mn = u < mn ? u : mn;
            mx = v > mx ? v : mx;
        }
        uint64_t lo = mn, hi = mx;   // at least kt keys are <= hi throughout
        while (lo < hi) {
            const uint64_t mid = lo + ((hi - lo) >> 1);
            int n = 0;
#pragma unroll
            for (int j = 0; j < NK; ++j) n += __popcll(__ballot(key[j] <= mid));
            if (n >= S.kt) {
                hi = mid;
                if (n <= S.cap) break;
            } else {
                lo = mid + 1;
            }
        }
        cut = hi;
    }
    int n = 0;
#pragma unroll
    for (int j = 0; j < NK; ++j) {
        const bool in = key[j] <= cut;
        const uint64_t m = __ballot(in);
        if (in) a[n + __popcll(m & ((1ull << lane) - 1ull))] = key[j];
        n += __popcll(m);
    }
    int P = 64;
    while (P < n) P <<= 1;
    for (int i = n + lane; i < P; i += 64) a[i] = KEY_EMPTY;
    sort_lds_wave(a, P);
    for (int i = lane; i < S.kt; i += 64) {
        const uint64_t v = i < P ? a[i] : KEY_EMPTY;
        S.list[q * S.kt + i] = v;
        put_result(S, q, i, v);
    }
    if (lane == 0) {
        S.thr[q] = S.kt <= n ? a[S.kt - 1] : KEY_EMPTY;
        if (S.first) S.over[q] = 0;
    }
}

// One workgroup per query: the kt smallest of the list so far and the keys the last stage
// appended.
__global__ void __launch_bounds__(256) knn_select_kernel(SelArgs S)
{
    __shared__ uint64_t a[SELCAP];
    __shared__ int pre[MAX_SPLITS + 1];
    __shared__ int part[4];
    __shared__ int over;
    const int q = blockIdx.x, tid = threadIdx.x, lane = __lane_id(), w = tid >> 6;
    int total = 0;
    if (S.dense_rows > 0) {
        total = S.dense_rows;
        for (int i = tid; i < total; i += 256) a[i] = S.buf[(int64_t)q * total + i];
    } else {
        // prefix sums of the segment counts (up to four per thread)
        if (tid == 0) over = S.first ? 0 : S.over[q];
        __syncthreads();
        int c[4], sum = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int sgm = 4 * tid + j;
            c[j] = sgm < S.splits ? S.cnt[(int64_t)q * S.splits + sgm] : 0;
            if (c[j] > S.capseg) over = 1;
            sum += c[j];
        }
        int inc = sum;
        for (int off = 1; off < 64; off <<= 1) {
            const int v = __shfl_up(inc, off, 64);
            if (lane >= off) inc += v;
        }
        if (lane == 63) part[w] = inc;
        __syncthreads();
        int base = inc - sum;
        for (int j = 0; j < w; ++j) base += part[j];
        total = part[0] + part[1] + part[2] + part[3];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            pre[4 * tid + j] = base;
            base += c[j];
        }
        if (total + S.kt > SELCAP && tid == 0) over = 1;
        __syncthreads();
        if (over) {
            if (tid == 0) give_up(S, q);
            return;
        }
        for (int i = tid; i < total; i += 256) {
            int lo = 0, hi = S.splits - 1;   // the last segment whose prefix is <= i
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (pre[mid] <= i) lo = mid;
                else hi = mid - 1;
            }
            a[i] = S.buf[((int64_t)q * S.splits + lo) * S.capseg + (i - pre[lo])];
        }
        for (int i = tid; i < S.kt; i += 256) a[total + i] = S.list[(int64_t)q * S.kt + i];
        total += S.kt;
    }
    int P = 64;
    while (P < total) P <<= 1;
    for (int i = total + tid; i < P; i += 256) a[i] = KEY_EMPTY;
    sort_lds(a, P);
    for (int i = tid; i < S.kt; i += 256) {
        const uint64_t v = i < P ? a[i] : KEY_EMPTY;
        S.list[(int64_t)q * S.kt + i] = v;
        put_result(S, q, i, v);
    }
    if (tid == 0) {
        S.thr[q] = S.kt <= P ? a[S.kt - 1] : KEY_EMPTY;
        if (S.first) S.over[q] = 0;
    }
}

}  // namespace knn_tile
}  // namespace sa
