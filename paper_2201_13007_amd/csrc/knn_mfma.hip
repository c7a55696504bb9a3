// Exact k nearest neighbours on the matrix cores, for integer-valued data and for finite
// floats, and the choice between this path and the double-precision scan of knn.hip.
//
// Exactness.  When every coordinate is an integer in [-255, 255] and d <= 256, bf16 holds
// each coordinate exactly, each product is an integer below 2^16 and every partial sum of
// a dot product stays below 256 * 255^2 < 2^24 in magnitude, so the fp32 accumulators of
// v_mfma_f32_16x16x32_bf16 hold the exact integer dot product whatever order the
// additions take.  The squared distance |q|^2 + |x|^2 - 2 q.x (or -q.x for the inner
// product) is then formed in 32-bit integers and rounded once to float, which is the key
// the scan produces, bit for bit.
//
// Both forms run the staged product-and-filter of knn_tile.h.  A product passes a cheap
// test first: round(|x|^2 - 2 q.x) <= round(B_q) with B_q = T_q - |q|^2, where T_q bounds
// from above every integer distance whose float rounding does not exceed the query's
// threshold key; only passing products build a 64-bit key and are compared with it.
//
// Float data (d <= 1024).  Each coordinate is split into bf16 parts x = h + l + r
// (h and l rounded to nearest even, so |x - h| <= 2^-8 |x| and |r| <= 2^-16 |x|) and
// q.x is approximated by qh.xh + qh.xl + ql.xh on the matrix cores with fp32 accumulation.
// Its error is at most c |q| |x| with c = 3.1 2^-16 + (3d + 2) 2^-24 (the omitted terms,
// then every fp32 rounding of the 3d products), so every approximate distance is within E_q of the exact
// one, with E_q from |q| and the largest |x| (doubled for safety).  For L2 all points are
// first moved by the base mean (distances unchanged, norms and so the bound smaller).  The
// stages keep the kt smallest approximate keys (128 up to k = 96, at least k + 32 beyond);
// the exact kernel rescores them with the scan's own FP64 arithmetic and keeps the k smallest exact keys.  Every
// point outside the list is then at least (kt-th approximate distance - E_q) away; if
// that exceeds the k-th exact key, none can enter the k best, and the result is the
// scan's, bit for bit.  The queries that cannot show that margin (ties within the bound)
// are listed and rescored by the scan alone.
#include "knn_tile.h"

#include <algorithm>
#include <cmath>
#include <numeric>
#include <vector>

namespace sa {
namespace {

constexpr int MNT = 256;   // four wavefronts

using knn_tile::SelArgs;
using knn_tile::TileArgs;
using knn_tile::TROWS;

struct PrepArgs {
    const float *x;
    int64_t n, ld, rows;   // rows: n rounded up to whole tiles (base) or workgroups (queries)
    int32_t d, ks;
    int64_t ntile, mul;    // base: position 64 t + o holds row o * ntile + (t * mul) % ntile; mul 0: its own row
    int32_t metric;
    unsigned char *out;    // blocks in operand order (knn_tile.h); null: only the check
    float *norm;           // base: |x|^2 (exact integers; 0 for the inner product), +inf for padding
    int32_t *qnorm;        // queries: |q|^2
    int32_t *tab;
    int32_t *bad;
    int32_t *max_norm;     // largest |x|^2 (null: not wanted)
    float scale;           // the copy holds scale * x (a power of two of either sign)
};

// One wavefront per block of 16 rows: the bf16 copy in operand order (zero padded), the
// exact integer squared norms, and a flag raised by any value that is not an integer in
// [-255, 255] (NaN included); once it is raised the remaining blocks do nothing.
__global__ void __launch_bounds__(256) knn_prep_kernel(PrepArgs P)
{
    const int lane = __lane_id();
    const int64_t blk = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (blk * 16 >= P.rows || __hip_atomic_load(P.bad, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return;
    const int r = lane & 15, g = lane >> 4;
    int64_t row = blk * 16 + r;
    if (P.mul) {
        const int64_t t = blk >> 2, off = (t * P.mul) % P.ntile;
        if ((blk & 3) == 0 && lane == 0) P.tab[t] = (int32_t)off;
        row = ((blk & 3) * 16 + r) * P.ntile + off;
    }
    const float *src = P.x + row * P.ld;
    int sum = 0;
    bool bad = false;
    for (int ks = 0; ks < P.ks; ++ks) {
        const int c = 32 * ks + 8 * g;
        float4 v[2];
#pragma unroll
        for (int h = 0; h < 2; ++h)
            v[h] = row < P.n && c + 4 * h < P.d ? *reinterpret_cast<const float4 *>(src + c + 4 * h) : make_float4(0.f, 0.f, 0.f, 0.f);
        const float f[8] = {v[0].x, v[0].y, v[0].z, v[0].w, v[1].x, v[1].y, v[1].z, v[1].w};
        knn_tile::bf16x8 o;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const bool ok = fabsf(f[i]) <= 255.f && f[i] == rintf(f[i]);
            bad |= !ok;
            const int iv = ok ? (int)f[i] : 0;
            sum += iv * iv;
            o[i] = (__bf16)(ok ? P.scale * f[i] : 0.f);
        }
        if (P.out) *reinterpret_cast<knn_tile::bf16x8 *>(P.out + (blk * P.ks + ks) * 1024 + 16 * lane) = o;
    }
    sum += __shfl_xor(sum, 16, 64);
    sum += __shfl_xor(sum, 32, 64);
    if (__ballot(bad) && lane == 0) atomicOr(P.bad, 1);
    if (P.max_norm) {
        int mx = sum;
        for (int o = 1; o < 16; o <<= 1) mx = max(mx, __shfl_xor(mx, o, 64));
        // (most blocks see a larger value there already: one address, few atomics)
        if (lane == 0 && mx > __hip_atomic_load(P.max_norm, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            atomicMax(P.max_norm, mx);
    }
    if (g == 0 && P.out) {
        const int nv = P.metric == SA_L2 ? sum : 0;
        if (P.qnorm) P.qnorm[blk * 16 + r] = nv;
        else P.norm[blk * 16 + r] = row < P.n ? (float)nv : __builtin_inff();
    }
}

// ---------------------------------------------------------------- stages (host)

struct Stage {
    int t0, t1, wq, qtiles, splits, capseg;
    int lane_keys;   // keys per lane of a selection by one wavefront; 0: by a workgroup
};

constexpr int QCHUNK = 65536;   // queries per pass over the base: bounds the buffers at 0.65 to 1.3 GB (kt = 24 to 320)

// The stages of one pass over the base for nq queries (wide: the 128 x 128 kernel, tile
// pairs): a first sample of the tiles, then each up to r times as many.  A stage lets
// about kt (r - 1) rows pass per query.  Few queries are bound by launches (a product and
// a selection each stage, some 15 us): a sample of 1024 rows and r up to 16; many by the
// keys (each passing one breaks the product loop for some hundred cycles and is then
// selected from): 256 rows up to kt = 64, 512 up to 128, and r up to 6.  Both within what
// a selection holds.
//   A workgroup takes 256 queries where that leaves 512 workgroups (two per CU), else 128
// or 64 (the stages of few tiles); a stage is split over two to four times the workgroups
// that the device holds (1024 to 2048), which bounds what an uneven last round costs.
//   From 256 queries up a wavefront selects per query, below a workgroup does (mostly: see `one`).
std::vector<Stage> plan_stages(int ntile, int kt, int64_t nq, bool wide)
{
    std::vector<Stage> st;
    const bool many = nq >= 4096;
    const int unit = wide ? 2 : 1;
    // Few queries over a base of up to 2048 rows: one stage.  From lists of up to 64 a wavefront
    // selects there too.  One query over 1,100 x 128 integers, k = 1: 102 us in two stages, 97 in
    // one, 72 with the wavefront; 100 over 2,000 x 512 floats: 224 and 192.
    const bool one = nq < 256 && ntile <= 32;
    const int m0 = one ? ntile : std::min(ntile, many && kt <= 64 ? 4 : many && kt <= 128 ? 8 : 16);
    const double rmax = std::min(many ? 6.0 : 16.0, std::max(3.0, 1024.0 / kt));
    const double ratio = (double)ntile / m0;
    const int ns = ratio > 1.0 ? std::max(1, (int)std::ceil(std::log(ratio) / std::log(rmax))) : 0;
    const double r = ns > 0 ? std::pow(ratio, 1.0 / ns) : 1.0;
    int t0 = 0;
    for (int i = 0; i <= ns; ++i) {
        int t1 = i == ns ? ntile : std::min(ntile, (int)(m0 * std::pow(r, i) / 2.0 + 0.5) * 2);
        if (i == 0) t1 = m0;
        if (t1 <= t0) continue;
        const int ntl = t1 - t0, most_splits = std::min(std::max(1, ntl / unit), knn_tile::MAX_SPLITS);
        Stage s{t0, t1, 2, 0, 1, 0, 0};
        if (!wide)
            for (s.wq = nq <= 64 ? 1 : nq <= 128 ? 2 : 4; s.wq > 1 && (nq + 64 * s.wq - 1) / (64 * s.wq) * most_splits < 512;)
                s.wq /= 2;
        s.qtiles = (int)((nq + 64 * s.wq - 1) / (64 * s.wq));
        const int target = (int64_t)ntl * s.qtiles >= 65536 ? 2048 : 1024;
        s.splits = std::max(1, std::min(target / s.qtiles, most_splits));
        double keys = (double)ntl * TROWS;   // a selection's keys, and its room for them
        if (t0 > 0) {
            // room for twice the expected keys and six deviations
            const double all = 2.0 * kt * ((double)ntl / t0), mu = all / s.splits;
            const int most = ((ntl + s.splits - 1) / s.splits + unit) * TROWS;
            s.capseg = std::min(most, ((int)(mu + 6.0 * std::sqrt(mu) + 16.0) + 1) / 2 * 2);
            keys = kt + all + 6.0 * std::sqrt(all);
        }
        if ((nq >= 256 || (one && kt <= 64)) && s.splits <= 256) {
            s.lane_keys = 4;
            while (s.lane_keys < 32 && 64 * s.lane_keys < keys) s.lane_keys *= 2;
        }
        st.push_back(s);
        t0 = t1;
    }
    return st;
}

// buffer bytes of a stage for nq queries
size_t stage_bytes(const Stage &s, int64_t nq)
{
    return s.t0 == 0 ? (size_t)nq * (s.t1 - s.t0) * TROWS * 8 : (size_t)nq * s.splits * s.capseg * 8;
}

// odd multiplier near 0.618 ntile that is prime to ntile: the tile permutation
int64_t tile_mul(int64_t ntile)
{
    int64_t m = std::max<int64_t>(1, (int64_t)(0.6180339887498949 * (double)ntile));
    while (std::gcd(m, ntile) != 1) ++m;
    return m;
}

struct DeviceBlock {
    void *p = nullptr;
    ~DeviceBlock()
    {
        if (p) (void)hipFree(p);
    }
};

size_t align256(size_t v) { return (v + 255) / 256 * 256; }

using TKernel = void (*)(TileArgs);

struct Kernels {
    TKernel k[3];   // for 64, 128 and 256 queries per workgroup
    TKernel of(int wq) const { return k[wq == 4 ? 2 : wq == 2 ? 1 : 0]; }
};

using SKernel = void (*)(SelArgs);

SKernel pick_select(int lane_keys)
{
    switch (lane_keys) {
    case 4: return knn_tile::knn_select_wave_kernel<4>;
    case 8: return knn_tile::knn_select_wave_kernel<8>;
    case 16: return knn_tile::knn_select_wave_kernel<16>;
    default: return knn_tile::knn_select_wave_kernel<32>;
    }
}

// The stages of one chunk of queries (A holds everything but the stage's own fields).
// lds_wq: bytes of LDS of the product kernel per 64 queries of its workgroup, on top of lds0
// out: where the last selection leaves results (ids null: nowhere)
int run_stages(TileArgs A, const std::vector<Stage> &st, const Kernels &kern, size_t lds0, size_t lds_wq, int kt,
               uint64_t *list, uint64_t *thr, int32_t *over, const SelArgs &out, hipStream_t s)
{
    bool first = true;
    int sort_cap = 64;
    while (sort_cap < 2 * kt) sort_cap *= 2;
    for (const Stage &g : st) {
        A.t0 = g.t0; A.t1 = g.t1; A.qtiles = g.qtiles; A.splits = g.splits; A.capseg = g.capseg; A.dense = g.t0 == 0 ? 1 : 0;
        A.thr = thr;
        const int64_t jobs = (int64_t)g.splits * A.qtiles, per = (jobs + 7) / 8;
        hipLaunchKernelGGL(kern.of(g.wq), dim3((unsigned)(8 * per)), dim3(MNT), lds0 + lds_wq * g.wq, s, A);
        SA_HIP(hipGetLastError());
        SelArgs S = out;
        if (&g != &st.back()) S.ids = nullptr;
        S.buf = A.buf; S.cnt = A.cnt; S.splits = g.splits; S.capseg = g.capseg;
        S.dense_rows = A.dense ? (g.t1 - g.t0) * TROWS : 0;
        S.kt = kt; S.nq = A.nq; S.first = first ? 1 : 0;
        S.list = list; S.thr = thr; S.over = over;
        S.cap = sort_cap;
        if (g.lane_keys > 0)
            hipLaunchKernelGGL(pick_select(g.lane_keys), dim3((unsigned)((A.nq + 3) / 4)), dim3(256), 32 * (size_t)sort_cap,
                               s, S);
        else
            hipLaunchKernelGGL(knn_tile::knn_select_kernel, dim3((unsigned)A.nq), dim3(256), 0, s, S);
        SA_HIP(hipGetLastError());
        first = false;
    }
    return SA_OK;
}

// ---------------------------------------------------------------- float data

// column sums of the base in double (L2 centring): one workgroup per row chunk, float4
// columns, as many rows at a time as the threads allow (d <= 1024)
__global__ void __launch_bounds__(256) knn_colsum_kernel(const float *x, int64_t n, int d, int64_t ld, int64_t chunk,
                                                         double *sum)
{
    __shared__ double part[256][4];
    const int nc = d >> 2, groups = 256 / nc, g = threadIdx.x / nc, c = threadIdx.x % nc;
    const int64_t r0 = (int64_t)blockIdx.x * chunk, r1 = r0 + chunk < n ? r0 + chunk : n;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    if (g < groups)
        for (int64_t r = r0 + g; r < r1; r += groups) {
            const float4 v = *reinterpret_cast<const float4 *>(x + r * ld + 4 * c);
            s[0] += (double)v.x; s[1] += (double)v.y; s[2] += (double)v.z; s[3] += (double)v.w;
        }
#pragma unroll
    for (int i = 0; i < 4; ++i) part[threadIdx.x][i] = s[i];
    __syncthreads();
    for (int e = threadIdx.x; e < d; e += 256) {
        double t = 0.0;
        for (int h = 0; h < groups; ++h) t += part[h * nc + (e >> 2)][e & 3];
        atomicAdd(sum + e, t);
    }
}

__global__ void knn_mean_kernel(const double *sum, int d, double n, float *mean)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c < d) mean[c] = (float)(sum[c] / n);
}

// float -> bf16 bits, rounded to nearest even (finite inputs; an overflow rounds to inf)
__device__ __forceinline__ uint16_t bf16_rne_bits(float v)
{
    const uint32_t u = __float_as_uint(v);
    return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}

struct FPrepArgs {
    const float *x;
    int64_t n, ld, rows;
    int32_t d, ks;
    int64_t ntile, mul;    // as in PrepArgs
    const float *mean;     // L2: subtracted from every coordinate (null: none)
    int32_t zero_norm;     // write 0 for |x|^2 (base rows under the inner product)
    unsigned char *out;    // blocks in operand order, the high and the low parts
    float *norm;           // |x|^2 (rounded once from double); base: +inf for padding
    int32_t *tab;          // base: the permutation; null: queries
    unsigned *max_norm2;   // bits of the largest |x|^2 (null: not wanted; non-negative floats order as unsigned)
    int32_t *bad;          // any value the matrix-core path cannot take
};

// One wavefront per block of 16 rows.  (With one atomic per row on the largest norm and on
// the flag, 200,000 rows took 2.3 ms.)  Values the path cannot take are replaced by zero
// and flagged: the stages that are already enqueued run on valid rows either way.
__global__ void __launch_bounds__(256) knn_prep_float_kernel(FPrepArgs P)
{
    const int lane = __lane_id();
    const int64_t blk = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (blk * 16 >= P.rows) return;
    const int r = lane & 15, g = lane >> 4;
    int64_t row = blk * 16 + r;
    if (P.mul) {
        const int64_t t = blk >> 2, off = (t * P.mul) % P.ntile;
        if ((blk & 3) == 0 && lane == 0) P.tab[t] = (int32_t)off;
        row = ((blk & 3) * 16 + r) * P.ntile + off;
    }
    const float *src = P.x + row * P.ld;
    unsigned char *const out = P.out + blk * P.ks * 2048 + 16 * lane;
    double sum = 0.0;
    bool bad = false;
    for (int ks = 0; ks < P.ks; ++ks) {
        const int c = 32 * ks + 8 * g;
        float f[8];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const bool in = row < P.n && c + 4 * h < P.d;
            const float4 v = in ? *reinterpret_cast<const float4 *>(src + c + 4 * h) : make_float4(0.f, 0.f, 0.f, 0.f);
            const float4 m = in && P.mean ? *reinterpret_cast<const float4 *>(P.mean + c + 4 * h) : make_float4(0.f, 0.f, 0.f, 0.f);
            const float x4[4] = {v.x, v.y, v.z, v.w}, m4[4] = {m.x, m.y, m.z, m.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const bool fin = fabsf(x4[i]) <= 3.0e38f;
                bad |= !fin;
                f[4 * h + i] = fin ? x4[i] - m4[i] : 0.f;
            }
        }
        uint16_t hb[8], lb[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            // nonzero magnitudes below 2^-60 could give subnormal bf16 parts, which the matrix
            // cores may flush: such data goes to the scan
            bad |= f[i] != 0.f && fabsf(f[i]) < 0x1p-60f;
            hb[i] = bf16_rne_bits(f[i]);
            lb[i] = bf16_rne_bits(f[i] - __uint_as_float((uint32_t)hb[i] << 16));   // (the difference is exact)
            sum += (double)f[i] * (double)f[i];
        }
        *reinterpret_cast<uint4 *>(out + ks * 1024) =
            make_uint4(hb[0] | (uint32_t)hb[1] << 16, hb[2] | (uint32_t)hb[3] << 16, hb[4] | (uint32_t)hb[5] << 16,
                       hb[6] | (uint32_t)hb[7] << 16);
        *reinterpret_cast<uint4 *>(out + (P.ks + ks) * 1024) =
            make_uint4(lb[0] | (uint32_t)lb[1] << 16, lb[2] | (uint32_t)lb[3] << 16, lb[4] | (uint32_t)lb[5] << 16,
                       lb[6] | (uint32_t)lb[7] << 16);
    }
    sum += __shfl_xor(sum, 16, 64);
    sum += __shfl_xor(sum, 32, 64);
    const float nf = (float)sum;
    if (__ballot(bad) && lane == 0 && !__hip_atomic_load(P.bad, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicOr(P.bad, 1);
    if (P.max_norm2) {
        unsigned mx = row < P.n ? __float_as_uint(nf) : 0u;
        for (int o = 1; o < 16; o <<= 1) {
            const unsigned v = (unsigned)__shfl_xor((int)mx, o, 64);
            mx = v > mx ? v : mx;
        }
        if (lane == 0 && mx > __hip_atomic_load(P.max_norm2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            atomicMax(P.max_norm2, mx);
    }
    if (g == 0) P.norm[blk * 16 + r] = P.tab && row >= P.n ? __builtin_inff() : P.zero_norm ? 0.f : nf;
}

struct EArgs {
    const float *base;
    int64_t n, ld;
    const float *queries;
    int64_t q0, ldq;
    int32_t d, k, kt, metric, exclude_self;
    const uint64_t *list;       // [query][kt] best approximate keys (distance less |q|^2 for L2)
    const int32_t *over;
    const float *qn;            // |q|^2 per query (the candidate pass's)
    const unsigned *max_norm2;
    int32_t *ids;
    float *dists;
    int32_t *failed;            // count of queries whose list could not show the margin
    int32_t *failed_list;       // those queries, in any order
};

// One workgroup per query, one candidate per thread: the exact keys of the candidates with
// the scan's arithmetic (double, index order, separately rounded multiply and add, one
// rounding to float) and the k smallest, then the margin test.  A point outside the list
// has an approximate distance of at least the list's last one, so its exact distance is
// at least that less E_q; if that exceeds the k-th exact key by more than a few float
// units (the keys are roundings), no outside point can enter the k best.
__global__ void __launch_bounds__(320) knn_exact_kernel(EArgs E)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    int P = 64;
    while (P < E.kt) P <<= 1;
    uint64_t *const key = reinterpret_cast<uint64_t *>(smem);     // [P]
    float *const qs = reinterpret_cast<float *>(key + P);          // [d]
    const int tid = threadIdx.x;
    const int64_t q = blockIdx.x, qg = E.q0 + q;
    const int64_t points = E.n - (E.exclude_self ? 1 : 0);
    // (an overflowed buffer, or a list short of points that exist: products that were no numbers)
    if (E.over[q] || (points > 0 && E.list[q * E.kt + (points < E.kt ? points : E.kt) - 1] == KEY_EMPTY)) {
        if (tid == 0) E.failed_list[atomicAdd(E.failed, 1)] = (int32_t)qg;
        return;
    }
    for (int c = tid; c < E.d; c += blockDim.x) qs[c] = E.queries[qg * E.ldq + c];
    for (int i = E.kt + tid; i < P; i += blockDim.x) key[i] = KEY_EMPTY;
    __syncthreads();
    const uint64_t ak = E.list[q * E.kt + tid];
    uint64_t ek = KEY_EMPTY;
    if (ak != KEY_EMPTY) {
        const int32_t id = key_id(ak);
        const float4 *x = reinterpret_cast<const float4 *>(E.base + (int64_t)id * E.ld);
        double acc = 0.0;
        if (E.metric == SA_L2) {
#pragma unroll 4
            for (int c = 0; c < E.d / 4; ++c) {
                const float4 a = reinterpret_cast<const float4 *>(qs)[c], b = x[c];
                double t;
                t = (double)a.x - (double)b.x; acc += t * t;
                t = (double)a.y - (double)b.y; acc += t * t;
                t = (double)a.z - (double)b.z; acc += t * t;
                t = (double)a.w - (double)b.w; acc += t * t;
            }
        } else {
#pragma unroll 4
            for (int c = 0; c < E.d / 4; ++c) {
                const float4 a = reinterpret_cast<const float4 *>(qs)[c], b = x[c];
                acc += (double)a.x * (double)b.x;
                acc += (double)a.y * (double)b.y;
                acc += (double)a.z * (double)b.z;
                acc += (double)a.w * (double)b.w;
            }
        }
        ek = make_key(E.metric == SA_L2 ? (float)acc : (float)(-acc), id);
    }
    key[tid] = ek;
    knn_tile::sort_lds(key, P);
    if (points > E.kt) {
        // (for L2 the last term also covers the rounding of the centred coordinates)
        const double c = 3.1 / 65536.0 + (3.0 * E.d + 2.0) / 16777216.0;
        const double nq_ = sqrt((double)E.qn[q]), nm = sqrt((double)__uint_as_float(*E.max_norm2));
        // (the last term: fp32 products and partial sums below 2^-126 that may be flushed)
        const double tiny = (3.0 * E.d + 2.0) * 0x1p-126;
        const double err = E.metric == SA_L2 ? 2.0 * (2.0 * c * nq_ * nm + 8.0 / 16777216.0 * (nq_ + nm) * (nq_ + nm) + 2.0 * tiny)
                                             : 2.0 * (c * nq_ * nm + 2.0 / 16777216.0 * nq_ * nm + tiny);
        const double Kk = key_dist(key[E.k - 1]);
        const double last = (double)key_dist(E.list[q * E.kt + E.kt - 1]) + (E.metric == SA_L2 ? (double)E.qn[q] : 0.0);
        if (!(last - err > Kk + fabs(Kk) * (1.0 / 1048576.0))) {
            if (tid == 0) E.failed_list[atomicAdd(E.failed, 1)] = (int32_t)qg;
            return;
        }
    }
    for (int j = tid; j < E.k; j += blockDim.x) {
        const uint64_t kj = j < P ? key[j] : KEY_EMPTY;
        const bool ok = kj != KEY_EMPTY;
        E.ids[qg * E.k + j] = ok ? key_id(kj) : -1;
        E.dists[qg * E.k + j] = ok ? key_dist(kj) : __builtin_inff();
    }
}

// ---------------------------------------------------------------- one call (host)

// Sizes and device memory of one form for chunks of qc queries.
struct Plan {
    bool integer, wide;
    int ks, kt;
    int64_t ntile, qc, qpad;
    std::vector<Stage> st;
    size_t o_xn, o_tab, o_fail, o_buf, o_cnt, o_qt, o_qn, o_over, o_list, o_thr, o_sum, o_mean, o_flags, total;
};

Plan make_plan(bool integer, int64_t n, int32_t d, int64_t nq, int32_t k, int64_t qc)
{
    Plan P;
    P.integer = integer;
    P.ks = (d + 31) / 32;
    if (integer && P.ks == 5) P.ks = 6;
    if (integer && P.ks == 7) P.ks = 8;
    P.wide = !integer && P.ks > 4;
    // integer data: the k best (a threshold from fewer than 24 keys strays too far); float
    // data: candidates enough that the margin holds on ordinary data, one per thread of
    // the exact kernel
    P.kt = integer ? std::max(k, 24) : k <= 96 ? 128 : (k + 32 + 63) / 64 * 64;
    if (P.kt > 320) P.kt = 320;
    P.ntile = (n + 2 * TROWS - 1) / (2 * TROWS) * 2;
    P.qc = qc;
    P.qpad = (qc + 255) / 256 * 256;
    P.st = plan_stages((int)P.ntile, P.kt, qc, P.wide);
    size_t buf = 0, cnt = 0, o = 0;
    for (const Stage &g : P.st) {
        buf = std::max(buf, stage_bytes(g, qc));
        cnt = std::max(cnt, (size_t)qc * g.splits * 4);
    }
    const size_t row = (size_t)P.ks * (integer ? 64 : 128);   // bytes of a stored row
    auto take = [&](size_t bytes) {
        const size_t at = o;
        o += align256(bytes);
        return at;
    };
    take((size_t)P.ntile * TROWS * row);
    P.o_xn = take((size_t)P.ntile * TROWS * 4);
    P.o_tab = take((size_t)P.ntile * 4);
    P.o_fail = take((size_t)nq * 4);
    P.o_buf = take(buf);
    P.o_cnt = take(cnt);
    P.o_qt = take((size_t)P.qpad * row);
    P.o_qn = take((size_t)P.qpad * 4);
    P.o_over = take((size_t)qc * 4);
    P.o_list = take((size_t)qc * P.kt * 8);
    P.o_thr = take((size_t)qc * 8);
    P.o_sum = take(integer ? 0 : (size_t)d * 8);
    P.o_mean = take(integer ? 0 : (size_t)d * 4);
    P.o_flags = take(16);
    P.total = o;
    return P;
}

template <int KS, int NP, int FORM>
Kernels resident()
{
    return {{knn_tile::knn_tile_kernel<KS, NP, 1, FORM>, knn_tile::knn_tile_kernel<KS, NP, 2, FORM>,
             knn_tile::knn_tile_kernel<KS, NP, 4, FORM>}};
}

template <int FORM>
Kernels int_kernels(int ks)
{
    switch (ks) {
    case 1: return resident<1, 1, FORM>();
    case 2: return resident<2, 1, FORM>();
    case 3: return resident<3, 1, FORM>();
    case 4: return resident<4, 1, FORM>();
    case 6: return resident<6, 1, FORM>();
    default: return resident<8, 1, FORM>();
    }
}

Kernels float_kernels(int ks)
{
    switch (ks) {
    case 1: return resident<1, 2, knn_tile::FLOAT>();
    case 2: return resident<2, 2, knn_tile::FLOAT>();
    case 3: return resident<3, 2, knn_tile::FLOAT>();
    case 4: return resident<4, 2, knn_tile::FLOAT>();
    default: return {{knn_tile::knn_tile_wide_kernel, knn_tile::knn_tile_wide_kernel, knn_tile::knn_tile_wide_kernel}};
    }
}

// dynamic LDS of the product kernel: tile_lds + tile_lds_wq per 64 queries
size_t tile_lds(const Plan &P)
{
    return P.wide ? 2 * 32 * 1024 : 2 * ((size_t)4096 * P.ks * (P.integer ? 1 : 2) + 256);
}

size_t tile_lds_wq(const Plan &P) { return P.wide ? 64 * 12 : 64 * 16; }

hipError_t raise_lds(const Plan &P, const Kernels &kern)
{
    for (const Stage &g : P.st) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern.of(g.wq)),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize,
                                                 (int)(tile_lds(P) + tile_lds_wq(P) * g.wq));
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

struct Call {
    const float *base;
    int64_t n;
    int32_t d;
    int64_t ld;
    const float *queries;
    int64_t nq, ldq;
    int32_t k, metric, exclude_self;
    int32_t *ids;
    float *dists;
    hipStream_t s;
};

TileArgs tile_args(const Plan &P, const Call &c, unsigned char *m)
{
    TileArgs A;
    A.xt = m; A.xn = reinterpret_cast<float *>(m + P.o_xn); A.tab = reinterpret_cast<int32_t *>(m + P.o_tab);
    A.qt = m + P.o_qt; A.qn = m + P.o_qn;
    A.n = c.n; A.ntile = (int32_t)P.ntile; A.nks = P.ks;
    A.s = P.integer ? 1.f : c.metric == SA_L2 ? -2.f : -1.f;
    A.exclude_self = c.exclude_self;
    A.buf = reinterpret_cast<uint64_t *>(m + P.o_buf); A.cnt = reinterpret_cast<int32_t *>(m + P.o_cnt);
    return A;
}

// The listed queries' rows are written by the scan; every other row is final.
int rescan(const Call &c, int64_t count, const int32_t *failed_list)
{
    const int rc = launch_knn_scan(c.base, c.n, c.d, c.ld, c.queries, count, c.ldq, c.k, c.metric, c.exclude_self, c.ids,
                                   c.dists, c.s, failed_list);
    if (rc != SA_OK) return rc;
    SA_HIP(hipStreamSynchronize(c.s));
    return SA_OK;
}

// The integer form if every coordinate qualifies; *ran tells whether it did.  Synchronous.
int run_integer(const Plan &P, const Call &c, unsigned char *m, bool *ran)
{
    const hipStream_t s = c.s;
    // [0] not integer data, [1] overflowed queries, [2] largest |x|^2, [3] largest |q|^2
    int32_t *const flags = reinterpret_cast<int32_t *>(m + P.o_flags);
    int32_t *const failed_list = reinterpret_cast<int32_t *>(m + P.o_fail), *const qn = reinterpret_cast<int32_t *>(m + P.o_qn);
    unsigned char *const qt = m + P.o_qt;
    SA_HIP(hipMemsetAsync(flags, 0, 16, s));
    // (queries are stored times the factor of the distance: -2 q.x, or -q.x)
    auto prep = [&](const float *x, int64_t rows, int64_t stride, int64_t padded, int64_t mul, unsigned char *out,
                    int32_t *qnorm, int32_t *mx) {
        PrepArgs a{x, rows, stride, padded, c.d, P.ks, P.ntile, mul, c.metric, out, reinterpret_cast<float *>(m + P.o_xn),
                   qnorm, reinterpret_cast<int32_t *>(m + P.o_tab), flags, mx,
                   qnorm ? (c.metric == SA_L2 ? -2.f : -1.f) : 1.f};
        hipLaunchKernelGGL(knn_prep_kernel, dim3((unsigned)((padded / 16 + 3) / 4)), dim3(256), 0, s, a);
        return hipGetLastError();
    };
    const bool self = c.queries == c.base && c.ldq == c.ld && c.nq <= c.n;
    // the queries first: where they are not integers, the base's blocks see the flag and do
    // nothing (the whole check took 0.42 ms for 1M x 96 floats when it read every row)
    if (c.nq <= P.qc) SA_HIP(prep(c.queries, c.nq, c.ldq, P.qpad, 0, qt, qn, flags + 3));
    else if (!self) SA_HIP(prep(c.queries, c.nq, c.ldq, (c.nq + 15) / 16 * 16, 0, nullptr, nullptr, flags + 3));
    SA_HIP(prep(c.base, c.n, c.ld, P.ntile * TROWS, tile_mul(P.ntile), m, nullptr, flags + 2));
    int32_t hf[4] = {0, 0, 0, 0};
    SA_HIP(hipMemcpyAsync(hf, flags, 16, hipMemcpyDeviceToHost, s));
    SA_HIP(hipStreamSynchronize(s));
    if (hf[0]) return SA_OK;
    const double nx = hf[2], nq2 = self ? hf[2] : hf[3];
    const bool fold = nx + 2.0 * std::sqrt(nx * nq2) < 16777216.0;
    const Kernels kern = fold ? int_kernels<knn_tile::FOLDED>(P.ks) : int_kernels<knn_tile::INT>(P.ks);
    SA_HIP(raise_lds(P, kern));
    TileArgs A = tile_args(P, c, m);
    uint64_t *const list = reinterpret_cast<uint64_t *>(m + P.o_list), *const thr = reinterpret_cast<uint64_t *>(m + P.o_thr);
    int32_t *const over = reinterpret_cast<int32_t *>(m + P.o_over);
    for (int64_t q0 = 0; q0 < c.nq; q0 += P.qc) {
        const int64_t cn = std::min(P.qc, c.nq - q0);
        if (c.nq > P.qc) SA_HIP(prep(c.queries + q0 * c.ldq, cn, c.ldq, P.qpad, 0, qt, qn, nullptr));
        A.q0 = q0; A.nq = (int32_t)cn;
        SelArgs out{};
        out.ids = c.ids; out.dists = c.dists; out.q0 = q0; out.k = c.k; out.failed = flags + 1; out.failed_list = failed_list;
        const int rc = run_stages(A, P.st, kern, tile_lds(P), tile_lds_wq(P), P.kt, list, thr, over, out, s);
        if (rc != SA_OK) return rc;
    }
    // (one stage: every distance was kept, none can have overflowed)
    if (P.st.size() > 1) SA_HIP(hipMemcpyAsync(hf, flags, 16, hipMemcpyDeviceToHost, s));
    SA_HIP(hipStreamSynchronize(s));
    *ran = true;
    return hf[1] > 0 ? rescan(c, hf[1], failed_list) : SA_OK;
}

// The float form; *ran is false on non-finite data and on magnitudes it cannot take (the
// caller then runs the scan).  Queries that cannot show their margin are rescored by the
// scan here.  Synchronous.
int run_float(const Plan &P, const Call &c, unsigned char *m, bool *ran)
{
    const hipStream_t s = c.s;
    unsigned *const flags = reinterpret_cast<unsigned *>(m + P.o_flags);   // [0] max |x|^2, [1] bad, [2] failed
    int32_t *const bad = reinterpret_cast<int32_t *>(flags + 1), *const failed = reinterpret_cast<int32_t *>(flags + 2);
    int32_t *const failed_list = reinterpret_cast<int32_t *>(m + P.o_fail);
    SA_HIP(hipMemsetAsync(flags, 0, 16, s));
    const float *mean = nullptr;
    if (c.metric == SA_L2) {
        // distances do not change when every point moves by the base mean, and the bound,
        // which grows with the norms, shrinks
        double *const sum = reinterpret_cast<double *>(m + P.o_sum);
        SA_HIP(hipMemsetAsync(sum, 0, (size_t)c.d * 8, s));
        const int64_t chunk = std::max<int64_t>(16, (c.n + 2047) / 2048);
        hipLaunchKernelGGL(knn_colsum_kernel, dim3((unsigned)((c.n + chunk - 1) / chunk)), dim3(256), 0, s, c.base, c.n, c.d,
                           c.ld, chunk, sum);
        SA_HIP(hipGetLastError());
        hipLaunchKernelGGL(knn_mean_kernel, dim3((unsigned)((c.d + 255) / 256)), dim3(256), 0, s, sum, c.d, (double)c.n,
                           reinterpret_cast<float *>(m + P.o_mean));
        SA_HIP(hipGetLastError());
        mean = reinterpret_cast<float *>(m + P.o_mean);
    }
    auto prep = [&](const float *x, int64_t rows, int64_t stride, int64_t padded, bool is_base) {
        FPrepArgs a{x, rows, stride, padded, c.d, P.ks, P.ntile, is_base ? tile_mul(P.ntile) : 0, mean,
                    is_base && c.metric != SA_L2, is_base ? m : m + P.o_qt,
                    reinterpret_cast<float *>(m + (is_base ? P.o_xn : P.o_qn)),
                    is_base ? reinterpret_cast<int32_t *>(m + P.o_tab) : nullptr, is_base ? flags : nullptr, bad};
        hipLaunchKernelGGL(knn_prep_float_kernel, dim3((unsigned)((padded / 16 + 3) / 4)), dim3(256), 0, s, a);
        return hipGetLastError();
    };
    SA_HIP(prep(c.base, c.n, c.ld, P.ntile * TROWS, true));
    const Kernels kern = float_kernels(P.ks);
    SA_HIP(raise_lds(P, kern));
    TileArgs A = tile_args(P, c, m);
    uint64_t *const list = reinterpret_cast<uint64_t *>(m + P.o_list), *const thr = reinterpret_cast<uint64_t *>(m + P.o_thr);
    int32_t *const over = reinterpret_cast<int32_t *>(m + P.o_over);
    size_t sorted = 64;
    while (sorted < (size_t)P.kt) sorted *= 2;
    for (int64_t q0 = 0; q0 < c.nq; q0 += P.qc) {
        const int64_t cn = std::min(P.qc, c.nq - q0);
        SA_HIP(prep(c.queries + q0 * c.ldq, cn, c.ldq, P.qpad, false));
        A.q0 = q0; A.nq = (int32_t)cn;
        const int rc = run_stages(A, P.st, kern, tile_lds(P), tile_lds_wq(P), P.kt, list, thr, over, SelArgs{}, s);
        if (rc != SA_OK) return rc;
        EArgs E{c.base, c.n, c.ld, c.queries, q0, c.ldq, c.d, c.k, P.kt, c.metric, c.exclude_self, list, over,
                reinterpret_cast<float *>(m + P.o_qn), flags, c.ids, c.dists, failed, failed_list};
        hipLaunchKernelGGL(knn_exact_kernel, dim3((unsigned)cn), dim3(P.kt), 8 * sorted + 4 * (size_t)c.d, s, E);
        SA_HIP(hipGetLastError());
    }
    unsigned hf[4] = {0, 0, 0, 0};
    SA_HIP(hipMemcpyAsync(hf, flags, 16, hipMemcpyDeviceToHost, s));
    SA_HIP(hipStreamSynchronize(s));
    if (hf[1] != 0) return SA_OK;
    *ran = true;
    if (hf[2] == 0) return SA_OK;
    const int rc = rescan(c, hf[2], failed_list);
    if (rc == SA_OK) knn_rescanned = hf[2];
    return rc;
}

}  // namespace

thread_local int64_t knn_rescanned = 0;

namespace {

// Which forms a call may run.  What an explicit SA_KNN_MFMA takes: k <= 128 (integer data,
// d <= 256) and k <= 96 (float, d <= 1024); SA_KNN_AUTO also takes every larger k (up to
// 256) when the base has at least 2048 rows: below, the scan is done before the stages are.
struct Forms {
    bool integer, flt;
};

Forms knn_forms(int64_t n, int32_t d, int32_t k, int32_t path, bool any_k = true)
{
    const bool large_k = any_k && path == SA_KNN_AUTO && n >= 2048;
    Forms f;
    f.integer = path != SA_KNN_SCAN && n >= 1 && d <= 256 && (k <= 128 || large_k);
    f.flt = path != SA_KNN_SCAN && n >= 1 && d <= 1024 && (k <= 96 || large_k);
    return f;
}

// the plans of the forms f for chunks of qc queries (the integer form's first); returns
// the bytes of device memory that either needs
size_t knn_plans(const Forms &f, int64_t n, int32_t d, int64_t nq, int32_t k, int64_t qc, std::vector<Plan> &plan)
{
    plan.clear();
    if (f.integer) plan.push_back(make_plan(true, n, d, nq, k, qc));
    if (f.flt) plan.push_back(make_plan(false, n, d, nq, k, qc));
    return plan.empty() ? 0 : std::max(plan.front().total, plan.back().total);
}

}  // namespace

size_t knn_workspace_bytes(int64_t n, int32_t d, int64_t nq, int32_t k, int32_t path)
{
    const Forms f = knn_forms(n, d, k, path);
    std::vector<Plan> plan;
    return nq > 0 ? knn_plans(f, n, d, nq, k, std::min<int64_t>(nq, QCHUNK), plan) : 0;
}

int launch_knn(const float *base, int64_t n, int32_t d, int64_t ld, const float *queries, int64_t nq, int64_t ldq,
               int32_t k, int32_t metric, int32_t exclude_self, int32_t *ids, float *dists, int32_t path,
               int32_t *path_used, void *ws, size_t ws_bytes, hipStream_t stream)
{
    if (path_used) *path_used = SA_KNN_AUTO;
    knn_rescanned = 0;
    if (path != SA_KNN_AUTO && path != SA_KNN_SCAN && path != SA_KNN_MFMA)
        return set_error(SA_EINVAL, "unknown kNN path %d", path);
    if (nq == 0) return SA_OK;
    Forms f = knn_forms(n, d, k, path);
    if (path == SA_KNN_MFMA && !f.integer && !f.flt)
        return set_error(SA_EUNSUPPORTED, "the MFMA kNN path needs n >= 1 and d <= 256, k <= 128 (integer data) or "
                         "d <= 1024, k <= 96 (n=%lld, d=%d, k=%d)", (long long)n, d, k);
    DeviceBlock mem;
    std::vector<Plan> plan;
    for (int64_t qc = std::min<int64_t>(nq, QCHUNK); f.integer || f.flt;) {
        // one block for whichever form runs; smaller chunks of queries if it does not fit
        const size_t need = knn_plans(f, n, d, nq, k, qc, plan);
        if (ws ? need <= ws_bytes : hipMalloc(&mem.p, need) == hipSuccess) break;
        if (!ws) {
            (void)hipGetLastError();
            mem.p = nullptr;
        }
        const Forms least = knn_forms(n, d, k, path, false);
        if (qc > 1024) {
            qc = std::max<int64_t>(1024, qc / 2);
        } else if (!ws && (f.integer != least.integer || f.flt != least.flt)) {
            // forms that only SA_KNN_AUTO's larger k allows must not cost the call: the scan
            // needs no memory
            f = least;
            qc = std::min<int64_t>(nq, QCHUNK);
        } else {
            return ws ? set_error(SA_ECAPACITY, "workspace of %zu bytes is smaller than the %zu bytes needed", ws_bytes, need)
                      : set_error(SA_ENOMEM, "hipMalloc of the bf16 copies failed");
        }
    }
    if (f.integer || f.flt) {
        bool ran = false;
        unsigned char *const m = static_cast<unsigned char *>(ws ? ws : mem.p);
        const Call c{base, n, d, ld, queries, nq, ldq, k, metric, exclude_self, ids, dists, stream};
        int rc = SA_OK;
        if (f.integer) rc = run_integer(plan.front(), c, m, &ran);
        // not integer data (or too wide for it): the float form
        if (rc == SA_OK && !ran && f.flt) rc = run_float(plan.back(), c, m, &ran);
        if (rc != SA_OK) return rc;
        if (ran) {
            if (path_used) *path_used = SA_KNN_MFMA;
            return SA_OK;
        }
        if (path == SA_KNN_MFMA)
            return set_error(SA_EUNSUPPORTED, "the MFMA kNN path needs integer coordinates in [-255, 255] (d <= 256, "
                             "k <= 128) or finite floats with d <= 1024 and k <= 96");
    }
    const int rc = launch_knn_scan(base, n, d, ld, queries, nq, ldq, k, metric, exclude_self, ids, dists, stream);
    if (rc != SA_OK) return rc;
    SA_HIP(hipStreamSynchronize(stream));
    if (path_used) *path_used = SA_KNN_SCAN;
    return SA_OK;
}

}  // namespace sa
