// Graph construction for the search (the paper takes a prebuilt NSG graph, Sec. 2.2;
// this builds the fixed-width graph the kernels read): the medoid entry point, row
// pruning of exact candidate lists, and a connectivity repair.
//
// Every distance here is computed by one thread walking the dimensions in index order in
// double precision (separately rounded multiply and add) and rounded once to float, so
// each pruning and bridging decision is reproducible bit for bit.
#include "sa_internal.h"

#include <algorithm>
#include <cmath>
#include <vector>

namespace sa {
namespace {

__device__ float dist_seq(const float *a, const float *b, int d, int metric)
{
    double acc = 0.0;
    if (metric == SA_L2) {
        for (int i = 0; i < d; i += 4) {
            const float4 x = *reinterpret_cast<const float4 *>(a + i);
            const float4 y = *reinterpret_cast<const float4 *>(b + i);
            double t;
            t = (double)x.x - (double)y.x; acc += t * t;
            t = (double)x.y - (double)y.y; acc += t * t;
            t = (double)x.z - (double)y.z; acc += t * t;
            t = (double)x.w - (double)y.w; acc += t * t;
        }
        return (float)acc;
    }
    for (int i = 0; i < d; i += 4) {
        const float4 x = *reinterpret_cast<const float4 *>(a + i);
        const float4 y = *reinterpret_cast<const float4 *>(b + i);
        acc += (double)x.x * (double)y.x;
        acc += (double)x.y * (double)y.y;
        acc += (double)x.z * (double)y.z;
        acc += (double)x.w * (double)y.w;
    }
    return (float)(-acc);
}

// ---------------------------------------------------------------- medoid

constexpr int MED_CHUNK = 4096;

// Sum in double, one addend after the other, of x[rows[i] * ld] (rows null: row i) over i <
// cnt: two groups of 32 loads in turn, one in flight while the other is added.  The order of
// the additions is fixed, so the loads in flight are all that hides their latency (one load
// at a time: 1.02 ms for 4,096-row chunks of 150K x 128 floats, against 0.09 ms).
__device__ __forceinline__ double seq_sum(const float *x, int64_t ld, const int32_t *rows, int64_t cnt)
{
    constexpr int U = 32;
    float a[2][U];
    double s = 0.0;
    auto load = [&](float (&v)[U], int64_t i0) {
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const int64_t i = i0 + j < cnt ? i0 + j : cnt - 1;
            v[j] = x[(rows ? (int64_t)rows[i] : i) * ld];
        }
    };
    auto add = [&](const float (&v)[U], int64_t i0) {
#pragma unroll
        for (int j = 0; j < U; ++j)
            if (i0 + j < cnt) s += (double)v[j];
    };
    if (cnt <= 0) return s;
    load(a[0], 0);
    for (int64_t i = 0; i < cnt; i += 2 * U) {
        load(a[1], i + U < cnt ? i + U : cnt - 1);
        add(a[0], i);
        load(a[0], i + 2 * U < cnt ? i + 2 * U : cnt - 1);
        add(a[1], i + U);
    }
    return s;
}

// column sums of chunks of rows: one wavefront per 64 columns and chunk
__global__ void __launch_bounds__(64) colsum_partial(const float *base, int64_t n, int d, int64_t ld, int64_t chunk, double *part)
{
    const int64_t r0 = (int64_t)blockIdx.x * chunk;
    const int c = blockIdx.y * 64 + threadIdx.x;
    if (c >= d) return;
    part[(int64_t)blockIdx.x * d + c] = seq_sum(base + r0 * ld + c, ld, nullptr, min(chunk, n - r0));
}

__global__ void colsum_final(const double *part, int64_t nchunks, int d, int64_t n, double *mean)
{
    for (int c = blockIdx.x * blockDim.x + threadIdx.x; c < d; c += gridDim.x * blockDim.x) {
        double s = 0.0;
        for (int64_t b = 0; b < nchunks; ++b) s += part[b * d + c];
        mean[c] = s / (double)n;
    }
}

__global__ void dist_to_mean(const float *base, int64_t n, int d, int64_t ld, const double *mean, double *bestd,
                             int64_t *besti)
{
    __shared__ double sd[256];
    __shared__ int64_t si[256];
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    double acc = INFINITY;
    int64_t id = INT64_MAX;
    if (r < n) {
        acc = 0.0;
        for (int c = 0; c < d; ++c) {
            double t = (double)base[r * ld + c] - mean[c];
            acc += t * t;
        }
        id = r;
    }
    sd[threadIdx.x] = acc;
    si[threadIdx.x] = id;
    __syncthreads();
    for (int s = blockDim.x / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            double od = sd[threadIdx.x + s];
            int64_t oi = si[threadIdx.x + s];
            if (od < sd[threadIdx.x] || (od == sd[threadIdx.x] && oi < si[threadIdx.x])) {
                sd[threadIdx.x] = od;
                si[threadIdx.x] = oi;
            }
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        bestd[blockIdx.x] = sd[0];
        besti[blockIdx.x] = si[0];
    }
}

// ---------------------------------------------------------------- pruning

__global__ void prune_kernel(const float *base, int64_t n, int d, int64_t ld, int metric, const int32_t *cand,
                             int kc, int R, int mode, int32_t *adj)
{
    __shared__ int32_t kept_all[4][64];
    const int wv = threadIdx.x >> 6, lane = __lane_id();
    const int64_t p = (int64_t)blockIdx.x * 4 + wv;
    if (p >= n) return;
    int32_t *kept = kept_all[wv];
    int32_t c_mine = lane < kc ? cand[p * kc + lane] : -1;
    if (c_mine >= n) c_mine = -1;   // malformed candidates are ignored like padding
    int nk = 0;
    if (mode == 0) {
        const uint64_t m = __ballot(c_mine >= 0);
        const int pos = __popcll(m & ((1ull << lane) - 1ull));
        if (c_mine >= 0 && pos < R) kept[pos] = c_mine;
        nk = min(R, __popcll(m));
    } else {
        const float dpc_mine = c_mine >= 0 ? dist_seq(base + p * ld, base + (int64_t)c_mine * ld, d, metric) : 0.f;
        for (int j = 0; j < kc && nk < R; ++j) {
            const int32_t c = __shfl(c_mine, j, 64);
            if (c < 0) continue;
            const float dpc = __shfl(dpc_mine, j, 64);
            bool occl = false;
            if (lane < nk) {
                const int32_t s = kept[lane];
                occl = dist_seq(base + (int64_t)s * ld, base + (int64_t)c * ld, d, metric) < dpc;
            }
            if (__ballot(occl) == 0) {
                __builtin_amdgcn_wave_barrier();
                if (lane == 0) kept[nk] = c;
                __builtin_amdgcn_wave_barrier();
                ++nk;
            }
        }
    }
    __builtin_amdgcn_wave_barrier();
    for (int j = lane; j < R; j += 64) adj[p * R + j] = j < nk ? kept[j] : -1;
}

// ---------------------------------------------------------------- repair helpers

// For several vertices at once: results[j] = the smallest key (distance to us[j], id)
// over the marked vertices with a free slot (grid.y: groups of NM_Q of them); results start
// as KEY_EMPTY.  A thread takes one vertex against NM_Q queries, whose chunks of 32
// dimensions sit in LDS, so its row is read once for all (each query by itself: 9.4 ms for
// 256 against 150K x 128, eight at a time 1.6).
constexpr int NM_Q = 8;

__global__ void __launch_bounds__(256) nearest_marked_batch(const float *base, int64_t n, int d, int64_t ld, int metric,
                                                            const uint8_t *mask, const int32_t *deg, int R,
                                                            const int32_t *us, int nus, unsigned long long *results)
{
    __shared__ float qs[NM_Q][32];
    const int64_t w = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int j0 = blockIdx.y * NM_Q;
    const bool in = w < n && mask[w] && deg[w] < R;
    const float *x = base + (in ? w : 0) * ld;
    double acc[NM_Q];
#pragma unroll
    for (int j = 0; j < NM_Q; ++j) acc[j] = 0.0;
    for (int c0 = 0; c0 < d; c0 += 32) {
        __syncthreads();
        for (int i = threadIdx.x; i < NM_Q * 32; i += 256) {
            const int j = i >> 5, c = c0 + (i & 31);
            qs[j][i & 31] = j0 + j < nus && c < d ? base[(int64_t)us[j0 + j] * ld + c] : 0.f;
        }
        __syncthreads();
        if (!in) continue;
        const int cn = min(32, d - c0);
        for (int c = 0; c < cn; c += 4) {
            const float4 v = *reinterpret_cast<const float4 *>(x + c0 + c);
            const float xv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < NM_Q; ++j) {
                    const float q = qs[j][c + i];
                    if (metric == SA_L2) {
                        const double t = (double)xv[i] - (double)q;
                        acc[j] += t * t;
                    } else {
                        acc[j] += (double)xv[i] * (double)q;
                    }
                }
        }
    }
#pragma unroll
    for (int j = 0; j < NM_Q; ++j) {
        unsigned long long key = in ? make_key(metric == SA_L2 ? (float)acc[j] : (float)(-acc[j]), (int32_t)w) : KEY_EMPTY;
        for (int o = 32; o > 0; o >>= 1) {
            const unsigned long long k = __shfl_xor(key, o, 64);
            key = k < key ? k : key;
        }
        if (__lane_id() == 0 && j0 + j < nus && key < __hip_atomic_load(results + j0 + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            atomicMin(results + j0 + j, key);
    }
}

__global__ void fill_u64_n(unsigned long long *p, int64_t cnt, unsigned long long v)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < cnt) p[i] = v;
}

// ---------------------------------------------------------------- rows and scans

// deg[v]: entries of row v before the first negative one (prefix), or not negative (all)
__global__ void __launch_bounds__(256) row_degrees(const int32_t *adj, int64_t n, int R, int prefix, int32_t *deg)
{
    const int lane = __lane_id();
    for (int64_t v = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); v < n; v += (int64_t)gridDim.x * 4) {
        const uint64_t neg = __ballot(lane >= R || adj[v * R + (lane < R ? lane : 0)] < 0);
        if (lane == 0) deg[v] = prefix ? (neg ? __builtin_ctzll(neg) : 64) : 64 - __popcll(neg);
    }
}

constexpr int SCAN_CHUNK = 2048;   // elements per workgroup of the prefix sum

// exclusive prefix sums of cnt[0 .. n) into out[0 .. n] (out[n]: the total), in three
// launches: sums of chunks, their prefix, the elements
__global__ void __launch_bounds__(256) scan_sums(const int32_t *cnt, int64_t n, int64_t *sums)
{
    __shared__ int64_t part[4];
    const int64_t i0 = (int64_t)blockIdx.x * SCAN_CHUNK;
    int64_t t = 0;
    for (int j = threadIdx.x; j < SCAN_CHUNK; j += 256)
        if (i0 + j < n) t += cnt[i0 + j];
    for (int o = 32; o > 0; o >>= 1) t += __shfl_xor((long long)t, o, 64);
    if (__lane_id() == 0) part[threadIdx.x >> 6] = t;
    __syncthreads();
    if (threadIdx.x == 0) sums[blockIdx.x] = part[0] + part[1] + part[2] + part[3];
}

__global__ void __launch_bounds__(64) scan_chunks(int64_t *sums, int64_t nchunk, int64_t *total)
{
    const int lane = __lane_id();
    int64_t run = 0;
    for (int64_t i0 = 0; i0 < nchunk; i0 += 64) {
        const int64_t v = i0 + lane < nchunk ? sums[i0 + lane] : 0;
        int64_t inc = v;
        for (int o = 1; o < 64; o <<= 1) {
            const int64_t u = __shfl_up((long long)inc, o, 64);
            if (lane >= o) inc += u;
        }
        if (i0 + lane < nchunk) sums[i0 + lane] = run + inc - v;
        run += __shfl((long long)inc, 63, 64);
    }
    if (lane == 0) *total = run;
}

__global__ void __launch_bounds__(256) scan_write(const int32_t *cnt, int64_t n, const int64_t *sums, int64_t *out)
{
    __shared__ int64_t part[4];
    const int lane = __lane_id(), w = threadIdx.x >> 6;
    int64_t run = sums ? sums[blockIdx.x] : 0;
    for (int j0 = 0; j0 < SCAN_CHUNK; j0 += 256) {
        const int64_t i = (int64_t)blockIdx.x * SCAN_CHUNK + j0 + threadIdx.x;
        const int64_t v = i < n ? cnt[i] : 0;
        int64_t inc = v;
        for (int o = 1; o < 64; o <<= 1) {
            const int64_t u = __shfl_up((long long)inc, o, 64);
            if (lane >= o) inc += u;
        }
        if (lane == 63) part[w] = inc;
        __syncthreads();
        int64_t base = run;
        for (int k = 0; k < w; ++k) base += part[k];
        if (i < n) out[i] = base + inc - v;
        run += part[0] + part[1] + part[2] + part[3];
        __syncthreads();
    }
    if (!sums && threadIdx.x == 0) out[n] = run;
}

// sums: room for (n + SCAN_CHUNK - 1) / SCAN_CHUNK entries
hipError_t prefix_sums(const int32_t *cnt, int64_t n, int64_t *sums, int64_t *out, hipStream_t s)
{
    const int64_t nchunk = (n + SCAN_CHUNK - 1) / SCAN_CHUNK;
    if (nchunk == 1) {
        hipLaunchKernelGGL(scan_write, dim3(1), dim3(256), 0, s, cnt, n, (const int64_t *)nullptr, out);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(scan_sums, dim3((unsigned)nchunk), dim3(256), 0, s, cnt, n, sums);
    hipLaunchKernelGGL(scan_chunks, dim3(1), dim3(64), 0, s, sums, nchunk, out + n);
    hipLaunchKernelGGL(scan_write, dim3((unsigned)nchunk), dim3(256), 0, s, cnt, n, sums, out);
    return hipGetLastError();
}

__global__ void fill_i32(int32_t *p, int64_t cnt, int32_t v)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < cnt) p[i] = v;
}

// A launch takes fewer than 2^32 work items along x, which a wavefront a row reaches at 2^26
// rows and a thread an edge at 2^32 edges: such kernels walk their work in strides of the grid.
unsigned blocks_for(int64_t cnt, int per) { return (unsigned)std::min<int64_t>((cnt + per - 1) / per, 1 << 23); }

// ---------------------------------------------------------------- reverse edges

// In-edges of the vertices that have room, counted (in null) or, counting back down, written
// as keys (d(c, p), p) in any order behind start[c]
__global__ void in_edges(const float *base, int64_t n, int d, int64_t ld, int metric, const int32_t *adj, int R,
                         const int32_t *deg, int32_t *cnt, const int64_t *start, uint64_t *in)
{
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n * R; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t p = e / R;
        const int32_t c = adj[e];
        if (c < 0 || c >= n || deg[c] >= R) continue;
        const int pos = in ? atomicSub(cnt + c, 1) - 1 : atomicAdd(cnt + c, 1);
        if (in) in[start[c] + pos] = make_key(dist_seq(base + (int64_t)c * ld, base + p * ld, d, metric), (int32_t)p);
    }
}

// sorts one key per lane, ascending
__device__ __forceinline__ uint64_t sort64(uint64_t v)
{
    const int lane = __lane_id();
    for (int k = 2; k <= 64; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            const uint64_t o = (uint64_t)__shfl_xor((unsigned long long)v, j, 64);
            const bool low = (lane & j) == 0, up = (lane & k) == 0;
            v = (low == up) == (o < v) ? o : v;
        }
    return v;
}

// One wavefront per vertex with room: the 64 smallest in-edge keys above the last ones
// taken, by merging sorted chunks of 64 into a sorted list held one key per lane; each is
// appended unless the row holds its vertex, and the list is read again if 64 were not
// enough (at most R of them can be known already).  On the host this was the longest part
// of a graph build (60 ms of 197 at 150K x 128).
__global__ void __launch_bounds__(256) append_in_edges(int64_t n, int R, const int32_t *deg, const int64_t *start,
                                                       const uint64_t *in, int32_t *adj, unsigned long long *added)
{
    const int lane = __lane_id();
    for (int64_t c = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); c < n; c += (int64_t)gridDim.x * 4) {
        int len = deg[c];
        const int64_t b = start[c], e = start[c + 1];
        if (len >= R || b == e) continue;
        const int before = len;
        int32_t row = lane < len ? adj[c * R + lane] : -1;
        uint64_t last = 0;
        bool some = false, more = true;
        while (more && len < R) {
            uint64_t best = KEY_EMPTY;
            for (int64_t i0 = b; i0 < e; i0 += 64) {
                uint64_t v = i0 + lane < e ? in[i0 + lane] : KEY_EMPTY;
                if (some && v <= last) v = KEY_EMPTY;
                const uint64_t worst = (uint64_t)__shfl((unsigned long long)best, 63, 64);
                if (__ballot(v < worst) == 0) continue;
                v = sort64(v);
                // the smaller of best[l] and v[63 - l] are the 64 smallest, bitonic in l
                const uint64_t r = (uint64_t)__shfl((unsigned long long)v, 63 - lane, 64);
                best = r < best ? r : best;
                for (int j = 32; j > 0; j >>= 1) {
                    const uint64_t o = (uint64_t)__shfl_xor((unsigned long long)best, j, 64);
                    best = ((lane & j) == 0) == (o < best) ? o : best;
                }
            }
            const int got = __popcll(__ballot(best != KEY_EMPTY));
            for (int i = 0; i < got && len < R; ++i) {
                const int32_t p = key_id((uint64_t)__shfl((unsigned long long)best, i, 64));
                if (__ballot(row == p)) continue;
                if (lane == len) row = p;
                ++len;
            }
            more = got == 64;
            some = true;
            last = (uint64_t)__shfl((unsigned long long)best, 63, 64);
        }
        if (lane >= before && lane < len) adj[c * R + lane] = row;
        if (lane == 0 && len > before) atomicAdd(added, (unsigned long long)(len - before));
    }
}

// ---------------------------------------------------------------- repair

// Union-find over the edges: a root only ever gets a smaller root as its parent, so every
// component ends with its smallest vertex as root.
__device__ __forceinline__ int32_t uf_load(int32_t *par, int32_t v)
{
    return __hip_atomic_load(par + v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ int32_t uf_root(int32_t *par, int32_t v)
{
    int32_t p = uf_load(par, v);
    while (p != v) {
        const int32_t g = uf_load(par, p);
        if (g != p) __hip_atomic_store(par + v, g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        v = p;
        p = g;
    }
    return v;
}

__global__ void uf_init(int32_t *par, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) par[i] = (int32_t)i;
}

__global__ void uf_hook(const int32_t *adj, int64_t n, int R, int32_t *par)
{
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n * R; e += (int64_t)gridDim.x * blockDim.x) {
        const int32_t u = adj[e];
        if (u < 0 || u >= n) continue;
        int32_t a = uf_root(par, (int32_t)(e / R)), b = uf_root(par, u);
        while (a != b) {
            const int32_t hi = a > b ? a : b, lo = a > b ? b : a;
            const int32_t old = atomicCAS(par + hi, hi, lo);
            if (old == hi) break;   // hi was still a root
            a = uf_root(par, old);
            b = uf_root(par, lo);
        }
    }
}

__global__ void uf_flatten(int32_t *par, int64_t n, int32_t *root, int32_t *is_root)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int32_t r = uf_root(par, (int32_t)i);
    root[i] = r;
    is_root[i] = r == i;
}

// comp[v] = number of v's component (in the order of their smallest vertices)
__global__ void comp_of(const int32_t *root, const int64_t *number, int64_t n, int32_t *comp)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) comp[i] = (int32_t)number[root[i]];
}

// mean of each group g < nc of rows: members[start[g] .. start[g + 1]), summed in that order, and
// of the n rows themselves (g = nc); one wavefront per 64 columns and group, all at once: a
// large group's sum takes some 50 ns a row (1M rows: 52 ms), one addition after the other
__global__ void __launch_bounds__(64) group_means(const float *base, int64_t n, int d, int64_t ld, const int32_t *members,
                                                  const int64_t *start, int64_t nc, double *mean)
{
    const int64_t g = blockIdx.x;
    const int c = blockIdx.y * 64 + threadIdx.x;
    if (c >= d) return;
    const int64_t b = g < nc ? start[g] : 0, cnt = g < nc ? start[g + 1] - b : n;
    const double s = g < nc ? seq_sum(base + c, ld, members + b, cnt) : seq_sum(base + c, ld, nullptr, n);
    mean[g * d + c] = s / (double)cnt;
}

// squared distance of every row to its group's mean (comp null: group 0), in double
__global__ void mean_dists(const float *base, int64_t n, int d, int64_t ld, const double *mean, const int32_t *comp,
                           double *out)
{
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    const double *m = mean + (comp ? (int64_t)comp[v] * d : 0);
    double acc = 0.0;
    for (int i = 0; i < d; i += 4) {
        const float4 x = *reinterpret_cast<const float4 *>(base + v * ld + i);
        double t;
        t = (double)x.x - m[i]; acc += t * t;
        t = (double)x.y - m[i + 1]; acc += t * t;
        t = (double)x.z - m[i + 2]; acc += t * t;
        t = (double)x.w - m[i + 3]; acc += t * t;
    }
    out[v] = acc;
}

// the nearest member of each group, ties to the smaller id: first the distance (bits of a
// non-negative double order as integers), then the id
__global__ void nearest_member(const double *dist, const int32_t *comp, int64_t n, int pass, unsigned long long *bestd,
                               int32_t *best)
{
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    const unsigned long long b = (unsigned long long)__double_as_longlong(dist[v]);
    if (pass == 0) {
        if (b < __hip_atomic_load(bestd + comp[v], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMin(bestd + comp[v], b);
    } else if (b == bestd[comp[v]]) {
        atomicMin(best + comp[v], (int32_t)v);
    }
}

// out[i][j] = distance of rows us[i] and ws[j]
__global__ void pair_dists(const float *base, int d, int64_t ld, int metric, const int32_t *us, int64_t nu,
                           const int32_t *ws, int64_t nw, float *out)
{
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < nu * nw; e += (int64_t)gridDim.x * blockDim.x)
        out[e] = dist_seq(base + (int64_t)us[e / nw] * ld, base + (int64_t)ws[e % nw] * ld, d, metric);
}

constexpr int LINK_REPS = 4096;   // representatives the link kernel can sort in LDS

// One workgroup per gateway vertex v = src[a]: links to representatives, in key order,
// kept unless a kept one is nearer to the candidate than v is (rd: distances between
// representatives, dv: from the sources), then the nearest of the others, up to R less
// the local edges kept.
__global__ void __launch_bounds__(256) link_kernel(const int32_t *src, int64_t nc, const int32_t *rep, const int32_t *comp,
                                                   const float *rd, const float *dv, int R, int keep_rep, int keep_hub,
                                                   int P, int32_t *links)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    uint64_t *const key = reinterpret_cast<uint64_t *>(smem);             // [P]
    uint8_t *const used = reinterpret_cast<uint8_t *>(key + P);            // [P]
    const int64_t a = blockIdx.x;
    const int32_t v = src[a];
    const int cap = R - (a < nc ? keep_rep : keep_hub);
    for (int i = threadIdx.x; i < P; i += 256) {
        key[i] = i < nc && rep[i] != v ? make_key(dv[a * nc + i], rep[i]) : KEY_EMPTY;
        used[i] = 0;
    }
    for (int k = 2; k <= P; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            __syncthreads();
            for (int i = threadIdx.x; i < P / 2; i += 256) {
                const int lo = ((i & ~(j - 1)) << 1) | (i & (j - 1)), hi = lo | j;
                const uint64_t x = key[lo], y = key[hi];
                if ((x > y) == ((lo & k) == 0)) {
                    key[lo] = y;
                    key[hi] = x;
                }
            }
        }
    __syncthreads();
    if (threadIdx.x >= 64) return;
    const int lane = __lane_id();
    int nk = 0;
    int32_t mine = -1, mine_comp = 0;   // lane l: the l-th link and its component
    for (int i = 0; i < P && nk < cap; ++i) {
        const uint64_t k = key[i];
        if (k == KEY_EMPTY) break;
        const int32_t id = key_id(k), c = comp[id];
        const bool occl = lane < nk && rd[(int64_t)mine_comp * nc + c] < key_dist(k);
        if (__ballot(occl)) continue;
        if (lane == nk) {
            mine = id;
            mine_comp = c;
        }
        if (lane == 0) used[i] = 1;
        ++nk;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    for (int i = 0; i < P && nk < cap; ++i) {
        if (key[i] == KEY_EMPTY) break;
        if (used[i]) continue;
        if (lane == nk) mine = key_id(key[i]);
        ++nk;
    }
    if (lane < R) links[a * R + lane] = lane < nk ? mine : -1;
}

// the new rows of the gateway vertices: the first local edges that are no links, then the links
__global__ void __launch_bounds__(64) gateway_rows(const int32_t *src, int64_t nc, const int32_t *links, int R, int keep_rep,
                                                   int keep_hub, int32_t *adj)
{
    const int lane = __lane_id();
    const int64_t a = blockIdx.x;
    int32_t *const row = adj + (int64_t)src[a] * R;
    const int kl = a < nc ? keep_rep : keep_hub;
    const int32_t old = lane < R ? row[lane] : -1, lk = lane < R ? links[a * R + lane] : -1;
    int len = 0;
    int32_t out = -1;
    for (int r = 0; r < R && len < kl; ++r) {
        const int32_t u = __shfl(old, r, 64);
        if (u < 0 || __ballot(lk == u)) continue;
        if (lane == len) out = u;
        ++len;
    }
    for (int r = 0; r < R; ++r) {
        const int32_t u = __shfl(lk, r, 64);
        if (u < 0) continue;
        if (lane == len) out = u;
        ++len;
    }
    if (lane < R) row[lane] = out;
}

__global__ void put_rows(const int32_t *src, int64_t cnt, const int32_t *rows, int R, int32_t *adj)
{
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < cnt * R; e += (int64_t)gridDim.x * blockDim.x)
        adj[(int64_t)src[e / R] * R + e % R] = rows[e];
}

// One level of a breadth-first walk: the out-neighbours of the vertices at level cur get
// cur + 1; *changed is set if there was one.
__global__ void __launch_bounds__(256) bfs_level(const int32_t *adj, int64_t n, int R, int32_t *level, int32_t cur, int32_t *changed)
{
    const int lane = __lane_id();
    const int64_t v0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 64;
    const int64_t v = v0 + lane;
    uint64_t front = __ballot(v < n && level[v < n ? v : 0] == cur);
    bool any = false;
    for (; front; front &= front - 1) {
        const int64_t f = v0 + __builtin_ctzll(front);
        const int32_t u = lane < R ? adj[f * R + lane] : -1;
        if (u >= 0 && u < n && level[u] < 0) {
            level[u] = cur + 1;   // (every writer of this launch writes the same)
            any = true;
        }
    }
    if (__ballot(any) && lane == 0) *changed = 1;
}

__global__ void level_marks(const int32_t *level, int64_t n, uint8_t *mark)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) mark[i] = level[i] >= 0;
}

// rows ids[i] of src (row_words 32-bit words, stride words apart) to dst row i
__global__ void gather_rows(const int32_t *src, int64_t stride, int row_words, const int32_t *ids, int64_t cnt, int32_t *dst)
{
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < cnt * row_words; e += (int64_t)gridDim.x * blockDim.x)
        dst[e] = src[(int64_t)ids[e / row_words] * stride + e % row_words];
}

__global__ void apply_edits(const int64_t *pos, const int32_t *val, int64_t cnt, int32_t *adj)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < cnt) adj[pos[i]] = val[i];
}

// host-side distance with the same arithmetic as dist_seq
float host_dist(const float *a, const float *b, int d, int metric)
{
    double acc = 0.0;
    if (metric == SA_L2) {
        for (int i = 0; i < d; ++i) {
            double t = (double)a[i] - (double)b[i];
            acc += t * t;
        }
        return (float)acc;
    }
    for (int i = 0; i < d; ++i) acc += (double)a[i] * (double)b[i];
    return (float)(-acc);
}

bool key_less_host(float da, int32_t ia, float db, int32_t ib) { return da < db || (da == db && ia < ib); }

// device buffer that frees itself
template <typename T>
struct DevBuf {
    T *p = nullptr;
    hipError_t alloc(size_t count) { return hipMalloc(reinterpret_cast<void **>(&p), sizeof(T) * (count ? count : 1)); }
    ~DevBuf()
    {
        if (p) (void)hipFree(p);
    }
};

}  // namespace

int medoid_device(const float *base, int64_t n, int d, int64_t ld, int32_t *out, hipStream_t s)
{
    const int64_t nchunks = (n + MED_CHUNK - 1) / MED_CHUNK;
    const int64_t nblk = (n + 255) / 256;
    DevBuf<double> part, mean, bestd;
    DevBuf<int64_t> besti;
    if (part.alloc(nchunks * d) != hipSuccess || mean.alloc(d) != hipSuccess || bestd.alloc(nblk) != hipSuccess ||
        besti.alloc(nblk) != hipSuccess)
        return set_error(SA_ENOMEM, "medoid: device allocation failed");
    hipLaunchKernelGGL(colsum_partial, dim3((unsigned)nchunks, (unsigned)((d + 63) / 64)), dim3(64), 0, s, base, n, d, ld,
                       (int64_t)MED_CHUNK, part.p);
    hipLaunchKernelGGL(colsum_final, dim3((d + 127) / 128), dim3(128), 0, s, part.p, nchunks, d, n, mean.p);
    hipLaunchKernelGGL(dist_to_mean, dim3((unsigned)nblk), dim3(256), 0, s, base, n, d, ld, mean.p, bestd.p, besti.p);
    SA_HIP(hipGetLastError());
    std::vector<double> hd(nblk);
    std::vector<int64_t> hi(nblk);
    SA_HIP(hipMemcpyAsync(hd.data(), bestd.p, sizeof(double) * nblk, hipMemcpyDeviceToHost, s));
    SA_HIP(hipMemcpyAsync(hi.data(), besti.p, sizeof(int64_t) * nblk, hipMemcpyDeviceToHost, s));
    SA_HIP(hipStreamSynchronize(s));
    double bd = INFINITY;
    int64_t bi = -1;
    for (int64_t b = 0; b < nblk; ++b)
        if (hd[b] < bd || (hd[b] == bd && hi[b] < bi)) {
            bd = hd[b];
            bi = hi[b];
        }
    *out = (int32_t)bi;
    return SA_OK;
}

int prune_device(const float *base, int64_t n, int d, int64_t ld, int metric, const int32_t *cand, int kc, int R,
                 int mode, int32_t *adj, hipStream_t s)
{
    if (n == 0) return SA_OK;
    hipLaunchKernelGGL(prune_kernel, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, s, base, n, d, ld, metric, cand, kc,
                       R, mode, adj);
    SA_HIP(hipGetLastError());
    return SA_OK;
}

namespace {

// one device allocation cut into parts
struct Arena {
    unsigned char *p = nullptr;
    size_t at = 0;
    template <typename T>
    size_t want(int64_t count)
    {
        const size_t o = at;
        at += (sizeof(T) * (size_t)(count > 0 ? count : 1) + 255) / 256 * 256;
        return o;
    }
    hipError_t alloc() { return hipMalloc(reinterpret_cast<void **>(&p), at); }
    template <typename T>
    T *get(size_t o) const { return reinterpret_cast<T *>(p + o); }
    ~Arena()
    {
        if (p) (void)hipFree(p);
    }
};

}  // namespace

int reverse_edges_device(const float *base, int64_t n, int d, int64_t ld, int metric, int32_t *adj_dev, int R,
                         int64_t *added_out, hipStream_t s)
{
    if (added_out) *added_out = 0;
    if (n < 1) return SA_OK;
    const int64_t ne = n * R, nchunk = (n + SCAN_CHUNK - 1) / SCAN_CHUNK;
    Arena A;
    const size_t o_deg = A.want<int32_t>(n), o_start = A.want<int64_t>(n + 1), o_sums = A.want<int64_t>(nchunk);
    const size_t o_cnt = A.want<int32_t>(n), o_added = A.want<unsigned long long>(1);   // (zeroed together)
    if (A.alloc() != hipSuccess) return set_error(SA_ENOMEM, "reverse edges: device allocation failed");
    int32_t *const deg = A.get<int32_t>(o_deg), *const cnt = A.get<int32_t>(o_cnt);
    int64_t *const start = A.get<int64_t>(o_start);
    unsigned long long *const added = A.get<unsigned long long>(o_added);
    hipLaunchKernelGGL(row_degrees, dim3(blocks_for(n, 4)), dim3(256), 0, s, adj_dev, n, R, 1, deg);
    const int64_t zeroed = (int64_t)(o_added + 8 - o_cnt) / 4;
    hipLaunchKernelGGL(fill_i32, dim3(blocks_for(zeroed, 256)), dim3(256), 0, s, cnt, zeroed, 0);
    hipLaunchKernelGGL(in_edges, dim3(blocks_for(ne, 256)), dim3(256), 0, s, base, n, d, ld, metric, adj_dev, R, deg, cnt,
                       (const int64_t *)nullptr, (uint64_t *)nullptr);
    SA_HIP(hipGetLastError());
    SA_HIP(prefix_sums(cnt, n, A.get<int64_t>(o_sums), start, s));
    int64_t total = 0;
    SA_HIP(hipMemcpyAsync(&total, start + n, 8, hipMemcpyDeviceToHost, s));
    SA_HIP(hipStreamSynchronize(s));
    Arena K;
    const size_t o_in = K.want<uint64_t>(total);
    if (K.alloc() != hipSuccess) return set_error(SA_ENOMEM, "reverse edges: device allocation failed");
    uint64_t *const in = K.get<uint64_t>(o_in);
    hipLaunchKernelGGL(in_edges, dim3(blocks_for(ne, 256)), dim3(256), 0, s, base, n, d, ld, metric, adj_dev, R, deg, cnt,
                       (const int64_t *)start, in);
    hipLaunchKernelGGL(append_in_edges, dim3(blocks_for(n, 4)), dim3(256), 0, s, n, R, deg, start, in, adj_dev, added);
    SA_HIP(hipGetLastError());
    unsigned long long h = 0;
    SA_HIP(hipMemcpyAsync(&h, added, 8, hipMemcpyDeviceToHost, s));
    SA_HIP(hipStreamSynchronize(s));
    if (added_out) *added_out = (int64_t)h;
    return SA_OK;
}

namespace {

// Links of the gateway vertices on the host, for more representatives than link_kernel
// sorts: dv[a][c] distances of source a (nc representatives first) to representative c.
void host_links(const std::vector<int32_t> &src, const std::vector<int32_t> &rep, const std::vector<float> &dv, int R,
                int keep_local, int hub_keep_local, std::vector<int32_t> &links)
{
    const int64_t nc = (int64_t)rep.size();
    struct Cd {
        float d;
        int32_t id, c;
        bool used;
    };
    std::vector<Cd> cand;
    for (int64_t a = 0; a < (int64_t)src.size(); ++a) {
        const int cap = R - (a < nc ? keep_local : hub_keep_local);
        if (cap <= 0) continue;
        cand.clear();
        for (int64_t c = 0; c < nc; ++c)
            if (rep[c] != src[a]) cand.push_back({dv[(size_t)(a * nc + c)], rep[c], (int32_t)c, false});
        std::sort(cand.begin(), cand.end(), [](const Cd &x, const Cd &y) { return key_less_host(x.d, x.id, y.d, y.id); });
        int32_t *out = &links[(size_t)a * R];
        std::vector<int32_t> kc;
        for (auto &c : cand) {
            if ((int)kc.size() >= cap) break;
            bool keep = true;
            for (int32_t x : kc)
                if (dv[(size_t)x * nc + c.c] < c.d) {
                    keep = false;
                    break;
                }
            if (keep) {
                kc.push_back(c.c);
                c.used = true;
            }
        }
        int kept = 0;
        for (int32_t x : kc) out[kept++] = rep[x];
        for (auto &c : cand) {
            if (kept >= cap) break;
            if (!c.used) out[kept++] = c.id;
        }
    }
}

// Weakly connected components of n rows, numbered by their smallest vertices; returns how many.
int64_t host_components(const std::vector<int32_t> &adj, int64_t n, int R, std::vector<int32_t> &comp)
{
    std::vector<int32_t> par((size_t)n);
    for (int64_t i = 0; i < n; ++i) par[i] = (int32_t)i;
    const auto root = [&](int32_t x) {
        while (par[x] != x) x = par[x] = par[par[x]];
        return x;
    };
    for (int64_t v = 0; v < n; ++v)
        for (int r = 0; r < R; ++r) {
            const int32_t u = adj[v * R + r];
            if (u < 0 || u >= n) continue;
            const int32_t a = root((int32_t)v), b = root(u);
            if (a != b) par[std::max(a, b)] = std::min(a, b);
        }
    comp.resize((size_t)n);
    int64_t nc = 0;
    for (int64_t i = 0; i < n; ++i) {   // (a root is the smallest vertex of its component)
        const int32_t x = root((int32_t)i);
        comp[i] = x == i ? (int32_t)nc++ : comp[x];
    }
    return nc;
}

// Puts rows back that a repair which then fails has written: its caller's rows are either
// repaired or as they were.
struct RowsBack {
    const int32_t *src = nullptr, *rows = nullptr;
    int64_t cnt = 0;
    int32_t *adj;
    int R;
    hipStream_t s;
    RowsBack(int32_t *adj_, int R_, hipStream_t s_) : adj(adj_), R(R_), s(s_) {}
    ~RowsBack()
    {
        if (cnt == 0) return;
        hipLaunchKernelGGL(put_rows, dim3(blocks_for(cnt * R, 256)), dim3(256), 0, s, src, cnt, rows, R, adj);
        (void)hipStreamSynchronize(s);
    }
};

}  // namespace

int repair_device(const float *base, int64_t n, int d, int64_t ld, int metric, int32_t *adj_dev, int R,
                  int32_t entry, int keep_local, int hubs, int hub_keep_local, int64_t *bridges_out,
                  int64_t *ncomp_out, hipStream_t s)
{
    const int64_t ne = n * R, nchunk = (n + SCAN_CHUNK - 1) / SCAN_CHUNK;
    const int dcol = (d + 63) / 64;
    // Components and reachability of up to 2^17 edges come from a copy of the rows on the host:
    // some twenty launches and three looks at their results take 200 us on any connected graph,
    // the copy and the host 61 us at 300 rows of 32 and 442 at 3,000 (against 540).
    const bool small = ne <= (1 << 17);
    std::vector<int32_t> hadj, hcomp;
    Arena A;
    const size_t o_par = A.want<int32_t>(n), o_root = A.want<int32_t>(n), o_flag = A.want<int32_t>(n), o_num = A.want<int64_t>(n + 1);
    const size_t o_sums = A.want<int64_t>(nchunk), o_dist = A.want<double>(n), o_mark = A.want<uint8_t>(n), o_chg = A.want<int32_t>(1);
    const dim3 bn(blocks_for(n, 256)), t256(256);
    const auto copy_rows = [&]() -> int {
        hadj.resize((size_t)ne);
        SA_HIP(hipMemcpyAsync(hadj.data(), adj_dev, sizeof(int32_t) * ne, hipMemcpyDeviceToHost, s));
        SA_HIP(hipStreamSynchronize(s));
        return SA_OK;
    };

    // (1) weakly connected components, numbered by smallest member
    int64_t nc = 0;
    if (small) {
        const int rc = copy_rows();
        if (rc != SA_OK) return rc;
        nc = host_components(hadj, n, R, hcomp);
    }
    if (!small || nc > 1)
        if (A.alloc() != hipSuccess) return set_error(SA_ENOMEM, "repair: device allocation failed");
    int32_t *par = A.get<int32_t>(o_par);
    if (!small) {
        int32_t *const root = A.get<int32_t>(o_root), *const flag = A.get<int32_t>(o_flag);
        int64_t *const num = A.get<int64_t>(o_num);
        hipLaunchKernelGGL(uf_init, bn, t256, 0, s, par, n);
        hipLaunchKernelGGL(uf_hook, dim3(blocks_for(ne, 256)), t256, 0, s, adj_dev, n, R, par);
        hipLaunchKernelGGL(uf_flatten, bn, t256, 0, s, par, n, root, flag);
        SA_HIP(hipGetLastError());
        SA_HIP(prefix_sums(flag, n, A.get<int64_t>(o_sums), num, s));
        SA_HIP(hipMemcpyAsync(&nc, num + n, 8, hipMemcpyDeviceToHost, s));
        SA_HIP(hipStreamSynchronize(s));
    }
    if (ncomp_out) *ncomp_out = nc;

    // (2) gateway rows for the representatives (each component's medoid), the entry and the
    // hubs (the vertices nearest to the mean of all rows)
    Arena D;
    RowsBack back(adj_dev, R, s);   // (before D goes)
    if (nc > 1) {
        int32_t *const comp = par;   // (the union-find is done with it)
        double *const dist = A.get<double>(o_dist);
        if (small) {
            SA_HIP(hipMemcpyAsync(comp, hcomp.data(), sizeof(int32_t) * n, hipMemcpyHostToDevice, s));
        } else {
            hipLaunchKernelGGL(comp_of, bn, t256, 0, s, A.get<int32_t>(o_root), A.get<int64_t>(o_num), n, comp);
            hcomp.resize((size_t)n);
            SA_HIP(hipMemcpyAsync(hcomp.data(), comp, sizeof(int32_t) * n, hipMemcpyDeviceToHost, s));
            SA_HIP(hipStreamSynchronize(s));
        }
        std::vector<int32_t> members((size_t)n);
        std::vector<int64_t> start((size_t)nc + 1, 0);
        for (int64_t i = 0; i < n; ++i) start[hcomp[i] + 1]++;
        for (int64_t c = 0; c < nc; ++c) start[c + 1] += start[c];
        {
            std::vector<int64_t> fill(start.begin(), start.end() - 1);
            for (int64_t i = 0; i < n; ++i) members[fill[hcomp[i]]++] = (int32_t)i;
        }
        Arena C;
        const size_t o_mem = C.want<int32_t>(n), o_start = C.want<int64_t>(nc + 1), o_mean = C.want<double>((nc + 1) * d);
        const size_t o_best = C.want<unsigned long long>(nc), o_rep = C.want<int32_t>(nc);
        if (C.alloc() != hipSuccess) return set_error(SA_ENOMEM, "repair: device allocation failed");
        int32_t *const rep_dev = C.get<int32_t>(o_rep);
        int64_t *const start_dev = C.get<int64_t>(o_start);
        double *const mean = C.get<double>(o_mean);
        SA_HIP(hipMemcpyAsync(C.get<int32_t>(o_mem), members.data(), sizeof(int32_t) * n, hipMemcpyHostToDevice, s));
        SA_HIP(hipMemcpyAsync(start_dev, start.data(), sizeof(int64_t) * (nc + 1), hipMemcpyHostToDevice, s));
        const bool want_hubs = hubs > 1;
        hipLaunchKernelGGL(group_means, dim3((unsigned)(nc + (want_hubs ? 1 : 0)), (unsigned)dcol), dim3(64), 0, s, base, n, d,
                           ld, C.get<int32_t>(o_mem), start_dev, nc, mean);
        hipLaunchKernelGGL(mean_dists, bn, t256, 0, s, base, n, d, ld, mean, comp, dist);
        hipLaunchKernelGGL(fill_u64_n, dim3(blocks_for(nc, 256)), t256, 0, s, C.get<unsigned long long>(o_best), nc,
                           (unsigned long long)KEY_EMPTY);
        hipLaunchKernelGGL(fill_i32, dim3(blocks_for(nc, 256)), t256, 0, s, rep_dev, nc, INT32_MAX);
        for (int pass = 0; pass < 2; ++pass)
            hipLaunchKernelGGL(nearest_member, bn, t256, 0, s, dist, comp, n, pass, C.get<unsigned long long>(o_best), rep_dev);
        SA_HIP(hipGetLastError());
        std::vector<int32_t> rep((size_t)nc);
        SA_HIP(hipMemcpyAsync(rep.data(), rep_dev, sizeof(int32_t) * nc, hipMemcpyDeviceToHost, s));
        std::vector<double> hd;
        if (want_hubs) {
            hipLaunchKernelGGL(mean_dists, bn, t256, 0, s, base, n, d, ld, mean + nc * d, (const int32_t *)nullptr, dist);
            SA_HIP(hipGetLastError());
            hd.resize((size_t)n);
            SA_HIP(hipMemcpyAsync(hd.data(), dist, sizeof(double) * n, hipMemcpyDeviceToHost, s));
        }
        SA_HIP(hipStreamSynchronize(s));
        std::vector<uint8_t> is_rep((size_t)n, 0);
        for (int64_t c = 0; c < nc; ++c) is_rep[rep[c]] = 1;
        std::vector<int32_t> src(rep);
        if (!is_rep[entry]) src.push_back(entry);
        if (want_hubs) {
            struct H {
                double d;
                int32_t v;
            };
            std::vector<H> hv;
            hv.reserve((size_t)n);
            for (int64_t v = 0; v < n; ++v)
                if (!is_rep[v] && v != entry) hv.push_back({hd[v], (int32_t)v});
            const size_t take = std::min(hv.size(), (size_t)(hubs - 1));
            std::partial_sort(hv.begin(), hv.begin() + take, hv.end(),
                              [](const H &x, const H &y) { return x.d < y.d || (x.d == y.d && x.v < y.v); });
            for (size_t j = 0; j < take; ++j) src.push_back(hv[j].v);
        }
        const int64_t nsrc = (int64_t)src.size();
        const size_t o_src = D.want<int32_t>(nsrc), o_dv = D.want<float>(nsrc * nc), o_links = D.want<int32_t>(nsrc * R);
        const size_t o_old = D.want<int32_t>(nsrc * R);
        if (D.alloc() != hipSuccess) return set_error(SA_ENOMEM, "repair: device allocation failed");
        int32_t *const src_dev = D.get<int32_t>(o_src), *const links = D.get<int32_t>(o_links);
        float *const dv = D.get<float>(o_dv);
        SA_HIP(hipMemcpyAsync(src_dev, src.data(), sizeof(int32_t) * nsrc, hipMemcpyHostToDevice, s));
        // rows 0 .. nc - 1: distances between representatives, for the occlusion test
        hipLaunchKernelGGL(pair_dists, dim3(blocks_for(nsrc * nc, 256)), t256, 0, s, base, d, ld, metric, src_dev, nsrc, rep_dev,
                           nc, dv);
        SA_HIP(hipGetLastError());
        if (nc <= LINK_REPS) {
            int P = 64;
            while (P < nc) P <<= 1;
            hipLaunchKernelGGL(link_kernel, dim3((unsigned)nsrc), t256, 9 * (size_t)P, s, src_dev, nc, rep_dev, comp, dv, dv, R,
                               keep_local, hub_keep_local, P, links);
            SA_HIP(hipGetLastError());
        } else {
            std::vector<float> hdv((size_t)(nsrc * nc));
            SA_HIP(hipMemcpyAsync(hdv.data(), dv, sizeof(float) * hdv.size(), hipMemcpyDeviceToHost, s));
            SA_HIP(hipStreamSynchronize(s));
            std::vector<int32_t> hl((size_t)nsrc * R, -1);
            host_links(src, rep, hdv, R, keep_local, hub_keep_local, hl);
            SA_HIP(hipMemcpyAsync(links, hl.data(), sizeof(int32_t) * hl.size(), hipMemcpyHostToDevice, s));
            SA_HIP(hipStreamSynchronize(s));
        }
        hipLaunchKernelGGL(gather_rows, dim3(blocks_for(nsrc * R, 256)), t256, 0, s, adj_dev, (int64_t)R, R, src_dev, nsrc,
                           D.get<int32_t>(o_old));
        SA_HIP(hipGetLastError());
        back.src = src_dev;
        back.rows = D.get<int32_t>(o_old);
        back.cnt = nsrc;
        hipLaunchKernelGGL(gateway_rows, dim3((unsigned)nsrc), dim3(64), 0, s, src_dev, nc, links, R, keep_local, hub_keep_local,
                           adj_dev);
        SA_HIP(hipGetLastError());
        SA_HIP(hipStreamSynchronize(s));
    }

    // (3) reachability: bridge every unreachable vertex, in id order, from the nearest
    // reachable vertex with a free slot
    std::vector<uint8_t> mark;
    if (small) {
        if (nc > 1) {
            const int rc = copy_rows();
            if (rc != SA_OK) return rc;
        }
        mark.assign((size_t)n, 0);
        std::vector<int32_t> walk(1, entry);
        mark[entry] = 1;
        for (size_t h = 0; h < walk.size(); ++h)
            for (int r = 0; r < R; ++r) {
                const int32_t u = hadj[(int64_t)walk[h] * R + r];
                if (u < 0 || u >= n || mark[u]) continue;
                mark[u] = 1;
                walk.push_back(u);
            }
    } else {
        int32_t *const level = A.get<int32_t>(o_root), *const changed = A.get<int32_t>(o_chg);
        hipLaunchKernelGGL(fill_i32, bn, t256, 0, s, level, n, -1);
        hipLaunchKernelGGL(fill_i32, dim3(1), dim3(64), 0, s, level + entry, (int64_t)1, 0);
        SA_HIP(hipGetLastError());
        // A level a launch, eight launches a look at the flag; what is not finished after 128
        // levels is a long thin graph, which the host walks faster (a level is some 6 us here).
        bool done = false;
        for (int32_t cur = 0; !done && cur < 128; cur += 8) {
            for (int32_t i = 0; i < 8; ++i) {
                if (i == 7) hipLaunchKernelGGL(fill_i32, dim3(1), dim3(64), 0, s, changed, (int64_t)1, 0);
                hipLaunchKernelGGL(bfs_level, dim3(blocks_for(n, 256)), t256, 0, s, adj_dev, n, R, level, cur + i, changed);
            }
            SA_HIP(hipGetLastError());
            int32_t h = 0;
            SA_HIP(hipMemcpyAsync(&h, changed, 4, hipMemcpyDeviceToHost, s));
            SA_HIP(hipStreamSynchronize(s));
            done = h == 0;
        }
        if (!done) {
            std::vector<int32_t> adj((size_t)ne), lv((size_t)n), walk;
            SA_HIP(hipMemcpyAsync(adj.data(), adj_dev, sizeof(int32_t) * ne, hipMemcpyDeviceToHost, s));
            SA_HIP(hipMemcpyAsync(lv.data(), level, sizeof(int32_t) * n, hipMemcpyDeviceToHost, s));
            SA_HIP(hipStreamSynchronize(s));
            for (int64_t v = 0; v < n; ++v)
                if (lv[v] >= 0) walk.push_back((int32_t)v);
            for (size_t h = 0; h < walk.size(); ++h)
                for (int r = 0; r < R; ++r) {
                    const int32_t u = adj[(int64_t)walk[h] * R + r];
                    if (u < 0 || u >= n || lv[u] >= 0) continue;
                    lv[u] = 0;
                    walk.push_back(u);
                }
            SA_HIP(hipMemcpyAsync(level, lv.data(), sizeof(int32_t) * n, hipMemcpyHostToDevice, s));
            SA_HIP(hipStreamSynchronize(s));
        }
        hipLaunchKernelGGL(level_marks, bn, t256, 0, s, level, n, A.get<uint8_t>(o_mark));
        hipLaunchKernelGGL(row_degrees, dim3(blocks_for(n, 4)), t256, 0, s, adj_dev, n, R, 0, A.get<int32_t>(o_flag));
        SA_HIP(hipGetLastError());
        mark.resize((size_t)n);
        SA_HIP(hipMemcpyAsync(mark.data(), A.get<uint8_t>(o_mark), n, hipMemcpyDeviceToHost, s));
        SA_HIP(hipStreamSynchronize(s));
    }
    std::vector<int32_t> lost;   // unreachable vertices, in id order
    for (int64_t v = 0; v < n; ++v)
        if (!mark[v]) lost.push_back((int32_t)v);
    int64_t added = 0;
    if (!lost.empty()) {
        // Only rows and vectors of unreachable vertices are looked at from here on: a walk
        // from one of them marks none but them.
        const int64_t nl = (int64_t)lost.size();
        constexpr int WIN = 256;
        constexpr size_t MAX_NEW = 4096;
        if (!A.p && A.alloc() != hipSuccess) return set_error(SA_ENOMEM, "repair: device allocation failed");
        int32_t *const deg = A.get<int32_t>(o_flag);
        uint8_t *const dmask = A.get<uint8_t>(o_mark);
        std::vector<int32_t> hdeg((size_t)n), lrow((size_t)nl * R);
        std::vector<float> lvec((size_t)nl * d);
        Arena G;
        const size_t o_ids = G.want<int32_t>(nl), o_rows = G.want<int32_t>(nl * R), o_vecs = G.want<float>(nl * d);
        const size_t o_us = G.want<int32_t>(WIN), o_res = G.want<unsigned long long>(WIN);
        if (G.alloc() != hipSuccess) return set_error(SA_ENOMEM, "repair: device allocation failed");
        int32_t *const ids = G.get<int32_t>(o_ids), *const dus = G.get<int32_t>(o_us);
        unsigned long long *const dres = G.get<unsigned long long>(o_res);
        if (small)
            for (int64_t e = 0; e < ne; ++e) hdeg[e / R] += hadj[e] >= 0 ? 1 : 0;
        else
            SA_HIP(hipMemcpyAsync(hdeg.data(), deg, sizeof(int32_t) * n, hipMemcpyDeviceToHost, s));
        SA_HIP(hipMemcpyAsync(ids, lost.data(), sizeof(int32_t) * nl, hipMemcpyHostToDevice, s));
        hipLaunchKernelGGL(gather_rows, dim3(blocks_for(nl * R, 256)), t256, 0, s, adj_dev, (int64_t)R, R, ids, nl,
                           G.get<int32_t>(o_rows));
        hipLaunchKernelGGL(gather_rows, dim3(blocks_for(nl * d, 256)), t256, 0, s, reinterpret_cast<const int32_t *>(base), ld, d,
                           ids, nl, G.get<int32_t>(o_vecs));
        SA_HIP(hipGetLastError());
        SA_HIP(hipMemcpyAsync(lrow.data(), G.get<int32_t>(o_rows), sizeof(int32_t) * lrow.size(), hipMemcpyDeviceToHost, s));
        SA_HIP(hipMemcpyAsync(lvec.data(), G.get<float>(o_vecs), sizeof(float) * lvec.size(), hipMemcpyDeviceToHost, s));
        SA_HIP(hipStreamSynchronize(s));
        auto slot_of = [&](int32_t v) { return (size_t)(std::lower_bound(lost.begin(), lost.end(), v) - lost.begin()); };
        // marks src and what its rows reach; newly gets them in the order met
        std::vector<int32_t> newly;
        auto mark_from = [&](int32_t src) {
            newly.clear();
            if (mark[src]) return;
            mark[src] = 1;
            newly.push_back(src);
            for (size_t h = 0; h < newly.size(); ++h) {
                const int32_t *row = &lrow[slot_of(newly[h]) * R];
                for (int r = 0; r < R; ++r) {
                    const int32_t u = row[r];
                    if (u < 0 || u >= n || mark[u]) continue;
                    mark[u] = 1;
                    newly.push_back(u);
                }
            }
        };
        // In id order, as one at a time, but the searches go out in windows of WIN vertices:
        // one launch finds, for each, the nearest vertex with a free slot among those marked
        // when the window starts; processing the window in order, each answer is corrected
        // with the vertices marked since (the same distance arithmetic on the host), and
        // found again alone if its vertex has no free slot left.  The edges are those the
        // one-at-a-time loop adds.  A window ends early once many vertices were marked in it.
        std::vector<int32_t> us;
        std::vector<unsigned long long> res(WIN);
        std::vector<int32_t> since;      // vertices marked since the window's searches
        std::vector<int64_t> edit_pos;   // the edges added
        std::vector<int32_t> edit_val;
        // nearest marked vertex with a free slot for each of q, under the current marks and degrees
        auto search = [&](const std::vector<int32_t> &q) -> int {
            SA_HIP(hipMemcpyAsync(dmask, mark.data(), n, hipMemcpyHostToDevice, s));
            SA_HIP(hipMemcpyAsync(deg, hdeg.data(), sizeof(int32_t) * n, hipMemcpyHostToDevice, s));
            SA_HIP(hipMemcpyAsync(dus, q.data(), sizeof(int32_t) * q.size(), hipMemcpyHostToDevice, s));
            hipLaunchKernelGGL(fill_u64_n, dim3(1), dim3(WIN), 0, s, dres, (int64_t)q.size(), (unsigned long long)KEY_EMPTY);
            hipLaunchKernelGGL(nearest_marked_batch, dim3(blocks_for(n, 256), blocks_for((int64_t)q.size(), NM_Q)), t256, 0, s,
                               base, n, d, ld, metric, dmask, deg, R, dus, (int)q.size(), dres);
            SA_HIP(hipGetLastError());
            SA_HIP(hipMemcpyAsync(res.data(), dres, sizeof(unsigned long long) * q.size(), hipMemcpyDeviceToHost, s));
            SA_HIP(hipStreamSynchronize(s));
            return SA_OK;
        };
        size_t next = 0;   // place in lost
        while (next < lost.size()) {
            us.clear();
            size_t at = next;
            for (; at < lost.size() && (int)us.size() < WIN; ++at)
                if (!mark[lost[at]]) us.push_back(lost[at]);
            if (us.empty()) break;
            int rc = search(us);
            if (rc != SA_OK) return rc;
            since.clear();
            next = at;
            for (size_t j = 0; j < us.size(); ++j) {
                const int32_t u = us[j];
                if (mark[u]) continue;
                const size_t su = slot_of(u);
                if (since.size() > MAX_NEW) {   // many new candidates: search the rest of the window again
                    next = su;
                    break;
                }
                // the window's answer is the best over the vertices marked at its start; those
                // that filled up since cannot be taken, and those marked since are candidates
                unsigned long long best = res[j];
                if (best != KEY_EMPTY && hdeg[key_id(best)] >= R) {
                    const std::vector<unsigned long long> saved(res);
                    if ((rc = search(std::vector<int32_t>{u})) != SA_OK) return rc;
                    best = res[0];
                    res = saved;
                } else {
                    for (int32_t w : since)
                        if (hdeg[w] < R) {
                            const unsigned long long k =
                                make_key(host_dist(&lvec[slot_of(w) * d], &lvec[su * d], d, metric), w);
                            if (k < best) best = k;
                        }
                }
                if (best == KEY_EMPTY) return set_error(SA_ECAPACITY, "repair: no reachable vertex has a free slot");
                const int32_t r = key_id(best);
                edit_pos.push_back((int64_t)r * R + hdeg[r]);
                edit_val.push_back(u);
                hdeg[r]++;
                ++added;
                mark_from(u);
                since.insert(since.end(), newly.begin(), newly.end());
            }
        }
        Arena E;
        const size_t o_pos = E.want<int64_t>(added), o_val = E.want<int32_t>(added);
        if (E.alloc() != hipSuccess) return set_error(SA_ENOMEM, "repair: device allocation failed");
        SA_HIP(hipMemcpyAsync(E.get<int64_t>(o_pos), edit_pos.data(), sizeof(int64_t) * added, hipMemcpyHostToDevice, s));
        SA_HIP(hipMemcpyAsync(E.get<int32_t>(o_val), edit_val.data(), sizeof(int32_t) * added, hipMemcpyHostToDevice, s));
        hipLaunchKernelGGL(apply_edits, dim3(blocks_for(added, 256)), t256, 0, s, E.get<int64_t>(o_pos), E.get<int32_t>(o_val),
                           added, adj_dev);
        SA_HIP(hipGetLastError());
        SA_HIP(hipStreamSynchronize(s));
    }
    back.cnt = 0;
    if (bridges_out) *bridges_out = added;
    return SA_OK;
}

}  // namespace sa
