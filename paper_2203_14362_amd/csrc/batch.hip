// Resident point tables and query batches.
//
// A table keeps the points in HBM sorted by the cell of a G x G grid over
// their bounding box (cells in Z order) and cut into chunks of CHUNK points
// with their exact bounding boxes.  A batch is a canvas set (one canvas per
// query).  Work is organised by (chunk, query) pairs whose boxes overlap: a
// wavefront holds a part of a chunk's points in registers and tests them
// against every query that can contain one of them, so a chunk is read from
// HBM once per pass for the whole batch.  Selection and join pairs use the
// paper's two-step Map (Sec. 5.1): a selection's probe pass keeps every pair's
// match bits, whose ids are counted per window of ids and put in order window
// by window; a join's count pass sizes every point's output range, a scan
// places the ranges in id order and a write pass fills them (few pairs are
// sorted as keys instead).  The join-count needs no pair list: its single probe
// launch finds each chunk's queries itself.
#include "common.h"
#include "exact.h"
#include "lookup.h"

#include <hipcub/hipcub.hpp>
#include <rocprim/device/device_scan.hpp>
#include <rocprim/iterator/transform_iterator.hpp>
#include <rocprim/warp/warp_scan.hpp>

#include <algorithm>
#include <cstdlib>
#include <cmath>
#include <cstring>
#include <new>
#include <utility>
#include <vector>

namespace spade {

constexpr int CHUNK = 4096;               // table points per chunk
constexpr int BT_THREADS = 256;           // batch probe workgroup
constexpr int BT_PER = CHUNK / BT_THREADS;
constexpr int GRID_MAX = 1024;            // table grid side

}  // namespace spade

struct spade_table {
    int device = 0;
    int64_t n = 0;        // points
    int64_t nfin = 0;     // points with finite coordinates (clustered prefix)
    int G = 1;
    double X0 = 0, Y0 = 0, sx = 0, sy = 0;
    int64_t nchunk = 0;
    spade::DevBuf x, y, ids, chunk_bb;
    size_t bytes() const { return x.cap + y.cap + ids.cap + chunk_bb.cap; }
};

namespace spade {

__device__ __forceinline__ unsigned long long okey(double v)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    return (b & 0x8000000000000000ull) ? ~b : (b | 0x8000000000000000ull);
}

static double from_okey(unsigned long long k)
{
    const unsigned long long b = (k & 0x8000000000000000ull) ? (k & 0x7fffffffffffffffull) : ~k;
    double d;
    std::memcpy(&d, &b, sizeof d);
    return d;
}

static int grid_of(int64_t n, int64_t cap = 65536)
{
    return (int)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, cap));
}

static int bits_of(uint64_t v)
{
    int b = 0;
    while (b < 64 && (v >> b) != 0) ++b;
    return b;
}

// Bounding box of the finite points: keys of (min x, -max x, min y, -max y).
__global__ __launch_bounds__(256) void k_pt_bbox(int64_t n, const double *X, const double *Y,
                                                 unsigned long long *bb)
{
    __shared__ unsigned long long s[4][256];
    unsigned long long k0 = ~0ull, k1 = ~0ull, k2 = ~0ull, k3 = ~0ull;
    const int64_t nth = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += nth) {
        const double x = X[i], y = Y[i];
        if (!isfinite(x) || !isfinite(y)) continue;
        k0 = min(k0, okey(x)); k1 = min(k1, okey(-x));
        k2 = min(k2, okey(y)); k3 = min(k3, okey(-y));
    }
    s[0][threadIdx.x] = k0; s[1][threadIdx.x] = k1; s[2][threadIdx.x] = k2; s[3][threadIdx.x] = k3;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            for (int q = 0; q < 4; ++q) s[q][threadIdx.x] = min(s[q][threadIdx.x], s[q][threadIdx.x + w]);
        __syncthreads();
    }
    if (threadIdx.x < 4) atomicMin(&bb[threadIdx.x], s[threadIdx.x][0]);
}

// Grid cell key of every point (non-finite points: G * G, sorted last).
// The bits of v (< 2^16) spread to the even bit positions.
__device__ __forceinline__ uint32_t spread_bits(uint32_t v)
{
    v = (v | (v << 8)) & 0x00ff00ffu;
    v = (v | (v << 4)) & 0x0f0f0f0fu;
    v = (v | (v << 2)) & 0x33333333u;
    v = (v | (v << 1)) & 0x55555555u;
    return v;
}

// Sort key of each point: the Z-order (Morton) index of its cell of the
// G x G grid, so that runs of consecutive cells, and hence table chunks,
// are compact in space; nonfinite points get nfkey, after every cell.
__global__ void k_pt_key(int64_t n, const double *X, const double *Y, double X0, double Y0, double sx,
                         double sy, int G, uint32_t nfkey, uint32_t *keys, uint32_t *idx)
{
    const int64_t nth = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += nth) {
        const double x = X[i], y = Y[i];
        uint32_t k = nfkey;
        if (isfinite(x) && isfinite(y)) {
            const int cx = (int)fmin((double)(G - 1), fmax(0.0, floor((x - X0) * sx)));
            const int cy = (int)fmin((double)(G - 1), fmax(0.0, floor((y - Y0) * sy)));
            k = spread_bits((uint32_t)cx) | (spread_bits((uint32_t)cy) << 1);
        }
        keys[i] = k;
        idx[i] = (uint32_t)i;
    }
}

__global__ void k_pt_gather(int64_t n, const uint32_t *perm, const double *X, const double *Y, double *x2,
                            double *y2)
{
    const int64_t nth = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += nth) {
        const uint32_t p = perm[i];
        x2[i] = X[p];
        y2[i] = Y[p];
    }
}

// The sorted points with a cell: the keys below nfkey (non-finite points
// have it).
__global__ void k_count_finite(int64_t n, const uint32_t *skeys, uint32_t nfkey, uint32_t *nfin)
{
    int64_t lo = 0, hi = n;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (skeys[mid] < nfkey) lo = mid + 1; else hi = mid;
    }
    *nfin = (uint32_t)lo;
}

// Exact bounding box of every chunk of the finite prefix (one wave per chunk).
__global__ __launch_bounds__(256) void k_chunk_bb(int64_t nfin, int64_t nchunk, const double *X,
                                                  const double *Y, double4 *bb)
{
    const int lane = threadIdx.x & 63;
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t nw = ((int64_t)gridDim.x * blockDim.x) >> 6;
    for (int64_t c = wave; c < nchunk; c += nw) {
        const int64_t b = c * CHUNK, e = std::min<int64_t>(nfin, b + CHUNK);
        double x0 = INFINITY, x1 = -INFINITY, y0 = INFINITY, y1 = -INFINITY;
        for (int64_t i = b + lane; i < e; i += 64) {
            x0 = fmin(x0, X[i]); x1 = fmax(x1, X[i]);
            y0 = fmin(y0, Y[i]); y1 = fmax(y1, Y[i]);
        }
        for (int d = 32; d > 0; d >>= 1) {
            x0 = fmin(x0, __shfl_xor(x0, d, 64)); x1 = fmax(x1, __shfl_xor(x1, d, 64));
            y0 = fmin(y0, __shfl_xor(y0, d, 64)); y1 = fmax(y1, __shfl_xor(y1, d, 64));
        }
        if (lane == 0) bb[c] = make_double4(x0, y0, x1, y1);
    }
}

// ------------------------------------------------------------ pairs

// Chunk c can hold a point of canvas q: its closed point box meets the
// canvas's half-open polygon box.
__device__ __forceinline__ bool overlaps(const double4 &b, const CanvasDesc &d)
{
    return !d.empty && b.z >= d.bx0 && b.x < d.bx1 && b.w >= d.by0 && b.y < d.by1;
}

// The (chunk, query) pairs, in query-major order with chunk-major lists of
// them.  A thread takes a chunk and PAIR_Q queries (blockIdx.y); FILL = false
// counts per query and per chunk, FILL lists them (the order of a query's
// pairs and of a chunk's list is not fixed).
constexpr int PAIR_Q = 32;

template <bool FILL>
__global__ __launch_bounds__(256) void k_pairs(int nq, int64_t nchunk, const double4 *bb, const CanvasDesc *cds,
                                               unsigned long long *qn, const unsigned long long *qbase,
                                               unsigned int *cn, const unsigned int *cbase, uint32_t *pq, uint32_t *pc,
                                               uint32_t *plist)
{
    const int lane = threadIdx.x & 63;
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const double4 b = c < nchunk ? bb[c] : make_double4(INFINITY, INFINITY, -INFINITY, -INFINITY);
    for (int q0 = blockIdx.y * PAIR_Q; q0 < nq; q0 += gridDim.y * PAIR_Q) {
        const int q1 = min(nq, q0 + PAIR_Q);
        uint32_t mine = 0u;   // the queries of this chunk, bit q - q0
        for (int q = q0; q < q1; ++q) {
            const bool on = overlaps(b, cds[q]);
            const unsigned long long m = __ballot(on);
            mine |= (on ? 1u : 0u) << (q - q0);
            if (!FILL && m && lane == 0) atomicAdd(&qn[q], (unsigned long long)__popcll(m));
        }
        if (!FILL) {
            if (mine) atomicAdd(&cn[c], (unsigned int)__popc(mine));
            continue;
        }
        uint32_t at = mine ? cbase[c] + atomicAdd(&cn[c], (unsigned int)__popc(mine)) : 0u;
        for (int q = q0; q < q1; ++q) {
            const bool on = (mine >> (q - q0)) & 1u;
            const unsigned long long m = __ballot(on);
            if (!m) continue;
            unsigned long long first = 0ull;
            if (lane == 0) first = atomicAdd(&qn[q], (unsigned long long)__popcll(m));
            const unsigned long long p =
                qbase[q] + (unsigned long long)__shfl((long long)first, 0, 64) + __popcll(m & ((1ull << lane) - 1ull));
            if (on) {
                pq[p] = (uint32_t)q;
                pc[p] = (uint32_t)c;
                plist[at++] = (uint32_t)p;
            }
        }
    }
}

// Exclusive scans of the per-query counts and the first tile of every query
// (workgroup 0) and of the per-chunk counts (workgroup 1) (qbase[nq],
// cbase[nchunk] = total); the counts cleared to serve as cursors, and qbase
// copied to the host's words.
constexpr int PS_THREADS = 1024;
constexpr int PS_REG = 12;

template <typename T, typename Get, typename Put>
__device__ void scan_block(int64_t n, T *wsum, Get get, Put put)
{
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int64_t per = (n + PS_THREADS - 1) / PS_THREADS, b = min(n, tid * per), e = min(n, b + per);
    // PS_REG values in flight, kept for the second pass when they are all
    T v[PS_REG], mine = 0;
    auto fetch = [&](int64_t i) {
#pragma unroll
        for (int k = 0; k < PS_REG; ++k) v[k] = i + k < e ? get(i + k) : (T)0;
    };
    for (int64_t i = b; i < e; i += PS_REG) {
        fetch(i);
#pragma unroll
        for (int k = 0; k < PS_REG; ++k) mine += v[k];
    }
    T inc = mine;
    for (int d = 1; d < 64; d <<= 1) {
        const T t = __shfl_up(inc, d, 64);
        if (lane >= d) inc += t;
    }
    if (lane == 63) wsum[wv] = inc;
    __syncthreads();
    T at = inc - mine;
    for (int w = 0; w < wv; ++w) at += wsum[w];
    for (int64_t i = b; i < e; i += PS_REG) {
        if (per > PS_REG) fetch(i);
#pragma unroll
        for (int k = 0; k < PS_REG; ++k)
            if (i + k < e) {
                put(i + k, at);
                at += v[k];
            }
    }
    if (tid == PS_THREADS - 1) put(n, at);
    __syncthreads();
}

__global__ __launch_bounds__(PS_THREADS) void k_pair_scan(int nq, int64_t nchunk, unsigned long long *qn,
                                                          unsigned long long *qbase, unsigned int *cn,
                                                          unsigned int *cbase, int tile, uint32_t *tfirst,
                                                          unsigned long long *hbase)
{
    __shared__ unsigned long long ws[PS_THREADS / 64];
    __shared__ uint32_t wt[PS_THREADS / 64];
    if (blockIdx.x == 0) {
        scan_block<unsigned long long>(nq, ws, [&](int64_t q) { return qn[q]; }, [&](int64_t q, unsigned long long at) {
            qbase[q] = at;
            __hip_atomic_store(&hbase[q], at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        });
        scan_block<uint32_t>(nq, wt, [&](int64_t q) { return (uint32_t)((qn[q] + tile - 1) / tile); },
                             [&](int64_t q, uint32_t at) { tfirst[q] = at; });
        for (int64_t q = threadIdx.x; q < nq; q += PS_THREADS) qn[q] = 0ull;
    } else {
        scan_block<uint32_t>(nchunk, wt, [&](int64_t c) { return cn[c]; }, [&](int64_t c, uint32_t at) { cbase[c] = at; });
        for (int64_t c = threadIdx.x; c < nchunk; c += PS_THREADS) cn[c] = 0u;
    }
    __threadfence_system();
}

// Canvas q of a set as a probe view (descriptor in device memory).
__device__ __forceinline__ CanvasView set_view(const CanvasDesc &d, const uint32_t *cells, const uint16_t *coarse,
                                               const Cand *cands,
                                               const Edge *ledges, const double2 *pspan)
{
    CanvasView v;
    v.X0 = d.X0; v.Y0 = d.Y0; v.sx = d.sx; v.sy = d.sy;
    v.bx0 = d.bx0; v.by0 = d.by0; v.bx1 = d.bx1; v.by1 = d.by1;
    v.W = d.W; v.H = d.H; v.Wt = d.Wt; v.Wc = d.Wc; v.Hc = d.Hc; v.blog = d.blog;
    v.cbyte = d.cbyte;
    v.M = d.M;
    v.cells = cells + d.cell_off;
    v.coarse = coarse + d.coarse_off;
    v.cands = cands;
    v.ledges = ledges;
    v.pspan = pspan;
    return v;
}

struct SetArgs {
    const CanvasDesc *cds;
    const uint32_t *cells;
    const uint16_t *coarse;
    const Cand *cands;
    const Edge *ledges;
    const double2 *pspan;
    const uint32_t *pid;          // layered set: caller's id of set polygon g (else g itself)
};

__device__ __forceinline__ uint32_t caller_id(const SetArgs &S, int64_t g)
{
    return S.pid ? S.pid[g] : (uint32_t)g;
}

constexpr uint32_t NO_WORD = 0xffffffffu;

// The canvas word of every point of a table chunk, when one word holds for
// all of them: the chunk's exact box lies inside the canvas's half-open box
// and every coarse block its pixels can fall in is uniform with that word
// (0, or an interior label + 1; the pixel map is monotonic, so the box's
// corner pixels bound every point's pixel).  Else NO_WORD.  Called by the
// whole workgroup (it synchronises).
__device__ uint32_t chunk_word(const CanvasView &v, const double4 cb)
{
    if (!(v.bx0 <= cb.x && cb.z < v.bx1 && v.by0 <= cb.y && cb.w < v.by1)) return NO_WORD;
    auto col = [&](double x) { return min((int)__dmul_rn(__dsub_rn(x, v.X0), v.sx), v.W - 1) >> v.blog; };
    auto row = [&](double y) { return min((int)__dmul_rn(__dsub_rn(y, v.Y0), v.sy), v.H - 1) >> v.blog; };
    const int c0 = col(cb.x), c1 = col(cb.z), r0 = row(cb.y), r1 = row(cb.w);
    const int nbx = c1 - c0 + 1, nb = nbx * (r1 - r0 + 1);
    if (nb > BT_THREADS) return NO_WORD;
    auto word = [&](int bx, int by) -> uint32_t {
        const int i = by * v.Wc + bx;
        return v.cbyte ? (uint32_t)((const uint8_t *)v.coarse)[i] : (uint32_t)v.coarse[i];
    };
    const uint32_t w0 = word(c0, r0);
    const int t = (int)threadIdx.x;
    const int same = (t >= nb) || word(c0 + t % nbx, r0 + t / nbx) == w0;
    const uint32_t full = v.cbyte ? COARSE_BYTE_FULL : (uint32_t)COARSE_FULL;
    return (__syncthreads_and(same) && w0 != full) ? w0 : NO_WORD;
}

// Inclusive prefix sum over the wavefront (rocPRIM's cross-lane warp scan).
__device__ __forceinline__ uint32_t wave_incl_sum(uint32_t v)
{
    uint32_t r;
    typename rocprim::warp_scan<uint32_t, 64>::storage_type storage;
    rocprim::warp_scan<uint32_t, 64>().inclusive_scan(v, r, storage, rocprim::plus<uint32_t>());
    return r;
}

// ------------------------------------------------------------ wavefront tasks
//
// A table chunk is probed by wavefronts of their own: a task is BW_PTS words
// of 64 consecutive table points, one point per lane and word, and needs no
// barrier.  The table is in Z order, so a task's box is small: most of the
// (task, canvas) tests end at the box or at the canvas's coarse blocks under
// it.  Few points per lane keep the registers low enough for six wavefronts per
// SIMD, which is what hides the chain of dependent reads (descriptor, coarse
// word, canvas word, record, edges) that bounds a probe.
constexpr int BW_PTS = 4;                        // words of 64 points per task
constexpr int BW_TASKS = CHUNK / (64 * BW_PTS);  // tasks per chunk
constexpr int BW_WORDS = CHUNK / 64;             // result words per chunk

__device__ __forceinline__ double uniform_f64(double v)
{
    const long long b = __double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Exact box of a task's points (NaN: no point); (min x, min y, max x, max y),
// the same in every lane.  Without points it is inverted.
template <int PTS>
__device__ __forceinline__ double4 task_box(const double *xs, const double *ys)
{
    double x0 = INFINITY, x1 = -INFINITY, y0 = INFINITY, y1 = -INFINITY;
#pragma unroll
    for (int u = 0; u < PTS; ++u) {
        x0 = fmin(x0, xs[u]); x1 = fmax(x1, xs[u]);
        y0 = fmin(y0, ys[u]); y1 = fmax(y1, ys[u]);
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
        x0 = fmin(x0, __shfl_xor(x0, d, 64)); x1 = fmax(x1, __shfl_xor(x1, d, 64));
        y0 = fmin(y0, __shfl_xor(y0, d, 64)); y1 = fmax(y1, __shfl_xor(y1, d, 64));
    }
    return make_double4(uniform_f64(x0), uniform_f64(y0), uniform_f64(x1), uniform_f64(y1));
}

// The canvas word of every point of a task, when one word holds for all of
// them: 0 when the points' exact box misses the canvas's half-open box;
// otherwise the box lies inside it and every coarse block its pixels can fall
// in (at most 64 are looked at, one per lane) is uniform with that word (the
// pixel map is monotonic, so the box's corner pixels bound every point's
// pixel).  Else NO_WORD.  Called by the whole wavefront; the result is uniform.
__device__ __forceinline__ uint32_t task_word(const CanvasView &v, const double4 cb, int lane)
{
    if (!(cb.z >= v.bx0 && cb.x < v.bx1 && cb.w >= v.by0 && cb.y < v.by1)) return 0u;
    if (!(v.bx0 <= cb.x && cb.z < v.bx1 && v.by0 <= cb.y && cb.w < v.by1)) return NO_WORD;
    auto col = [&](double x) { return min((int)__dmul_rn(__dsub_rn(x, v.X0), v.sx), v.W - 1) >> v.blog; };
    auto row = [&](double y) { return min((int)__dmul_rn(__dsub_rn(y, v.Y0), v.sy), v.H - 1) >> v.blog; };
    const int c0 = col(cb.x), c1 = col(cb.z), r0 = row(cb.y), r1 = row(cb.w);
    const int nbx = c1 - c0 + 1, nb = nbx * (r1 - r0 + 1);
    if (nb > 64) return NO_WORD;
    const int t = lane < nb ? lane : 0;
    const int i = (r0 + t / nbx) * v.Wc + c0 + t % nbx;
    const uint32_t w = v.cbyte ? (uint32_t)((const uint8_t *)v.coarse)[i] : (uint32_t)v.coarse[i];
    const uint32_t w0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)w);
    const uint32_t full = v.cbyte ? COARSE_BYTE_FULL : (uint32_t)COARSE_FULL;
    return (__all(w == w0) && w0 != full) ? w0 : NO_WORD;
}

// ------------------------------------------------------------ batch select

// Probe pass: hits[(p - p0) * BW_WORDS + j] = the points 64 j + lane of pair
// p's chunk (bit = lane) that lie in its query's polygon, for the pairs p0 <=
// p < p1.  Bound by the latency of its gathers: 3.0 ms for 130,574 (chunk,
// query) pairs, 35 us for 805.  With 16 points per thread of a 256-thread
// workgroup (158 registers, 2.2 wavefronts per SIMD, two barriers per pair)
// it took 5.0 ms and 158 us.  BY_PAIR: a task is one pair's words instead of a
// chunk's, for few pairs (the launch over all chunks mostly finds them
// without any: 805 pairs of 12,208 chunks 34 us, 25 us by pair).
template <bool BY_PAIR>
__global__ __launch_bounds__(BT_THREADS) void k_batch_hits(SetArgs S, int64_t nfin, int64_t nchunk, const double *X,
                                                           const double *Y, const unsigned int *cbase,
                                                           const uint32_t *plist, const uint32_t *pq,
                                                           const uint32_t *pc, uint32_t p0, uint32_t p1,
                                                           unsigned long long *hits)
{
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t ntask = (BY_PAIR ? (int64_t)(p1 - p0) : nchunk) * BW_TASKS;
    for (int64_t task = (int64_t)blockIdx.x * (BT_THREADS / 64) + wv; task < ntask;
         task += (int64_t)gridDim.x * (BT_THREADS / 64)) {
        const int64_t c = BY_PAIR ? (int64_t)pc[p0 + task / BW_TASKS] : task / BW_TASKS;
        const int part = (int)(task % BW_TASKS);
        const uint32_t t0 = BY_PAIR ? 0u : cbase[c], t1 = BY_PAIR ? 1u : cbase[c + 1];
        if (t0 == t1) continue;
        double xs[BW_PTS], ys[BW_PTS];
        unsigned long long valid[BW_PTS];
#pragma unroll
        for (int u = 0; u < BW_PTS; ++u) {
            const int64_t i = c * CHUNK + part * (64 * BW_PTS) + 64 * u + lane;
            xs[u] = i < nfin ? X[i] : NAN;
            ys[u] = i < nfin ? Y[i] : NAN;
            valid[u] = __ballot(i < nfin);
        }
        const double4 cb = task_box<BW_PTS>(xs, ys);
        for (uint32_t t = t0; t < t1; ++t) {
            const uint32_t p = BY_PAIR ? p0 + (uint32_t)(task / BW_TASKS) : plist[t];
            if (p < p0 || p >= p1) continue;
            const CanvasDesc d = S.cds[pq[p]];
            const CanvasView v = set_view(d, S.cells, S.coarse, S.cands, S.ledges, S.pspan);
            unsigned long long m[BW_PTS];
            const uint32_t cw = task_word(v, cb, lane);
            if (cw != NO_WORD) {
#pragma unroll
                for (int u = 0; u < BW_PTS; ++u) m[u] = cw != 0u ? valid[u] : 0ull;
            } else {
                Look lk[BW_PTS];
                uint32_t ws[BW_PTS];
#pragma unroll
                for (int u = 0; u < BW_PTS; ++u) lk[u] = look_coarse(v, v.coarse, xs[u], ys[u]);
#pragma unroll
                for (int u = 0; u < BW_PTS; ++u) ws[u] = lk[u].full ? ((gu32p)v.cells)[lk[u].fidx] : lk[u].word;
#pragma unroll
                for (int u = 0; u < BW_PTS; ++u) {
                    bool in = ws[u] != 0u;
                    if (ws[u] & BFLAG) {
                        in = false;
                        uint32_t rec = ws[u] & ~BFLAG;
                        while (true) {
                            const Cand cd = v.cands[rec];
                            if (cand_inside(v, cd, xs[u], ys[u])) in = true;
                            if (cd.meta & CAND_LAST) break;
                            ++rec;
                        }
                    }
                    m[u] = __ballot(in);
                }
            }
            unsigned long long mine = m[0];
#pragma unroll
            for (int u = 1; u < BW_PTS; ++u) mine = lane == u ? m[u] : mine;
            if (lane < BW_PTS) hits[(size_t)(p - p0) * BW_WORDS + part * BW_PTS + lane] = mine;
        }
    }
}

// Ordering the ids of the hit words.  A bucket is a query and a window of 2^L
// consecutive ids; the buckets, query by query, are in output order.  A tile
// is up to TILE_PAIRS pairs of one query: its ids are put in window order in
// LDS and stored as one block, with the start of every window in it.  Bucket
// totals come from those starts, a scan of them gives every bucket its output
// range, and every bucket is ordered with a bitmap of its window in LDS,
// filled from the query's tiles, whose set bits, read in order, are its ids.
//
// An id costs one 4-byte gather, one coalesced store and load, one coalesced
// store of the result and four LDS operations: 5.7 ns per 1,000 ids (340M ids
// of 128 stars over 50M points: tiles 0.90 ms, buckets 1.05 ms), bound by
// instruction issue in the buckets and by the gathers in the tiles.  Keys
// written query by query, counted per bucket and scattered with 4-byte stores
// took 14 ns.
constexpr int TILE_PAIRS = 4;
constexpr int TILE_IDS = TILE_PAIRS * CHUNK;
constexpr int TILE_THREADS = 1024;
constexpr int TILE_BINS = 4096;                 // windows of a query (2^31 ids at most)
constexpr int SORT_LBITS = 19;                  // largest window: a 64 KB LDS bitmap, two workgroups per CU
constexpr int SORT_LMIN = 16;                   // smallest one taken to spread few ids over the chip

__global__ __launch_bounds__(TILE_THREADS, 8) void k_hit_tiles(int nq, const uint32_t *tfirst,
                                                            const unsigned long long *qbase, uint32_t p0,
                                                            const uint32_t *pc, const unsigned long long *hits,
                                                            const uint32_t *ids, int L, int nbins, uint32_t *keys,
                                                            uint16_t *starts)
{
    constexpr int PER = TILE_IDS / TILE_THREADS;   // words of a wavefront
    static_assert(PER * (TILE_THREADS / 64) == TILE_PAIRS * BW_WORDS, "a wavefront takes whole words of one pair");
    extern __shared__ uint32_t tl[];
    __shared__ uint32_t wsum[TILE_THREADS / 64];
    uint32_t *bins = tl, *sorted = tl + ((nbins + 127) & ~63);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t tile = blockIdx.x;
    // the tile's query: the last one that starts at or before it
    int lo = 0, hi = nq - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (tfirst[mid] - tfirst[0] <= tile) lo = mid; else hi = mid - 1;
    }
    constexpr int WPP = BW_WORDS / PER;            // wavefronts per pair
    const uint32_t p = (uint32_t)qbase[lo] + (tile - (tfirst[lo] - tfirst[0])) * TILE_PAIRS + (uint32_t)(wv / WPP);
    const bool any = p < (uint32_t)qbase[lo + 1];
    uint32_t v[PER], rb[PER], on = 0u;
    for (int b = tid; b < nbins; b += TILE_THREADS) bins[b] = 0u;
    const int j0 = (wv % WPP) * PER;
    const unsigned long long *h = hits + (size_t)((any ? p : p0) - p0) * BW_WORDS + j0;
    const uint32_t *id0 = ids + (int64_t)(any ? pc[p] : 0u) * CHUNK + 64 * j0;
    if (any)
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const unsigned long long w = h[k];
            const uint32_t half = lane < 32 ? (uint32_t)w : (uint32_t)(w >> 32);
            on |= ((half >> (lane & 31)) & 1u) << k;
        }
#pragma unroll
    for (int k = 0; k < PER; ++k) v[k] = (on >> k) & 1u ? id0[64 * k + lane] : 0u;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        // window and rank in it (below 2^14) in one word; a lane without a
        // hit counts in a bin of its own, past the windows
        const uint32_t bin = (on >> k) & 1u ? v[k] >> L : (uint32_t)(nbins + lane);
        rb[k] = (bin << 14) | (atomicAdd(&bins[bin], 1u) & 0x3fffu);
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) asm volatile("" : "+v"(rb[k]));   // one register each, not its parts
    __syncthreads();
    // the windows' starts: an exclusive scan of the counts, a few per thread
    const int per = (nbins + TILE_THREADS - 1) / TILE_THREADS, b0 = min(nbins, tid * per), b1 = min(nbins, b0 + per);
    uint32_t mine = 0u;
#pragma nounroll
    for (int b = b0; b < b1; ++b) mine += bins[b];
    const uint32_t inc = wave_incl_sum(mine);
    if (lane == 63) wsum[wv] = inc;
    __syncthreads();
    uint32_t at = inc - mine, total = 0u;
#pragma nounroll
    for (int w = 0; w < TILE_THREADS / 64; ++w) {
        const uint32_t n = wsum[w];
        if (w < wv) at += n;
        total += n;
    }
    uint16_t *st = starts + (size_t)tile * (nbins + 1);
#pragma nounroll
    for (int b = b0; b < b1; ++b) {
        const uint32_t n = bins[b];
        bins[b] = at;
        st[b] = (uint16_t)at;
        at += n;
    }
    if (tid == 0) st[nbins] = (uint16_t)total;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; ++k)
        if ((on >> k) & 1u) sorted[bins[rb[k] >> 14] + (rb[k] & 0x3fffu)] = v[k];
    __syncthreads();
    uint32_t *dst = keys + (size_t)tile * TILE_IDS;
    for (uint32_t i = tid; i < total; i += TILE_THREADS) dst[i] = sorted[i];
}

// Counts alone: tot[q] += the ids of pair p of query q, a wavefront per pair.
__global__ __launch_bounds__(256) void k_hit_count(uint32_t p0, uint32_t p1, uint32_t q0, const uint32_t *pq,
                                                   const unsigned long long *hits, unsigned long long *tot)
{
    static_assert(BW_WORDS == 64, "a word per lane");
    const int lane = threadIdx.x & 63;
    for (uint32_t p = p0 + ((blockIdx.x * 256 + threadIdx.x) >> 6); p < p1; p += gridDim.x * 4) {
        const uint32_t c = wave_incl_sum((uint32_t)__popcll(hits[(size_t)(p - p0) * BW_WORDS + lane]));
        if (lane == 63 && c != 0u) atomicAdd(&tot[pq[p] - q0], (unsigned long long)c);
    }
}

// Bucket totals: tot[q * nbins + b] = ids of query q in window b, summed over
// the query's tiles (64 windows by 16 slices of the tiles per workgroup).
__global__ __launch_bounds__(TILE_THREADS) void k_bucket_tot(int nq, const uint32_t *tfirst, const uint16_t *starts,
                                                             int nbins, unsigned long long *tot)
{
    constexpr int SL = TILE_THREADS / 64;
    __shared__ uint32_t s[SL][64];
    const int lane = threadIdx.x & 63, sl = threadIdx.x >> 6;
    const int b = blockIdx.x * 64 + lane;
    for (int q = blockIdx.y; q < nq; q += gridDim.y) {
        const uint32_t t0 = tfirst[q] - tfirst[0], t1 = tfirst[q + 1] - tfirst[0];
        uint32_t n = 0u;
        if (b < nbins) {
#pragma unroll 4
            for (uint32_t t = t0 + sl; t < t1; t += SL) {
                const uint16_t *st = starts + (size_t)t * (nbins + 1) + b;
                n += (uint32_t)st[1] - (uint32_t)st[0];
            }
        }
        s[sl][lane] = n;
        __syncthreads();
        if (sl == 0) {
#pragma unroll
            for (int k = 1; k < SL; ++k) n += s[k][lane];
            if (b < nbins) tot[(size_t)q * nbins + b] = n;
        }
        __syncthreads();
    }
}

// Buckets b < nb in ascending id order: bucket b's ids, its window's run in
// each of its query's tiles, become the ids (window << L | bit) of the set
// bits of its LDS bitmap, written to out[offs[b] ...] below limit.  The bitmap
// is read in blocks of 64 words, one word per lane of a wavefront: each lane
// walks its word's set bits and puts their ids at their ranks in a stage in
// LDS, which the wavefront then stores to consecutive positions, BM_STAGE ids
// at a time.  The phases of a bucket (clear, fill, count, store) wait on one
// another, so the window is half of what one workgroup's LDS would hold and
// two workgroups share a CU.
constexpr int BKT_THREADS = 1024;
constexpr int BM_WORDS_MAX = (1 << SORT_LBITS) >> 5;
constexpr int BM_BLOCKS_MAX = BM_WORDS_MAX / 64;
constexpr int BM_STAGE = 192;
constexpr int BM_FLY = 4;                       // tiles' runs in flight per wavefront, two loads each

__global__ __launch_bounds__(BKT_THREADS, 8) void k_bucket_bitmap(int64_t nb, const unsigned long long *offs,
                                                               const uint32_t *tfirst, const uint16_t *starts,
                                                               const uint32_t *keys, int L, int nbins, uint32_t *out,
                                                               int64_t limit)
{
    extern __shared__ uint32_t bm[];            // 2^L bits, whole blocks of 64 words
    __shared__ uint32_t btot[BM_BLOCKS_MAX];    // set bits per block, then the blocks' offsets
    __shared__ uint32_t wsum[BKT_THREADS / 64];
    __shared__ uint32_t stages[BKT_THREADS / 64][BM_STAGE];
    const int nw = ((1 << L) >> 5) > 0 ? (1 << L) >> 5 : 1;
    const int nbk = (nw + 63) / 64;
    const uint32_t lmask = (1u << L) - 1u;
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    constexpr int NWAVE = BKT_THREADS / 64;
    uint32_t *stage = stages[wv];
    auto mark = [&](uint32_t id) {
        const uint32_t lo = id & lmask;
        atomicOr(&bm[lo >> 5], 1u << (lo & 31));
    };
    for (int64_t b = blockIdx.x; b < nb; b += gridDim.x) {
        const unsigned long long s0 = offs[b];
        if (offs[b + 1] == s0 || (int64_t)s0 >= limit) continue;   // uniform over the workgroup
        const int q = (int)(b / nbins), win = (int)(b % nbins);
        for (int w = threadIdx.x; w < nbk * 64; w += BKT_THREADS) bm[w] = 0u;
        __syncthreads();
        // each wavefront takes every NWAVE-th tile; the runs of 64 of its
        // tiles are looked up at once, one per lane
        const uint32_t t0 = tfirst[q] - tfirst[0], t1 = tfirst[q + 1] - tfirst[0];
        for (uint32_t tb = t0 + wv; tb < t1; tb += 64 * NWAVE) {
            const uint32_t tl = tb + (uint32_t)lane * NWAVE;
            uint32_t rs = 0u, rn = 0u;
            if (tl < t1) {
                const uint16_t *st = starts + (size_t)tl * (nbins + 1) + win;
                rs = st[0];
                rn = (uint32_t)st[1] - rs;
            }
            const int nt = (int)min(64u, (t1 - tb + NWAVE - 1) / NWAVE);
            for (int k0 = 0; k0 < nt; k0 += BM_FLY) {
                uint32_t a[BM_FLY], c[BM_FLY], len[BM_FLY];
                const uint32_t *src[BM_FLY];
#pragma unroll
                for (int u = 0; u < BM_FLY; ++u) {
                    const int k = min(k0 + u, 63);
                    len[u] = k0 + u < nt ? (uint32_t)__builtin_amdgcn_readlane((int)rn, k) : 0u;
                    src[u] = keys + (size_t)(tb + (uint32_t)k * NWAVE) * TILE_IDS +
                             (uint32_t)__builtin_amdgcn_readlane((int)rs, k);
                    a[u] = (uint32_t)lane < len[u] ? src[u][lane] : 0u;
                    c[u] = (uint32_t)lane + 64 < len[u] ? src[u][lane + 64] : 0u;
                }
#pragma unroll
                for (int u = 0; u < BM_FLY; ++u) {
                    if ((uint32_t)lane < len[u]) mark(a[u]);
                    if ((uint32_t)lane + 64 < len[u]) mark(c[u]);
                    for (uint32_t i = (uint32_t)lane + 128; i < len[u]; i += 64) mark(src[u][i]);
                }
            }
        }
        __syncthreads();
        // set bits per block of 64 words
        for (int k = wv; k < nbk; k += NWAVE) {
            const uint32_t c = wave_incl_sum((uint32_t)__popc(bm[k * 64 + lane]));
            if (lane == 63) btot[k] = c;
        }
        __syncthreads();
        // exclusive scan of the block totals (nbk <= BKT_THREADS)
        {
            const uint32_t v = threadIdx.x < nbk ? btot[threadIdx.x] : 0u;
            uint32_t inc = v;
            for (int d = 1; d < 64; d <<= 1) {
                const uint32_t t = __shfl_up(inc, d, 64);
                if (lane >= d) inc += t;
            }
            if (lane == 63) wsum[wv] = inc;
            __syncthreads();
            uint32_t pre = 0;
            for (int w = 0; w < wv; ++w) pre += wsum[w];
            if (threadIdx.x < nbk) btot[threadIdx.x] = pre + inc - v;
        }
        __syncthreads();
        const uint32_t hi = (uint32_t)win << L;
        for (int k = wv; k < nbk; k += NWAVE) {
            uint32_t word = bm[k * 64 + lane];
            const uint32_t c = (uint32_t)__popc(word);
            const uint32_t incl = wave_incl_sum(c);
            const uint32_t T = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
            const int64_t base = (int64_t)s0 + btot[k];
            const uint32_t first = hi | ((uint32_t)(k * 64 + lane) << 5);
            uint32_t at = incl - c;   // rank of this lane's next set bit in the block
            for (uint32_t r0 = 0; r0 < T; r0 += BM_STAGE) {
                const uint32_t m = min(T - r0, (uint32_t)BM_STAGE);
                while (word != 0u && at < r0 + m) {
                    stage[at - r0] = first | (uint32_t)(__ffs(word) - 1);
                    word &= word - 1u;
                    ++at;
                }
                __builtin_amdgcn_wave_barrier();
                for (uint32_t o = (uint32_t)lane; o < m; o += 64)
                    if (base + r0 + o < limit) out[base + r0 + o] = stage[o];
                __builtin_amdgcn_wave_barrier();
            }
        }
        __syncthreads();
    }
}

// Query starts from the bucket offsets, into the host's words: hoff[q] =
// offs[q * nbins], hoff[nq] = the total.
__global__ void k_query_off(int nq, int nbins, const unsigned long long *offs, unsigned long long *hoff)
{
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q <= nq) __hip_atomic_store(&hoff[q], offs[(size_t)q * nbins], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __threadfence_system();
}

// Both at once for few buckets (one workgroup): offs = exclusive scan of tot.
constexpr int64_t BUCKET_SCAN_MAX = 32768;   // 32 per thread; a library scan takes three launches

__global__ __launch_bounds__(PS_THREADS) void k_bucket_scan(int nq, int nbins, const unsigned long long *tot,
                                                            unsigned long long *offs, unsigned long long *hoff)
{
    __shared__ unsigned long long ws[PS_THREADS / 64];
    scan_block<unsigned long long>((int64_t)nq * nbins, ws, [&](int64_t i) { return tot[i]; },
                                   [&](int64_t i, unsigned long long at) { offs[i] = at; });
    for (int q = threadIdx.x; q <= nq; q += PS_THREADS)
        __hip_atomic_store(&hoff[q], offs[(size_t)q * nbins], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __threadfence_system();
}

// ------------------------------------------------------------ batch join pairs

// Pairs (point id, polygon id) of the table with a canvas set, ascending.
// The count pass sizes every point's list (pcnt by point id), a scan of the
// counts in id order gives every list its place in the output, and the write
// pass finds the matches again and writes each list, ordered, at its place:
// no sort of the pairs.  The lists are gathered in LDS first, so that a list
// goes out as one run of stores instead of one scattered store per pair.
//
// With both passes over 16 points per thread (193 and 232 registers, two
// wavefronts per SIMD, the write pass probing twice) and a library radix sort
// of 64-bit keys, 181M pairs of 20M points with 260 polygons in 43 layers took
// 2.8 + 6.2 + 5.5 + 0.5 ms.

constexpr int PW_BYTES = 4096;                          // LDS pool of a wavefront of the write pass
// Longer lists go through a bitmap.  200,000 points in n polygons each, layered
// (ids in any order), by insertion and by bitmap: n = 40 425 and 516 us, 48 484
// and 539, 64 1,655 and 587, 100 1,821 and 779.
constexpr uint32_t PW_LONG = 48;
constexpr int PL_WORDS = 2048;                          // its words of 32 ids per wavefront
constexpr size_t PAIR_HITS_MAX = (size_t)16 << 30;
// Sorted keys while the (chunk, query) overlaps have at most PK_OVER times the
// table's points, in a table of PK_LARGE points or more, and a PK_PART of them
// in a smaller one.  Lists and places of all points, and keys: one polygon, 30M
// points, 3,570 pairs 460 and 104 us, 11.3M pairs 1,206 and 586; 18M points,
// 0.36M to 6.8M pairs 336 to 723 and 218 to 427; 8M points, 0.37M pairs 216 and
// 212; 5M points, overlaps of a 20th of them 166 and 152, a tenth 172 and 187,
// a half 239 and 298 (a library sort of some 100,000 keys takes many launches).
// Every point in one polygon (64 cells), 30M points 2.4 and 1.3 ms.  Where points
// meet several queries lists are better: 30M points, 78M pairs 3.2 and 4.8 ms.
constexpr int64_t PK_LARGE = (int64_t)1 << 23, PK_PART = 16, PK_OVER = 2;

// Count pass over chunks [c0, c1).  hits, when given, keeps the points that
// matched: hits[(t - cbase[c0]) * BW_WORDS + j] for entry t of the chunks'
// query lists and word j.  *some_long is set by a list longer than PW_LONG.
__global__ __launch_bounds__(BT_THREADS) void k_batch_pcount(SetArgs S, int64_t nfin, int64_t c0, int64_t c1,
                                                             const double *X, const double *Y, const uint32_t *ids,
                                                             const unsigned int *cbase, const uint32_t *plist,
                                                             const uint32_t *pq, uint32_t *pcnt,
                                                             unsigned long long *hits, uint32_t *some_long)
{
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t tb = cbase[c0];
    for (int64_t task = c0 * BW_TASKS + (int64_t)blockIdx.x * (BT_THREADS / 64) + wv; task < c1 * BW_TASKS;
         task += (int64_t)gridDim.x * (BT_THREADS / 64)) {
        const int64_t c = task / BW_TASKS;
        const uint32_t t0 = cbase[c], t1 = cbase[c + 1];
        if (t0 == t1) continue;
        const int64_t i0 = c * CHUNK + (task % BW_TASKS) * (64 * BW_PTS) + lane;
        double xs[BW_PTS], ys[BW_PTS];
        unsigned long long valid[BW_PTS];
        uint32_t cnt[BW_PTS];
#pragma unroll
        for (int u = 0; u < BW_PTS; ++u) {
            const int64_t i = i0 + 64 * u;
            xs[u] = i < nfin ? X[i] : NAN;
            ys[u] = i < nfin ? Y[i] : NAN;
            valid[u] = __ballot(i < nfin);
            cnt[u] = 0u;
        }
        const double4 cb = task_box<BW_PTS>(xs, ys);
        for (uint32_t t = t0; t < t1; ++t) {
            const CanvasDesc d = S.cds[pq[plist[t]]];
            const CanvasView v = set_view(d, S.cells, S.coarse, S.cands, S.ledges, S.pspan);
            unsigned long long m[BW_PTS];   // the points of word u with a match
            const uint32_t cw = task_word(v, cb, lane);
            if (cw != NO_WORD) {
#pragma unroll
                for (int u = 0; u < BW_PTS; ++u) {
                    m[u] = cw != 0u ? valid[u] : 0ull;
                    cnt[u] += (uint32_t)((m[u] >> lane) & 1ull);
                }
            } else {
                Look lk[BW_PTS];
                uint32_t ws[BW_PTS];
#pragma unroll
                for (int u = 0; u < BW_PTS; ++u) lk[u] = look_coarse(v, v.coarse, xs[u], ys[u]);
#pragma unroll
                for (int u = 0; u < BW_PTS; ++u) ws[u] = lk[u].full ? ((gu32p)v.cells)[lk[u].fidx] : lk[u].word;
#pragma unroll
                for (int u = 0; u < BW_PTS; ++u) {
                    uint32_t got = ws[u] != 0u ? 1u : 0u;
                    if (ws[u] & BFLAG) {
                        got = 0u;
                        uint32_t rec = ws[u] & ~BFLAG;
                        while (true) {
                            const Cand cd = v.cands[rec];
                            got += cand_inside(v, cd, xs[u], ys[u]) ? 1u : 0u;
                            if (cd.meta & CAND_LAST) break;
                            ++rec;
                        }
                    }
                    cnt[u] += got;
                    m[u] = __ballot(got != 0u);
                }
            }
            unsigned long long mine = m[0];
#pragma unroll
            for (int u = 1; u < BW_PTS; ++u) mine = lane == u ? m[u] : mine;
            if (hits && lane < BW_PTS) hits[(size_t)(t - tb) * BW_WORDS + (task % BW_TASKS) * BW_PTS + lane] = mine;
        }
#pragma unroll
        for (int u = 0; u < BW_PTS; ++u) {
            if (cnt[u]) pcnt[ids[i0 + 64 * u]] = cnt[u];
            if (cnt[u] > PW_LONG) *some_long = 1u;
        }
    }
}

// fn(polygon id) for every match of point (x, y) with the canvas d that is
// known to have one: only the record of a boundary pixel that has no other is
// then the match without a test.
template <typename Fn>
__device__ __forceinline__ void point_matches(const SetArgs &S, const CanvasDesc &d, double x, double y, Fn fn)
{
    const CanvasView v = set_view(d, S.cells, S.coarse, S.cands, S.ledges, S.pspan);
    const uint32_t w = lookup(v, v.coarse, x, y);
    uint32_t rec = w & ~BFLAG, label = w - 1u;
    bool more = (w & BFLAG) != 0, first = true, in = true;
    do {
        if (more) {
            const Cand cd = v.cands[rec++];
            label = cd.poly;
            more = !(cd.meta & CAND_LAST);
            in = (first && !more) || cand_inside(v, cd, x, y);
            first = false;
        }
        if (in) fn(caller_id(S, d.poly_base + label));
    } while (more);
}

// Write pass over chunks [c0, c1), from the count pass's hit words: a
// wavefront takes 64 table points, one per lane, whose lists are gathered in
// its pool in LDS in ascending polygon id (an insertion per match), as many
// points at a time as the pool holds, and stored.  Only the points that
// matched look their canvas word up again.  Positions at or beyond cap are not
// written.
template <typename T>
__global__ __launch_bounds__(BT_THREADS) void k_batch_pwrite(SetArgs S, int64_t nfin, int64_t c0, int64_t c1,
                                                             const double *X, const double *Y, const uint32_t *ids,
                                                             const unsigned int *cbase, const uint32_t *plist,
                                                             const uint32_t *pq, const unsigned long long *hits,
                                                             const unsigned long long *offs, uint32_t *out_poly, int64_t cap)
{
    constexpr uint32_t POOL = PW_BYTES / sizeof(T);
    static_assert(PW_LONG <= POOL, "the pool holds a list");
    __shared__ T pools[BT_THREADS / 64][POOL];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    T *pool = pools[wv];
    const uint32_t tb = cbase[c0];
    for (int64_t word = c0 * BW_WORDS + (int64_t)blockIdx.x * (BT_THREADS / 64) + wv; word < c1 * BW_WORDS;
         word += (int64_t)gridDim.x * (BT_THREADS / 64)) {
        const int64_t c = word / BW_WORDS;
        const uint32_t t0 = cbase[c], t1 = cbase[c + 1];
        if (t0 == t1) continue;
        const int64_t i = word * 64 + lane;
        const bool valid = i < nfin;
        const double x = valid ? X[i] : NAN, y = valid ? Y[i] : NAN;
        int64_t o = 0;
        uint32_t n = 0u;
        if (valid) {
            const uint32_t id = ids[i];
            o = (int64_t)offs[id];
            n = o < cap ? (uint32_t)(offs[id + 1] - (unsigned long long)o) : 0u;
        }
        const uint32_t np = n > PW_LONG ? 0u : n;
        const uint32_t excl = wave_incl_sum(np) - np;
        unsigned long long todo = __ballot(np != 0u);
        while (todo) {
            const uint32_t base = (uint32_t)__builtin_amdgcn_readlane((int)excl, __ffsll((long long)todo) - 1);
            const bool now = ((todo >> lane) & 1ull) && excl + np - base <= POOL;
            T *list = pool + (now ? excl - base : 0u);
            uint32_t j = 0u;
            const unsigned long long of = __ballot(now);
            for (uint32_t t = t0; t < t1; ++t) {
                const unsigned long long m = hits[(size_t)(t - tb) * BW_WORDS + word % BW_WORDS] & of;
                if (m == 0ull) continue;
                const CanvasDesc &d = S.cds[pq[plist[t]]];
                if (!((m >> lane) & 1ull)) continue;
                point_matches(S, d, x, y, [&](uint32_t id) {
                    if (j >= np) return;
                    uint32_t at = j++;
                    while (at > 0u && (uint32_t)list[at - 1] > id) {
                        list[at] = list[at - 1];
                        --at;
                    }
                    list[at] = (T)id;
                });
            }
            if (now)
                for (uint32_t k = 0; k < np && o + k < cap; ++k) out_poly[o + k] = (uint32_t)list[k];
            todo &= ~of;
        }
    }
}

// The lists longer than PW_LONG (ends at once when there is none): a wavefront
// takes one point at a time, its lanes the canvases of the point's chunk, and
// marks the matches in a bitmap of ids in LDS, whose set bits, read in order,
// are the list, a window of ids after the other.  Linear in the list, where an
// insertion is quadratic: 600 polygons over each of 16,384 points, the call 1.9
// ms, by insertion 210.  Bound by the latency of the matches' lookups.
__global__ __launch_bounds__(BT_THREADS) void k_batch_plong(SetArgs S, int64_t nfin, int64_t c0, int64_t c1,
                                                            const double *X, const double *Y, const uint32_t *ids,
                                                            const unsigned int *cbase, const uint32_t *plist,
                                                            const uint32_t *pq, const unsigned long long *hits,
                                                            const unsigned long long *offs, const uint32_t *some_long,
                                                            uint32_t npoly, uint32_t *out_poly, int64_t cap)
{
    if (*some_long == 0u) return;
    __shared__ uint32_t maps[BT_THREADS / 64][PL_WORDS];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    uint32_t *map = maps[wv];
    auto sync = [] {   // order this wavefront's LDS accesses
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    const uint32_t tb = cbase[c0];
    for (int64_t word = c0 * BW_WORDS + (int64_t)blockIdx.x * (BT_THREADS / 64) + wv; word < c1 * BW_WORDS;
         word += (int64_t)gridDim.x * (BT_THREADS / 64)) {
        const int64_t c = word / BW_WORDS;
        const uint32_t t0 = cbase[c], t1 = cbase[c + 1];
        if (t0 == t1) continue;
        const int64_t i = word * 64 + lane;
        int64_t o = 0;
        uint32_t n = 0u;
        if (i < nfin) {
            const uint32_t id = ids[i];
            o = (int64_t)offs[id];
            n = o < cap ? (uint32_t)(offs[id + 1] - (unsigned long long)o) : 0u;
        }
        for (unsigned long long todo = __ballot(n > PW_LONG); todo; todo &= todo - 1) {
            const int b = __ffsll((long long)todo) - 1;
            const double x = X[word * 64 + b], y = Y[word * 64 + b];
            int64_t pos = __shfl(o, b, 64);
            uint32_t w0 = 0u;   // first id of the window, a multiple of 32
            while (w0 < npoly && pos < cap) {
                const uint32_t left = (npoly - w0 + 31u) / 32u;
                const int nw = (int)(left < (uint32_t)PL_WORDS ? left : (uint32_t)PL_WORDS);
                for (int k = lane; k < (nw + 63) / 64 * 64; k += 64) map[k] = 0u;
                sync();
                uint32_t next = npoly;   // the smallest id past the window
                for (uint32_t t = t0 + lane; t < t1; t += 64) {
                    if (!((hits[(size_t)(t - tb) * BW_WORDS + word % BW_WORDS] >> b) & 1ull)) continue;
                    point_matches(S, S.cds[pq[plist[t]]], x, y, [&](uint32_t id) {
                        if (id < w0) return;
                        const uint32_t k = (id - w0) / 32u;
                        if (k < (uint32_t)nw) atomicOr(&map[k], 1u << (id & 31u));
                        else next = min(next, id);
                    });
                }
                sync();
                for (int k0 = 0; k0 < nw; k0 += 64) {
                    uint32_t m = map[k0 + lane];
                    const uint32_t cnt = (uint32_t)__popc(m), incl = wave_incl_sum(cnt);
                    int64_t p = pos + (incl - cnt);
                    const uint32_t first = w0 + 32u * (uint32_t)(k0 + lane);
                    for (; m != 0u; m &= m - 1u, ++p)
                        if (p < cap) out_poly[p] = first + (uint32_t)(__ffs((int)m) - 1);
                    pos += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
                }
                sync();
#pragma unroll
                for (int d = 32; d > 0; d >>= 1) next = min(next, (uint32_t)__shfl_xor((int)next, d, 64));
                w0 = next < npoly ? next & ~31u : npoly;
            }
        }
    }
}

// The point ids of the lists: out_pt[offs[id] .. offs[id + 1]) = id, 64 ids
// per wavefront, whose output is one range (positions below cap).
__global__ __launch_bounds__(256) void k_pair_points(int64_t n, const unsigned long long *offs, uint32_t *out_pt,
                                                     int64_t cap)
{
    const int lane = threadIdx.x & 63;
    const int64_t nw = ((int64_t)gridDim.x * blockDim.x) >> 6;
    for (int64_t w = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6; w * 64 < n; w += nw) {
        const int64_t id = w * 64 + lane;
        const unsigned long long b = offs[w * 64];
        if ((int64_t)b >= cap) return;
        const unsigned long long e = offs[min(n, id + 1)];
        const unsigned long long end = offs[min(n, w * 64 + 64)];
        const uint32_t rel = (uint32_t)min<unsigned long long>(e - b, 0xffffffffull);   // end of this id's list
        if (end - b < 0xffffffffull) {
            const uint32_t T = (uint32_t)(end - b);
            for (uint32_t t = (uint32_t)lane; t - lane < T; t += 64) {
                int o = 0;   // the first lane whose list ends after t
#pragma unroll
                for (int st = 32; st > 0; st >>= 1)
                    if (__shfl(rel, o + st - 1, 64) <= t) o += st;
                if (t < T && (int64_t)(b + t) < cap) out_pt[b + t] = (uint32_t)(w * 64 + o);
            }
        } else {
            for (unsigned long long k = id ? offs[min(n, id)] : 0ull; k < e && (int64_t)k < cap; ++k) out_pt[k] = (uint32_t)id;
        }
    }
}

// The pairs of few (chunk, query) pairs as 64-bit keys (id << pbits | polygon
// id), in any order, to be sorted: for a table that is large beside them, the
// counts and places of all its points cost more.  A workgroup takes a pair, its
// wavefronts the pair's tasks as in k_batch_hits, and reserves its keys once
// (11.3M pairs of 30M points, 3,094 overlaps: 134 us; with an atomic per
// wavefront 582, bound by that address).  *cursor counts all of them; keys at
// or beyond room are not written.
constexpr int PK_THREADS = 64 * BW_TASKS;

__global__ __launch_bounds__(PK_THREADS) void k_batch_pkeys(SetArgs S, int64_t nfin, const double *X, const double *Y,
                                                            const uint32_t *ids, const uint32_t *pq, const uint32_t *pc,
                                                            uint32_t np, int pbits, unsigned long long *cursor,
                                                            unsigned long long *keys, unsigned long long room)
{
    __shared__ uint32_t wsum[BW_TASKS];
    __shared__ unsigned long long s_at;
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    for (uint32_t p = blockIdx.x; p < np; p += gridDim.x) {
        const int64_t i0 = (int64_t)pc[p] * CHUNK + wv * (64 * BW_PTS) + lane;
        double xs[BW_PTS], ys[BW_PTS];
#pragma unroll
        for (int u = 0; u < BW_PTS; ++u) {
            xs[u] = i0 + 64 * u < nfin ? X[i0 + 64 * u] : NAN;
            ys[u] = i0 + 64 * u < nfin ? Y[i0 + 64 * u] : NAN;
        }
        const CanvasDesc d = S.cds[pq[p]];
        const CanvasView v = set_view(d, S.cells, S.coarse, S.cands, S.ledges, S.pspan);
        const uint32_t cw = task_word(v, task_box<BW_PTS>(xs, ys), lane);
        uint32_t ws[BW_PTS];
        if (cw != NO_WORD) {
#pragma unroll
            for (int u = 0; u < BW_PTS; ++u) ws[u] = i0 + 64 * u < nfin ? cw : 0u;
        } else {
            Look lk[BW_PTS];
#pragma unroll
            for (int u = 0; u < BW_PTS; ++u) lk[u] = look_coarse(v, v.coarse, xs[u], ys[u]);
#pragma unroll
            for (int u = 0; u < BW_PTS; ++u) ws[u] = lk[u].full ? ((gu32p)v.cells)[lk[u].fidx] : lk[u].word;
        }
        auto records = [&](int u, auto fn) {
            for (uint32_t rec = ws[u] & ~BFLAG;; ++rec) {
                const Cand cd = v.cands[rec];
                if (cand_inside(v, cd, xs[u], ys[u])) fn(cd.poly);
                if (cd.meta & CAND_LAST) break;
            }
        };
        // a boundary point in one polygon or none gets that word; in several it
        // keeps its own and is tested again
        uint32_t mine = 0u;
#pragma unroll
        for (int u = 0; u < BW_PTS; ++u) {
            uint32_t got = ws[u] != 0u ? 1u : 0u;
            if (ws[u] & BFLAG) {
                uint32_t one = 0u;
                got = 0u;
                records(u, [&](uint32_t label) { ++got; one = label + 1u; });
                if (got <= 1u) ws[u] = one;
            }
            mine += got;
        }
        const uint32_t incl = wave_incl_sum(mine);
        if (lane == 63) wsum[wv] = incl;
        __syncthreads();
        uint32_t pre = 0u, total = 0u;
#pragma unroll
        for (int w = 0; w < BW_TASKS; ++w) {
            pre += w < wv ? wsum[w] : 0u;
            total += wsum[w];
        }
        if (threadIdx.x == 0) s_at = total != 0u ? atomicAdd(cursor, (unsigned long long)total) : 0ull;
        __syncthreads();
        unsigned long long at = s_at + pre + (incl - mine);
        auto put = [&](int u, uint32_t label) {
            if (at < room) keys[at] = ((unsigned long long)ids[i0 + 64 * u] << pbits) | caller_id(S, d.poly_base + label);
            ++at;
        };
        if (mine != 0u && keys != nullptr)
#pragma unroll
            for (int u = 0; u < BW_PTS; ++u) {
                if (ws[u] & BFLAG) records(u, [&](uint32_t label) { put(u, label); });
                else if (ws[u] != 0u) put(u, ws[u] - 1u);
            }
    }
}

__global__ void k_split_keys(int64_t n, const unsigned long long *keys, int pbits, uint32_t *pt, uint32_t *pg)
{
    const unsigned long long m = (1ull << pbits) - 1ull;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        pt[i] = (uint32_t)(keys[i] >> pbits);
        pg[i] = (uint32_t)(keys[i] & m);
    }
}

// ------------------------------------------------------------ batch join-count

constexpr int HSLOTS = 512;   // LDS hash slots per workgroup

// Whole-batch join-count in one launch, with no pair list: every workgroup
// takes table chunks (grid-stride), lists in LDS the canvases whose box meets
// the chunk's box (from qbox, a window of QL_MAX canvases at a time) and
// probes its points against them, counting per polygon in an LDS hash
// flushed with atomics per chunk.  Nothing is read back on the host between
// launches, so the call's
// launches are captured into a graph and replayed batch after batch, each
// replay reading the canvas set's descriptors as rebuilt for that batch.
constexpr int QL_MAX = 1024;
constexpr int64_t HIST_MAX_BATCH = 8192;   // polygons the count probe histograms in LDS

// Per-canvas boxes for the direct probe; a canvas with skip[q] set (counted
// by another launch) gets an empty box.
__global__ void k_qbox(int nq, const CanvasDesc *cds, const uint8_t *skip, double4 *qbox)
{
    for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < nq; q += gridDim.x * blockDim.x) {
        const CanvasDesc d = cds[q];
        qbox[q] = (d.empty || (skip && skip[q])) ? make_double4(INFINITY, INFINITY, -INFINITY, -INFINITY)
                                                 : make_double4(d.bx0, d.by0, d.bx1, d.by1);
    }
}

__global__ __launch_bounds__(BT_THREADS) void k_batch_count_direct(SetArgs S, int nq, int64_t nfin, int64_t nchunk,
                                                                   const double *X, const double *Y,
                                                                   const double4 *chunk_bb, const double4 *qbox,
                                                                   unsigned long long *counts)
{
    __shared__ unsigned long long hkey[HSLOTS];   // polygon id + 1 (0: empty)
    __shared__ uint32_t hval[HSLOTS];
    __shared__ uint32_t qlist[QL_MAX];
    __shared__ uint32_t s_nq;
    for (int64_t c = blockIdx.x; c < nchunk; c += gridDim.x) {
        const int64_t b = c * CHUNK;
        const double4 cb = chunk_bb[c];
        double xs[BT_PER], ys[BT_PER];
#pragma unroll
        for (int u = 0; u < BT_PER; ++u) {
            const int64_t i = b + (int64_t)u * BT_THREADS + threadIdx.x;
            xs[u] = i < nfin ? X[i] : NAN;
            ys[u] = i < nfin ? Y[i] : NAN;
        }
        for (int s = threadIdx.x; s < HSLOTS; s += BT_THREADS) { hkey[s] = 0ull; hval[s] = 0u; }
        for (int q0 = 0; q0 < nq; q0 += QL_MAX) {
            if (threadIdx.x == 0) s_nq = 0u;
            __syncthreads();
            for (int q = q0 + threadIdx.x; q < min(nq, q0 + QL_MAX); q += BT_THREADS) {
                const double4 qb = qbox[q];
                // the chunk's closed point box meets the canvas's half-open box
                if (cb.z >= qb.x && cb.x < qb.z && cb.w >= qb.y && cb.y < qb.w) qlist[atomicAdd(&s_nq, 1u)] = (uint32_t)q;
            }
            __syncthreads();
            const uint32_t nl = s_nq;
            for (uint32_t t = 0; t < nl; ++t) {
                const CanvasDesc d = S.cds[qlist[t]];
                const CanvasView v = set_view(d, S.cells, S.coarse, S.cands, S.ledges, S.pspan);
                auto add_n = [&](uint32_t label, uint32_t k) {
                    const unsigned long long key = (unsigned long long)caller_id(S, d.poly_base + label) + 1ull;
                    uint32_t h = (uint32_t)(key * 0x9E3779B97F4A7C15ull >> 55) & (HSLOTS - 1);
                    for (int probe = 0; probe < 8; ++probe, h = (h + 1) & (HSLOTS - 1)) {
                        unsigned long long cur = hkey[h];
                        if (cur == 0ull) {
                            cur = atomicCAS(&hkey[h], 0ull, key);
                            if (cur == 0ull) cur = key;
                        }
                        if (cur == key) { atomicAdd(&hval[h], k); return; }
                    }
                    atomicAdd(&counts[key - 1ull], (unsigned long long)k);
                };
                auto add = [&](uint32_t label) { add_n(label, 1u); };
                const uint32_t cw = chunk_word(v, cb);
                if (cw != NO_WORD) {
                    // one word for the whole chunk: its points all count for one polygon, or none
                    if (cw != 0u && threadIdx.x == 0) add_n(cw - 1u, (uint32_t)min<int64_t>(CHUNK, nfin - b));
                    continue;
                }
#pragma unroll
                for (int u = 0; u < BT_PER; ++u) {
                    const uint32_t w = lookup(v, v.coarse, xs[u], ys[u]);
                    if (w == 0u) continue;
                    if (!(w & BFLAG)) { add(w - 1u); continue; }
                    uint32_t rec = w & ~BFLAG;
                    while (true) {
                        const Cand cd = v.cands[rec];
                        if (cand_inside(v, cd, xs[u], ys[u])) add(cd.poly);
                        if (cd.meta & CAND_LAST) break;
                        ++rec;
                    }
                }
            }
            __syncthreads();
        }
        for (int s = threadIdx.x; s < HSLOTS; s += BT_THREADS)
            if (hkey[s]) atomicAdd(&counts[hkey[s] - 1ull], (unsigned long long)hval[s]);
        __syncthreads();
    }
}

__global__ void k_zero64(int64_t n, unsigned long long *p)
{
    const int64_t nth = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += nth) p[i] = 0ull;
}

__global__ void k_zero32(int64_t n, unsigned int *p)
{
    const int64_t nth = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += nth) p[i] = 0u;
}

static int num_cus_of(int device)
{
    int v = 0;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess || v <= 0) v = 256;
    return v;
}

// Counts widened for a scan that accumulates in 64 bits.
struct Widen {
    __host__ __device__ unsigned long long operator()(uint32_t v) const { return v; }
};

// Batch scratch: pairs in query-major order, their chunk-major lists.
struct Pairs {
    int64_t np = 0;
    uint32_t *pq = nullptr, *pc = nullptr, *plist = nullptr;
    unsigned int *cbase = nullptr;
    unsigned long long *qbase = nullptr;
    uint32_t *tfirst = nullptr;    // first tile of every query (tiles of TILE_PAIRS pairs)
    std::vector<int64_t> qfirst;   // host: first pair of every query, then the total
};

static int make_pairs(spade_ctx *ctx, const spade_canvas *set, const spade_table *t, Pairs &P)
{
    hipStream_t st = ctx->stream;
    const int nq = set->nc;
    const int64_t nchunk = t->nchunk;
    DevBuf &bq = ctx->scratch[S_KEYS];
    // 8-byte words: qn [nq] | qbase [nq + 1]; 4-byte: cn [nchunk] | cbase [nchunk + 1] | tfirst [nq + 1]
    const int64_t words = 2 * (int64_t)nq + 1;
    if (ensure(ctx, bq, 8 * (size_t)words + 4 * (size_t)(2 * nchunk + 1 + nq + 1))) return SPADE_E_NOMEM;
    unsigned long long *qn = (unsigned long long *)bq.p, *qbase = qn + nq;
    unsigned int *cn = (unsigned int *)(qn + words), *cbase = cn + nchunk;
    P.tfirst = cbase + nchunk + 1;
    unsigned long long *h = (unsigned long long *)ensure_pinned(ctx, 8 * (size_t)(nq + 1));
    if (!h) return set_error(ctx, SPADE_E_NOMEM, "pinned staging allocation failed");
    // (the counters, and the words between them)
    hipLaunchKernelGGL(k_zero32, dim3(grid_of(2 * words + nchunk, 4096)), dim3(256), 0, st, 2 * words + nchunk,
                       (unsigned int *)bq.p);
    SPADE_HIP(ctx, hipGetLastError());
    const CanvasDesc *cds = (const CanvasDesc *)set->dcds.p;
    const double4 *bb = (const double4 *)t->chunk_bb.p;
    const dim3 g((unsigned)std::max<int64_t>(1, (nchunk + 255) / 256), (unsigned)std::min((nq + PAIR_Q - 1) / PAIR_Q, 32768));
    if (nchunk > 0)
        hipLaunchKernelGGL(k_pairs<false>, g, dim3(256), 0, st, nq, nchunk, bb, cds, qn, nullptr, cn, nullptr, nullptr,
                           nullptr, nullptr);
    hipLaunchKernelGGL(k_pair_scan, dim3(2), dim3(PS_THREADS), 0, st, nq, nchunk, qn, qbase, cn, cbase, TILE_PAIRS, P.tfirst,
                       h);
    SPADE_HIP(ctx, hipGetLastError());
    SPADE_HIP(ctx, hipStreamSynchronize(st));
    P.qfirst.assign(h, h + nq + 1);
    const int64_t np = P.qfirst[(size_t)nq];
    if (np >= (int64_t)INT32_MAX) return set_error(ctx, SPADE_E_UNSUPPORTED, "too many (chunk, query) pairs in one batch");
    DevBuf &bp = ctx->scratch[S_VALS];
    if (ensure(ctx, bp, sizeof(uint32_t) * 3 * (size_t)std::max<int64_t>(np, 1))) return SPADE_E_NOMEM;
    P.np = np;
    ctx->batch_overlaps = np;
    P.pq = (uint32_t *)bp.p;
    P.pc = P.pq + std::max<int64_t>(np, 1);
    P.plist = P.pc + std::max<int64_t>(np, 1);
    P.cbase = cbase;
    P.qbase = qbase;
    if (np > 0) {
        hipLaunchKernelGGL(k_pairs<true>, g, dim3(256), 0, st, nq, nchunk, bb, cds, qn, (const unsigned long long *)qbase, cn,
                           (const unsigned int *)cbase, P.pq, P.pc, P.plist);
        SPADE_HIP(ctx, hipGetLastError());
    }
    return SPADE_OK;
}

static SetArgs set_args(const spade_canvas *set)
{
    SetArgs S;
    S.cds = (const CanvasDesc *)set->dcds.p;
    S.cells = (const uint32_t *)set->cells.p;
    S.coarse = (const uint16_t *)set->coarse.p;
    S.cands = (const Cand *)set->cands.p;
    S.ledges = (const Edge *)set->ledges.p;
    S.pspan = (const double2 *)set->pspan.p;
    S.pid = set->layered ? (const uint32_t *)set->pid.p : nullptr;
    return S;
}

}  // namespace spade

using namespace spade;

extern "C" {

int spade_ctx_set_pixels_per_vertex(spade_ctx *ctx, double ppv)
{
    if (!ctx) return SPADE_E_INVALID;
    SPADE_CTX_LOCK(ctx);
    if (!(ppv >= 1.0 && ppv <= 1e7)) return set_error(ctx, SPADE_E_INVALID, "pixels per vertex must be in [1, 1e7]");
    ctx->ppv = ppv;
    return SPADE_OK;
}

int spade_table_create(spade_ctx *ctx, const spade_points *pts, spade_table **out)
{
    if (!ctx) return SPADE_E_INVALID;
    SPADE_CTX_LOCK(ctx);
    if (!ctx || !out) return SPADE_E_INVALID;
    *out = nullptr;
    ctx->err.clear();
    if (hipSetDevice(ctx->device) != hipSuccess) return set_error(ctx, SPADE_E_HIP, "hipSetDevice failed");
    if (!pts || pts->n < 0 || (pts->n > 0 && (!pts->x || !pts->y)))
        return set_error(ctx, SPADE_E_INVALID, "invalid point arrays");
    if (pts->n > (int64_t)INT32_MAX) return set_error(ctx, SPADE_E_TOO_LARGE, "a table holds at most 2^31 - 1 points");
    hipStream_t st = ctx->stream;
    spade_table *t = new (std::nothrow) spade_table();
    if (!t) return set_error(ctx, SPADE_E_NOMEM, "host allocation failed");
    t->device = ctx->device;
    const int64_t n = pts->n;
    t->n = n;
    auto fail = [&](int rc) { spade_table_destroy(t); return rc; };
    const size_t ns = (size_t)std::max<int64_t>(n, 1);
    if (ensure(ctx, t->x, 8 * ns) || ensure(ctx, t->y, 8 * ns) || ensure(ctx, t->ids, 4 * ns)) return fail(SPADE_E_NOMEM);
    // bounding box and grid
    DevBuf &bb = ctx->scratch[S_BLOCKRED];
    if (ensure(ctx, bb, 64)) return fail(SPADE_E_NOMEM);
    SPADE_HIP(ctx, hipMemsetAsync(bb.p, 0xff, 32, st));
    if (n > 0) hipLaunchKernelGGL(k_pt_bbox, dim3(grid_of(n, 1024)), dim3(256), 0, st, n, pts->x, pts->y, (unsigned long long *)bb.p);
    unsigned long long *h = (unsigned long long *)ensure_pinned(ctx, 64);
    SPADE_HIP(ctx, hipMemcpyAsync(h, bb.p, 32, hipMemcpyDeviceToHost, st));
    SPADE_HIP(ctx, hipStreamSynchronize(st));
    double x0 = from_okey(h[0]), x1 = -from_okey(h[1]), y0 = from_okey(h[2]), y1 = -from_okey(h[3]);
    if (!(x0 <= x1)) { x0 = 0; x1 = 1; y0 = 0; y1 = 1; }
    const int G = (int)std::max<int64_t>(1, std::min<int64_t>(GRID_MAX, (int64_t)std::sqrt((double)n / 64.0)));
    t->G = G;
    t->X0 = x0; t->Y0 = y0;
    t->sx = (x1 > x0) ? G / (x1 - x0) : 0.0;
    t->sy = (y1 > y0) ? G / (y1 - y0) : 0.0;
    // cells in Z order: codes below P * P, P the power of two >= G
    int64_t P = 1;
    while (P < G) P <<= 1;
    const int64_t ncell = P * P;
    // sort by cell
    DevBuf &dk = ctx->scratch[S_KEYS], &dk2 = ctx->scratch[S_KEYS2], &dv = ctx->scratch[S_VALS];
    if (ensure(ctx, dk, 4 * ns) || ensure(ctx, dk2, 4 * ns) || ensure(ctx, dv, 4 * ns))
        return fail(SPADE_E_NOMEM);
    if (n > 0) {
        hipLaunchKernelGGL(k_pt_key, dim3(grid_of(n)), dim3(256), 0, st, n, pts->x, pts->y, t->X0, t->Y0, t->sx, t->sy,
                           G, (uint32_t)ncell, (uint32_t *)dk.p, (uint32_t *)dv.p);
        SPADE_HIP(ctx, hipGetLastError());
        DevBuf &cub = ctx->scratch[S_CUBTMP];
        size_t tb = 0;
        const int kb = std::max(1, bits_of((uint64_t)ncell));
        SPADE_HIP(ctx, hipcub::DeviceRadixSort::SortPairs(nullptr, tb, (const uint32_t *)dk.p, (uint32_t *)dk2.p,
                                                          (const uint32_t *)dv.p, (uint32_t *)t->ids.p, (int)n, 0, kb, st));
        if (ensure(ctx, cub, tb)) return fail(SPADE_E_NOMEM);
        SPADE_HIP(ctx, hipcub::DeviceRadixSort::SortPairs(cub.p, tb, (const uint32_t *)dk.p, (uint32_t *)dk2.p,
                                                          (const uint32_t *)dv.p, (uint32_t *)t->ids.p, (int)n, 0, kb, st));
        hipLaunchKernelGGL(k_pt_gather, dim3(grid_of(n)), dim3(256), 0, st, n, (const uint32_t *)t->ids.p, pts->x, pts->y,
                           (double *)t->x.p, (double *)t->y.p);
        hipLaunchKernelGGL(k_count_finite, dim3(1), dim3(1), 0, st, n, (const uint32_t *)dk2.p, (uint32_t)ncell,
                           (uint32_t *)bb.p);
        SPADE_HIP(ctx, hipGetLastError());
        uint32_t *hf = (uint32_t *)ensure_pinned(ctx, 64);
        SPADE_HIP(ctx, hipMemcpyAsync(hf, bb.p, 4, hipMemcpyDeviceToHost, st));
        SPADE_HIP(ctx, hipStreamSynchronize(st));
        t->nfin = hf[0];
    }
    t->nchunk = (t->nfin + CHUNK - 1) / CHUNK;
    if (ensure(ctx, t->chunk_bb, sizeof(double4) * (size_t)std::max<int64_t>(t->nchunk, 1))) return fail(SPADE_E_NOMEM);
    if (t->nchunk > 0) {
        hipLaunchKernelGGL(k_chunk_bb, dim3(grid_of(t->nchunk * 64, 8192)), dim3(256), 0, st, t->nfin, t->nchunk,
                           (const double *)t->x.p, (const double *)t->y.p, (double4 *)t->chunk_bb.p);
        SPADE_HIP(ctx, hipGetLastError());
    }
    SPADE_HIP(ctx, hipStreamSynchronize(st));
    *out = t;
    return SPADE_OK;
}

void spade_table_destroy(spade_table *t)
{
    if (!t) return;
    (void)hipSetDevice(t->device);
    free_buf(t->x);
    free_buf(t->y);
    free_buf(t->ids);
    free_buf(t->chunk_bb);
    delete t;
}

int spade_table_info(const spade_table *t, int64_t *n, int32_t *grid, int64_t *chunks, int64_t *device_bytes)
{
    if (!t) return SPADE_E_INVALID;
    if (n) *n = t->n;
    if (grid) *grid = t->G;
    if (chunks) *chunks = t->nchunk;
    if (device_bytes) *device_bytes = (int64_t)t->bytes();
    return SPADE_OK;
}

static int check_batch_args(spade_ctx *ctx, const spade_polys *polys, int32_t nq, const int64_t *qbound)
{
    ctx->err.clear();
    if (hipSetDevice(ctx->device) != hipSuccess) return set_error(ctx, SPADE_E_HIP, "hipSetDevice failed");
    if (!polys || nq < 1 || !qbound) return set_error(ctx, SPADE_E_INVALID, "a batch needs polygons and nq >= 1 queries");
    if (polys->n_polys < 0 || polys->n_rings < 0 || (!polys->poly_ring_off && polys->n_rings != polys->n_polys))
        return set_error(ctx, SPADE_E_INVALID, "malformed polygon set");
    if (polys->n_rings > 0 && (!polys->ring_vtx_off || !polys->vx || !polys->vy))
        return set_error(ctx, SPADE_E_INVALID, "ring_vtx_off / vx / vy is NULL");
    if (qbound[0] != 0 || qbound[nq] != polys->n_polys) return set_error(ctx, SPADE_E_INVALID, "qbound must run from 0 to n_polys");
    for (int q = 0; q < nq; ++q)
        if (qbound[q + 1] < qbound[q]) return set_error(ctx, SPADE_E_INVALID, "qbound must be non-decreasing");
    return SPADE_OK;
}

int spade_batch_build(spade_ctx *ctx, const spade_polys *polys, int32_t nq, const int64_t *qbound,
                      spade_canvas **out)
{
    if (!ctx) return SPADE_E_INVALID;
    SPADE_CTX_LOCK(ctx);
    if (!ctx || !out) return SPADE_E_INVALID;
    *out = nullptr;
    int rc0 = check_batch_args(ctx, polys, nq, qbound);
    if (rc0) return rc0;
    spade_canvas *cv = new (std::nothrow) spade_canvas();
    if (!cv) return set_error(ctx, SPADE_E_NOMEM, "host allocation failed");
    cv->device = ctx->device;
    const int rc = build_set(ctx, polys, nq, qbound, cv);
    if (rc) {
        spade_canvas_destroy(cv);
        return rc;
    }
    *out = cv;
    return SPADE_OK;
}

int spade_batch_rebuild(spade_ctx *ctx, const spade_polys *polys, int32_t nq, const int64_t *qbound,
                        spade_canvas *set)
{
    if (!ctx) return SPADE_E_INVALID;
    SPADE_CTX_LOCK(ctx);
    if (!ctx || !set) return ctx ? set_error(ctx, SPADE_E_INVALID, "NULL argument") : SPADE_E_INVALID;
    int rc = check_batch_args(ctx, polys, nq, qbound);
    if (rc) return rc;
    if (set->device != ctx->device) return set_error(ctx, SPADE_E_INVALID, "the canvas set lives on another device");
    if (set == ctx->plain) return set_error(ctx, SPADE_E_INVALID, "not a caller-owned canvas set");
    set->layered = false;
    set->n_layers = 0;
    return build_set(ctx, polys, nq, qbound, set);
}

int spade_batch_select(spade_ctx *ctx, const spade_canvas *set, const spade_table *t, uint32_t *out_ids, int64_t cap,
                       int64_t *out_off)
{
    if (!ctx) return SPADE_E_INVALID;
    SPADE_CTX_LOCK(ctx);
    if (!ctx || !set || !t || !out_off) return ctx ? set_error(ctx, SPADE_E_INVALID, "NULL argument") : SPADE_E_INVALID;
    ctx->err.clear();
    if (hipSetDevice(ctx->device) != hipSuccess) return set_error(ctx, SPADE_E_HIP, "hipSetDevice failed");
    const int nq = set->nc;
    if (set->layered) return set_error(ctx, SPADE_E_INVALID, "a layered set is queried with join calls");
    for (int q = 0; q < nq; ++q)
        if (set->descs[q].M != 1) return set_error(ctx, SPADE_E_INVALID, "batch selection needs exactly one polygon per query");
    if (cap < 0 || (cap > 0 && !out_ids)) return set_error(ctx, SPADE_E_INVALID, "bad output buffer");
    hipStream_t st = ctx->stream;
    ctx->timed_raster = false;
    Pairs P;
    int rc = make_pairs(ctx, set, t, P);
    if (rc) return rc;
    const SetArgs S = set_args(set);
    // Windows of the id buckets: the largest, or smaller ones while the
    // buckets are too few to fill the chip (a single served selection).
    const int cus = num_cus_of(ctx->device);
    const int idbits = std::max(1, bits_of((uint64_t)std::max<int64_t>(t->n - 1, 1)));
    int L = std::min(idbits, SORT_LBITS);
    auto bins_at = [&](int l) { return (int)(((uint64_t)std::max<int64_t>(t->n - 1, 0) >> l) + 1); };
    while (L > SORT_LMIN && (int64_t)nq * bins_at(L) < 2 * cus && bins_at(L - 1) <= TILE_BINS) --L;
    const int nbins = cap > 0 ? bins_at(L) : 1;   // counts alone need no windows
    // The queries are taken in groups.  A group's pairs, every query's rounded
    // up to whole tiles (a tile's keys take 64 KB however few pairs or ids it
    // has), have hit words of 512 bytes within the limit
    // (SPADE_HIT_MASK_LIMIT bytes, default 512 MiB: 2^20 pairs, so 2^18 tiles,
    // whose keys take 16 GiB), and its buckets are at most 2^26; or it is one
    // query.  Nearly always one group.
    size_t hits_max = (size_t)512 << 20;
    if (const char *e = getenv("SPADE_HIT_MASK_LIMIT")) hits_max = (size_t)strtoull(e, nullptr, 10);
    constexpr size_t PAIR_BYTES = sizeof(unsigned long long) * BW_WORDS;
    constexpr size_t TILE_BYTES = PAIR_BYTES * TILE_PAIRS;
    constexpr int64_t BUCKETS = (int64_t)1 << 26;
    DevBuf &bh = ctx->scratch[S_KEYS2], &bo = ctx->scratch[S_ENTF], &bs = ctx->scratch[S_LOOKBACK];
    const std::vector<int64_t> &hq = P.qfirst;   // first pair of every query
    std::vector<int> gq;                         // first query of every group, then nq
    int64_t pmost, tmost;                        // most pairs and tiles of a group
    int gmost;                                   // most queries of one
    auto tiles_of = [&](int q) { return (hq[(size_t)q + 1] - hq[(size_t)q] + TILE_PAIRS - 1) / TILE_PAIRS; };
    auto group_by = [&](size_t limit) {
        gq.assign(1, 0);
        pmost = tmost = gmost = 1;
        int64_t tiles = 0;
        for (int q = 0; q < nq; ++q) {
            const int qb = gq.back();
            if (q > qb && ((size_t)(tiles + tiles_of(q)) * TILE_BYTES > limit || (int64_t)(q + 1 - qb) * nbins > BUCKETS)) {
                gq.push_back(q);
                tiles = 0;
            }
            tiles += tiles_of(q);
            pmost = std::max(pmost, hq[(size_t)q + 1] - hq[(size_t)gq.back()]);
            tmost = std::max(tmost, tiles);
            gmost = std::max(gmost, q + 1 - gq.back());
        }
        gq.push_back(nq);
    };
    auto room = [&]() {
        return ensure(ctx, bh, PAIR_BYTES * (size_t)pmost) ||
               (cap > 0 && (ensure(ctx, bo, sizeof(uint32_t) * TILE_IDS * (size_t)tmost) ||
                            ensure(ctx, bs, sizeof(uint16_t) * (size_t)(nbins + 1) * (size_t)tmost)));
    };
    group_by(hits_max);
    while (room()) {
        if (gmost == 1 || hits_max < TILE_BYTES) return SPADE_E_NOMEM;   // one query at a time needs the least
        ctx->err.clear();
        hits_max = std::min(hits_max, (size_t)tmost * TILE_BYTES) / 2;
        group_by(hits_max);
    }
    unsigned long long *hits = (unsigned long long *)bh.p;
    uint32_t *keys = (uint32_t *)bo.p;
    uint16_t *starts = (uint16_t *)bs.p;
    // bc: bucket counts [nbmax + 1] | offsets [nbmax + 1]
    const size_t nbmax = (size_t)gmost * nbins;
    DevBuf &bc = ctx->scratch[S_VALS2], &cub = ctx->scratch[S_CUBTMP];
    if (ensure(ctx, bc, sizeof(unsigned long long) * 2 * (nbmax + 1))) return SPADE_E_NOMEM;
    unsigned long long *tot = (unsigned long long *)bc.p, *offs = tot + (nbmax + 1);
    unsigned long long *h = (unsigned long long *)ensure_pinned(ctx, 8 * ((size_t)gmost + 1));
    if (!h) return set_error(ctx, SPADE_E_NOMEM, "pinned staging allocation failed");
    // the bitmap in whole blocks of 64 words
    const size_t bm_lds = sizeof(uint32_t) * 64 * (size_t)((std::max(1, (1 << L) >> 5) + 63) / 64);
    const size_t tile_lds = sizeof(uint32_t) * ((size_t)((nbins + 127) & ~63) + TILE_IDS);
    SPADE_HIP(ctx, hipFuncSetAttribute((const void *)k_bucket_bitmap, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)bm_lds));
    SPADE_HIP(ctx, hipFuncSetAttribute((const void *)k_hit_tiles, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)tile_lds));
    out_off[0] = 0;
    // the timed probe of a batch selection is its probe pass (its first group's)
    if (ctx->timing) SPADE_HIP(ctx, hipEventRecord(ctx->ev[2], st));
    for (size_t k = 0; k + 1 < gq.size(); ++k) {
        const int q0 = gq[k], q1 = gq[k + 1], ng = q1 - q0;
        const uint32_t p0 = (uint32_t)hq[(size_t)q0], p1 = (uint32_t)hq[(size_t)q1];
        const int64_t nb = (int64_t)ng * nbins;
        uint32_t ntile = 0;
        for (int q = q0; q < q1; ++q) ntile += (uint32_t)tiles_of(q);
        const uint32_t *dtf = P.tfirst + q0;
        if (ntile == 0) {
            if (ctx->timing && k == 0) SPADE_HIP(ctx, hipEventRecord(ctx->ev[3], st));
            for (int q = q0; q < q1; ++q) out_off[q + 1] = out_off[q0];
            continue;
        }
        const bool by_pair = (int64_t)(p1 - p0) * 2 <= t->nchunk;
        const int64_t wgs = (by_pair ? (int64_t)(p1 - p0) : t->nchunk) * BW_TASKS / (BT_THREADS / 64);
        auto probe = [&](auto kern) {
            hipLaunchKernelGGL(kern, dim3((unsigned)std::min<int64_t>(wgs, 1 << 20)), dim3(BT_THREADS), 0, st, S, t->nfin,
                               t->nchunk, (const double *)t->x.p, (const double *)t->y.p, (const unsigned int *)P.cbase,
                               (const uint32_t *)P.plist, (const uint32_t *)P.pq, (const uint32_t *)P.pc, p0, p1, hits);
        };
        if (by_pair) probe(k_batch_hits<true>);
        else probe(k_batch_hits<false>);
        SPADE_HIP(ctx, hipGetLastError());
        if (ctx->timing && k == 0) SPADE_HIP(ctx, hipEventRecord(ctx->ev[3], st));
        if (cap > 0) {
            hipLaunchKernelGGL(k_hit_tiles, dim3(ntile), dim3(TILE_THREADS), tile_lds, st, ng, (const uint32_t *)dtf,
                               (const unsigned long long *)P.qbase + q0, p0, P.pc, hits, (const uint32_t *)t->ids.p, L,
                               nbins, keys, starts);
            hipLaunchKernelGGL(k_bucket_tot, dim3((nbins + 63) / 64, std::min(ng, 32768)), dim3(TILE_THREADS), 0, st, ng,
                               (const uint32_t *)dtf, (const uint16_t *)starts, nbins, tot);
        } else {
            hipLaunchKernelGGL(k_zero64, dim3(grid_of(ng, 4096)), dim3(256), 0, st, (int64_t)ng, tot);
            hipLaunchKernelGGL(k_hit_count, dim3((unsigned)std::min<int64_t>((p1 - p0 + 3) / 4, 1 << 16)), dim3(256), 0, st,
                               p0, p1, (uint32_t)q0, (const uint32_t *)P.pq, (const unsigned long long *)hits, tot);
        }
        SPADE_HIP(ctx, hipGetLastError());
        if (nb <= BUCKET_SCAN_MAX) {
            hipLaunchKernelGGL(k_bucket_scan, dim3(1), dim3(PS_THREADS), 0, st, ng, nbins, (const unsigned long long *)tot,
                               offs, h);
        } else {
            hipLaunchKernelGGL(k_zero64, dim3(1), dim3(64), 0, st, (int64_t)1, tot + nb);
            size_t tb = 0;
            SPADE_HIP(ctx, hipcub::DeviceScan::ExclusiveSum(nullptr, tb, tot, offs, (int)(nb + 1), st));
            if (ensure(ctx, cub, tb)) return SPADE_E_NOMEM;
            SPADE_HIP(ctx, hipcub::DeviceScan::ExclusiveSum(cub.p, tb, tot, offs, (int)(nb + 1), st));
            hipLaunchKernelGGL(k_query_off, dim3((ng + 256) / 256), dim3(256), 0, st, ng, nbins, offs, h);
        }
        // ids beyond cap are not written (a buffer that is too small still
        // receives the first cap ids)
        const int64_t base = out_off[q0];   // ids of the groups before
        if (base < cap)
            hipLaunchKernelGGL(k_bucket_bitmap, dim3((unsigned)std::min<int64_t>(nb, 65536)), dim3(BKT_THREADS), bm_lds,
                               st, nb, offs, (const uint32_t *)dtf, (const uint16_t *)starts, (const uint32_t *)keys, L,
                               nbins, out_ids + base, cap - base);
        SPADE_HIP(ctx, hipGetLastError());
        SPADE_HIP(ctx, hipStreamSynchronize(st));
        for (int q = q0; q <= q1; ++q) out_off[q] = base + (int64_t)h[q - q0];
    }
    if (out_off[nq] > cap) return set_error(ctx, SPADE_E_CAPACITY, "output capacity too small");
    return SPADE_OK;
}

}  // extern "C"

namespace spade {

void drop_batch_graph(spade_canvas *cv)
{
    if (cv->bexec) (void)hipGraphExecDestroy(cv->bexec);
    cv->bexec = nullptr;
    cv->bkey.clear();
}

// The batch join-count's launches (clear the counts, the canvas boxes, the
// one-pass probe) for the current buffers; all parameters are in `key`.
static hipError_t batch_count_launches(spade_ctx *ctx, const spade_canvas *set, const spade_table *t, int64_t M,
                                       uint64_t *out_counts, hipStream_t s, const uint8_t *skip = nullptr)
{
    const int nq = set->nc;
    if (M > 0) hipLaunchKernelGGL(k_zero64, dim3(grid_of(M, 4096)), dim3(256), 0, s, M, (unsigned long long *)out_counts);
    hipLaunchKernelGGL(k_qbox, dim3((nq + 255) / 256), dim3(256), 0, s, nq, (const CanvasDesc *)set->dcds.p, skip,
                       (double4 *)set->qbox.p);
    const SetArgs S = set_args(set);
    const int grid = (int)std::max<int64_t>(1, std::min<int64_t>(t->nchunk, (int64_t)num_cus_of(ctx->device) * 8));
    if (t->nchunk > 0 && M > 0)
        hipLaunchKernelGGL(k_batch_count_direct, dim3(grid), dim3(BT_THREADS), 0, s, S, nq, t->nfin, t->nchunk,
                           (const double *)t->x.p, (const double *)t->y.p, (const double4 *)t->chunk_bb.p,
                           (const double4 *)set->qbox.p, (unsigned long long *)out_counts);
    return hipGetLastError();
}

}  // namespace spade

extern "C" {

int spade_batch_join_count(spade_ctx *ctx, const spade_canvas *set, const spade_table *t, uint64_t *out_counts)
{
    if (!ctx) return SPADE_E_INVALID;
    SPADE_CTX_LOCK(ctx);
    if (!ctx || !set || !t) return ctx ? set_error(ctx, SPADE_E_INVALID, "NULL argument") : SPADE_E_INVALID;
    ctx->err.clear();
    if (hipSetDevice(ctx->device) != hipSuccess) return set_error(ctx, SPADE_E_HIP, "hipSetDevice failed");
    int64_t M = 0;
    for (const auto &d : set->descs) M += d.M;
    if (M > 0 && !out_counts) return set_error(ctx, SPADE_E_INVALID, "out_counts is NULL");
    hipStream_t st = ctx->stream;
    ctx->timed_raster = false;
    spade_canvas *cv = const_cast<spade_canvas *>(set);
    if (ensure(ctx, cv->qbox, sizeof(double4) * (size_t)std::max(set->nc, 1))) return SPADE_E_NOMEM;
    // The launches depend only on these values (every pointer and size they
    // take): a call with the same ones (the same set and table memory,
    // typically a rebuilt batch) replays the graph captured on the second
    // such call.
    const std::vector<uint64_t> key = {
        (uint64_t)(uintptr_t)set->dcds.p, (uint64_t)(uintptr_t)set->cells.p, (uint64_t)(uintptr_t)set->coarse.p,
        (uint64_t)(uintptr_t)set->cands.p, (uint64_t)(uintptr_t)set->ledges.p, (uint64_t)(uintptr_t)set->pspan.p,
        (uint64_t)(uintptr_t)set->qbox.p, (uint64_t)(uintptr_t)(set->layered ? set->pid.p : nullptr),
        (uint64_t)set->nc, (uint64_t)M, (uint64_t)(uintptr_t)t->x.p, (uint64_t)(uintptr_t)t->y.p,
        (uint64_t)(uintptr_t)t->chunk_bb.p, (uint64_t)t->nfin, (uint64_t)t->nchunk, (uint64_t)(uintptr_t)out_counts};
    // A canvas over at least a quarter of the table's box whose polygons fit
    // the count probe's LDS histogram is counted by that probe over all the
    // table's points (a canvas of a tessellation over the extent, say): it
    // streams them several times faster than the per-chunk probe looks them
    // up, which outweighs the per-chunk probe's one read of a chunk for all
    // the canvases that meet it.  Not for a layered set, whose counts go
    // through its polygon-id map.
    std::vector<int> routed;
    std::vector<uint8_t> hskip;   // read by an asynchronous copy: lives to the final synchronisation
    if (!set->layered) {
        const double tw = t->sx > 0 ? t->G / t->sx : 0.0, th = t->sy > 0 ? t->G / t->sy : 0.0;
        const double tx1 = t->X0 + tw, ty1 = t->Y0 + th;
        for (int q = 0; q < set->nc && t->nfin > 0; ++q) {
            const CanvasDesc &d = set->descs[(size_t)q];
            if (d.empty || d.M <= 0 || d.M > HIST_MAX_BATCH) continue;
            const double ox = std::min(d.bx1, tx1) - std::max(d.bx0, t->X0);
            const double oy = std::min(d.by1, ty1) - std::max(d.by0, t->Y0);
            if (ox > 0 && oy > 0 && ox * oy >= 0.25 * tw * th) routed.push_back(q);
        }
    }
    if (ctx->timing) SPADE_HIP(ctx, hipEventRecord(ctx->ev[2], st));
    hipError_t e;
    if (!routed.empty()) {
        e = hipSuccess;
        const uint8_t *skip = nullptr;
        int64_t Mrest = 0;
        if ((int)routed.size() < set->nc) {
            hskip.assign((size_t)set->nc, 0);
            for (int q : routed) hskip[(size_t)q] = 1;
            for (int q = 0; q < set->nc; ++q)
                if (!hskip[(size_t)q]) Mrest += set->descs[(size_t)q].M;
            DevBuf &bs = ctx->scratch[S_MISC];
            if (ensure(ctx, bs, (size_t)set->nc)) return SPADE_E_NOMEM;
            SPADE_HIP(ctx, hipMemcpyAsync(bs.p, hskip.data(), (size_t)set->nc, hipMemcpyHostToDevice, st));
            skip = (const uint8_t *)bs.p;
        }
        if (Mrest > 0) e = batch_count_launches(ctx, set, t, M, out_counts, st, skip);
        const bool timing = ctx->timing;
        ctx->timing = false;   // the batch call's events frame every launch
        spade_points tp{};
        tp.n = t->nfin;
        tp.x = (const double *)t->x.p;
        tp.y = (const double *)t->y.p;
        for (int q : routed) {
            if (e != hipSuccess) break;
            const CanvasDesc &d = set->descs[(size_t)q];
            spade_canvas one;
            one.view = view_of(set, q);
            const int rc2 = probe_count(ctx, &one, &tp, out_counts + d.poly_base);
            if (rc2) {
                ctx->timing = timing;
                return rc2;
            }
        }
        ctx->timing = timing;
    } else if (!ctx->graphs) {
        e = batch_count_launches(ctx, set, t, M, out_counts, st);
    } else if (cv->bexec && cv->bkey == key) {
        ++ctx->graph_replays;
        e = hipGraphLaunch(cv->bexec, st);
    } else if (cv->bkey != key) {
        drop_batch_graph(cv);
        cv->bkey = key;
        e = batch_count_launches(ctx, set, t, M, out_counts, st);
    } else {
        // second call with these parameters: capture (on an internal stream,
        // the caller's may be the null stream), then launch the graph
        e = hipSuccess;
        if (!ctx->capture && (e = hipStreamCreateWithFlags(&ctx->capture, hipStreamNonBlocking)) != hipSuccess) {
            (void)hipGetLastError();
            ctx->capture = nullptr;
        }
        hipGraph_t g = nullptr;
        hipGraphExec_t ex = nullptr;
        if (ctx->capture && hipStreamBeginCapture(ctx->capture, hipStreamCaptureModeThreadLocal) == hipSuccess) {
            const hipError_t e1 = batch_count_launches(ctx, set, t, M, out_counts, ctx->capture);
            const hipError_t e2 = hipStreamEndCapture(ctx->capture, &g);
            if (e1 == hipSuccess && e2 == hipSuccess && g &&
                hipGraphInstantiate(&ex, g, nullptr, nullptr, 0) == hipSuccess) {
                cv->bexec = ex;
                ++ctx->graph_captures;
            }
            if (g) (void)hipGraphDestroy(g);
        }
        (void)hipGetLastError();
        if (cv->bexec) e = hipGraphLaunch(cv->bexec, st);
        else {
            cv->bkey.clear();
            e = batch_count_launches(ctx, set, t, M, out_counts, st);
        }
    }
    if (e != hipSuccess) return hip_fail(ctx, e, "batch join-count launches");
    if (ctx->timing) SPADE_HIP(ctx, hipEventRecord(ctx->ev[3], st));
    SPADE_HIP(ctx, hipStreamSynchronize(st));
    return SPADE_OK;
}

// Join pairs by sorted keys, as far as room keys hold them (several polygons
// of a query may hold a point); done is left false when they don't, or when the
// memory is not there.
static int sorted_pairs(spade_ctx *ctx, const spade_table *t, const SetArgs &S, const Pairs &P, int64_t M,
                        unsigned long long room, uint32_t *out_pt, uint32_t *out_poly, int64_t cap, int64_t *n_out,
                        bool &done)
{
    hipStream_t st = ctx->stream;
    DevBuf &bk = ctx->scratch[S_ENTC], &bs = ctx->scratch[S_KEYS2], &bc = ctx->scratch[S_VALS2], &cub = ctx->scratch[S_CUBTMP];
    const int pbits = bits_of((uint64_t)(M - 1)), idbits = std::max(1, bits_of((uint64_t)(t->n - 1)));
    if (ensure(ctx, bc, sizeof(unsigned long long))) return SPADE_E_NOMEM;
    unsigned long long *cursor = (unsigned long long *)bc.p, *keys = nullptr, *sorted = nullptr;
    if (cap > 0 && P.np > 0) {
        if (ensure(ctx, bk, 8 * (size_t)room) || ensure(ctx, bs, 8 * (size_t)room)) {
            ctx->err.clear();
            return SPADE_OK;
        }
        keys = (unsigned long long *)bk.p;
        sorted = (unsigned long long *)bs.p;
    }
    unsigned long long *h = (unsigned long long *)ensure_pinned(ctx, 64);
    if (!h) return set_error(ctx, SPADE_E_NOMEM, "pinned staging allocation failed");
    hipLaunchKernelGGL(k_zero64, dim3(1), dim3(64), 0, st, (int64_t)1, cursor);
    if (ctx->timing) SPADE_HIP(ctx, hipEventRecord(ctx->ev[2], st));
    if (P.np > 0)
        hipLaunchKernelGGL(k_batch_pkeys, dim3((unsigned)std::min<int64_t>(P.np, 1 << 20)), dim3(PK_THREADS), 0, st, S,
                           t->nfin, (const double *)t->x.p, (const double *)t->y.p, (const uint32_t *)t->ids.p, P.pq, P.pc,
                           (uint32_t)P.np, pbits, cursor, keys, room);
    SPADE_HIP(ctx, hipGetLastError());
    SPADE_HIP(ctx, hipMemcpyAsync(h, cursor, sizeof(unsigned long long), hipMemcpyDeviceToHost, st));
    SPADE_HIP(ctx, hipStreamSynchronize(st));
    const int64_t total = (int64_t)h[0];
    if (cap > 0 && h[0] > room) return SPADE_OK;
    if (cap > 0 && total > 0) {
        size_t tb = 0;
        SPADE_HIP(ctx, hipcub::DeviceRadixSort::SortKeys(nullptr, tb, (const unsigned long long *)keys, sorted, (int)total, 0,
                                                         pbits + idbits, st));
        if (ensure(ctx, cub, std::max<size_t>(tb, 1))) {
            ctx->err.clear();
            return SPADE_OK;
        }
        SPADE_HIP(ctx, hipcub::DeviceRadixSort::SortKeys(cub.p, tb, (const unsigned long long *)keys, sorted, (int)total, 0,
                                                         pbits + idbits, st));
        const int64_t nw = std::min(total, cap);
        hipLaunchKernelGGL(k_split_keys, dim3(grid_of(nw)), dim3(256), 0, st, nw, (const unsigned long long *)sorted, pbits,
                           out_pt, out_poly);
        SPADE_HIP(ctx, hipGetLastError());
    }
    if (ctx->timing) SPADE_HIP(ctx, hipEventRecord(ctx->ev[3], st));
    SPADE_HIP(ctx, hipStreamSynchronize(st));
    *n_out = total;
    done = true;
    return total > cap ? set_error(ctx, SPADE_E_CAPACITY, "output capacity too small") : SPADE_OK;
}

int spade_batch_join_pairs(spade_ctx *ctx, const spade_canvas *set, const spade_table *t, uint32_t *out_pt,
                           uint32_t *out_poly, int64_t cap, int64_t *n_out)
{
    if (!ctx) return SPADE_E_INVALID;
    SPADE_CTX_LOCK(ctx);
    if (!ctx || !set || !t || !n_out) return ctx ? set_error(ctx, SPADE_E_INVALID, "NULL argument") : SPADE_E_INVALID;
    ctx->err.clear();
    *n_out = 0;
    if (hipSetDevice(ctx->device) != hipSuccess) return set_error(ctx, SPADE_E_HIP, "hipSetDevice failed");
    if (cap < 0 || (cap > 0 && (!out_pt || !out_poly))) return set_error(ctx, SPADE_E_INVALID, "bad output buffers");
    int64_t M = 0;
    for (const auto &d : set->descs) M += d.M;
    hipStream_t st = ctx->stream;
    ctx->timed_raster = false;
    if (M == 0 || t->nchunk == 0) return SPADE_OK;
    Pairs P;
    int rc = make_pairs(ctx, set, t, P);
    if (rc) return rc;
    const SetArgs S = set_args(set);
    const int64_t n = t->n;
    DevBuf &bc = ctx->scratch[S_VALS2], &bo = ctx->scratch[S_ENTC], &cub = ctx->scratch[S_CUBTMP];
    if (P.np * CHUNK <= (n >= PK_LARGE ? n * PK_OVER : n / PK_PART)) {
        bool done = false;
        const int64_t room = std::min<int64_t>({P.np * CHUNK, n + n / 8, INT32_MAX});
        rc = sorted_pairs(ctx, t, S, P, M, (unsigned long long)room, out_pt, out_poly, cap, n_out, done);
        if (rc || done) return rc;
    }
    // counts by point id, and their places (64-bit: a join may hold more than
    // 2^32 pairs)
    if (ensure(ctx, bc, sizeof(uint32_t) * (size_t)(n + 2)) || ensure(ctx, bo, sizeof(unsigned long long) * (size_t)(n + 1)))
        return SPADE_E_NOMEM;
    uint32_t *pcnt = (uint32_t *)bc.p, *some_long = pcnt + (n + 1);
    unsigned long long *offs = (unsigned long long *)bo.p;
    const auto counts64 = rocprim::make_transform_iterator((const uint32_t *)pcnt, Widen());
    size_t tb = 0;
    SPADE_HIP(ctx, rocprim::exclusive_scan(nullptr, tb, counts64, offs, 0ull, (size_t)(n + 1),
                                           rocprim::plus<unsigned long long>(), st));
    if (ensure(ctx, cub, std::max<size_t>(tb, 1))) return SPADE_E_NOMEM;
    unsigned long long *h = (unsigned long long *)ensure_pinned(ctx, 64);
    if (!h) return set_error(ctx, SPADE_E_NOMEM, "pinned staging allocation failed");
    // The count pass keeps every pair's matching points (512 bytes) for the
    // write pass.  Should they exceed 16 GiB, the chunks are taken in groups
    // whose words do not (a chunk has at most one pair per canvas), and each
    // group is counted again right before it is written.
    const int64_t per_chunk = (int64_t)sizeof(unsigned long long) * BW_WORDS * set->nc;
    int64_t group = t->nchunk;
    size_t hbytes = sizeof(unsigned long long) * BW_WORDS * (size_t)std::max<int64_t>(P.np, 1);
    DevBuf &bh = ctx->scratch[S_KEYS2];
    if (cap > 0 && (hbytes > PAIR_HITS_MAX || ensure(ctx, bh, hbytes))) {
        ctx->err.clear();
        size_t room = PAIR_HITS_MAX;
        group = std::max<int64_t>(1, (int64_t)(room / (size_t)per_chunk));
        while (ensure(ctx, bh, (size_t)(group * per_chunk))) {
            if (group == 1) return SPADE_E_NOMEM;
            ctx->err.clear();
            group = std::max<int64_t>(1, group / 4);
        }
    }
    unsigned long long *hits = cap > 0 ? (unsigned long long *)bh.p : nullptr;
    hipLaunchKernelGGL(k_zero32, dim3(grid_of(n + 2, 4096)), dim3(256), 0, st, n + 2, (unsigned int *)pcnt);
    if (ctx->timing) SPADE_HIP(ctx, hipEventRecord(ctx->ev[2], st));
    const auto task_grid = [&](int64_t chunks, int tasks) {
        return dim3((unsigned)std::max<int64_t>(1, std::min<int64_t>(chunks * tasks / (BT_THREADS / 64), 1 << 20)));
    };
    auto count = [&](int64_t c0, int64_t c1, unsigned long long *keep) {
        hipLaunchKernelGGL(k_batch_pcount, task_grid(c1 - c0, BW_TASKS), dim3(BT_THREADS), 0, st, S, t->nfin, c0, c1,
                           (const double *)t->x.p, (const double *)t->y.p, (const uint32_t *)t->ids.p, P.cbase, P.plist,
                           P.pq, pcnt, keep, some_long);
    };
    count(0, t->nchunk, group == t->nchunk ? hits : nullptr);
    SPADE_HIP(ctx, hipGetLastError());
    SPADE_HIP(ctx, rocprim::exclusive_scan(cub.p, tb, counts64, offs, 0ull, (size_t)(n + 1),
                                           rocprim::plus<unsigned long long>(), st));
    if (cap > 0) {
        for (int64_t c0 = 0; c0 < t->nchunk; c0 += group) {
            const int64_t c1 = std::min(t->nchunk, c0 + group);
            if (group < t->nchunk) count(c0, c1, hits);
            auto write = [&](auto kern, auto... args) {
                hipLaunchKernelGGL(kern, task_grid(c1 - c0, BW_WORDS), dim3(BT_THREADS), 0, st, S, t->nfin, c0, c1,
                                   (const double *)t->x.p, (const double *)t->y.p, (const uint32_t *)t->ids.p, P.cbase,
                                   P.plist, P.pq, (const unsigned long long *)hits, (const unsigned long long *)offs, args...,
                                   out_poly, cap);
            };
            // 16-bit lists hold the polygon ids of at most 2^16 polygons
            if (M <= 65536) write(k_batch_pwrite<uint16_t>);
            else write(k_batch_pwrite<uint32_t>);
            write(k_batch_plong, (const uint32_t *)some_long, (uint32_t)M);
        }
        hipLaunchKernelGGL(k_pair_points, dim3(grid_of(n)), dim3(256), 0, st, n, (const unsigned long long *)offs, out_pt,
                           cap);
        SPADE_HIP(ctx, hipGetLastError());
    }
    if (ctx->timing) SPADE_HIP(ctx, hipEventRecord(ctx->ev[3], st));
    SPADE_HIP(ctx, hipMemcpyAsync(h, offs + n, sizeof(unsigned long long), hipMemcpyDeviceToHost, st));
    SPADE_HIP(ctx, hipStreamSynchronize(st));
    *n_out = (int64_t)h[0];
    if (*n_out > cap) return set_error(ctx, SPADE_E_CAPACITY, "output capacity too small");
    return SPADE_OK;
}

}  // extern "C"
