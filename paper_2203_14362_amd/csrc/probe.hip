// Point probes against a discrete canvas: the paper's mask + multiway blend
// (aggregation) and mask + Map (selection / join) applied to a stream of
// points (Sec. 5.1, 5.2), as compute kernels.
//
// Every point is read once from HBM (FP64 structure of arrays, coalesced,
// non-temporal), rejected if it lies outside the half-open bounding box of
// the polygons and mapped to its pixel.  The pixel is classified in two
// levels: a coarse canvas held in LDS by every workgroup answers directly
// for blocks whose pixels share one label; points in any other block read their
// canvas word from the tile-major canvas in global memory (L2 / MALL).  A
// label is final; a boundary pixel needs the exact test of each candidate
// polygon.  Boundary points are compacted per wavefront (ballot + prefix
// count) into an LDS queue and tested in full wavefronts, so the rare,
// latency-bound exact tests do not stall the stream.
//
//   k_count  per-polygon counts: workgroup-private histograms in LDS
//            (additive blend), flushed into a context accumulator; the last
//            workgroup copies the counts out and clears the accumulator.
//            More polygons than that histogram holds: every point's polygon
//            goes to a 16-bit label that k_label_hist counts.
//   k_emit*  ordered output (point ids, or (point, polygon) pairs ascending):
//            the paper's two-step Map (a count pass per wavefront segment of
//            points that keeps every point's result, a scan of the segment
//            counts, a write pass from the results; points in several
//            polygons are probed again).
#include "common.h"
#include "exact.h"
#include "lookup.h"

#include <hipcub/hipcub.hpp>

#include <algorithm>
#include <mutex>
#include <string>

namespace spade {

constexpr int CNT_THREADS = 1024;         // count probe workgroup
constexpr int CNT_UNROLL = 5;             // points per thread per iteration (6 spills)
constexpr int QCAP = 64;                  // boundary queue entries per wavefront
constexpr int HIST_MAX = 8192;            // polygons counted in LDS
constexpr int EMIT_THREADS = 1024;
constexpr int EMIT_GROUP = 8;             // points per lane in flight (count pass)
constexpr int EMIT_WGROUP = 4;            // points per lane in flight (write pass)
constexpr int EMIT_WDRAIN = 8;            // words of the write pass sharing one boundary queue
constexpr size_t LDS_TOTAL = 160 * 1024;
constexpr size_t LDS_RESERVE = 2048;      // static LDS of the kernels
constexpr size_t QUEUE_BYTES = (size_t)(CNT_THREADS / 64) * QCAP * 20;
constexpr size_t EMIT_INDEX_BYTES = (size_t)(EMIT_THREADS / 64) * QCAP * sizeof(uint16_t);   // beside the queue, in the reserve

size_t coarse_lds_budget(int64_t M)
{
    // the labelling probe's queue also holds the points' indices
    size_t hist = (M <= HIST_MAX) ? sizeof(uint32_t) * (size_t)M : sizeof(uint32_t) * (CNT_THREADS / 64) * QCAP;
    size_t used = LDS_RESERVE + QUEUE_BYTES + hist;
    return used < LDS_TOTAL ? LDS_TOTAL - used : 0;
}

// ------------------------------------------------------------ join-count

// Exact test of a point against the records of its boundary pixel, two
// records at a time (most pixels have two; the slot after the last record
// exists and is never used); add(poly) for every polygon containing it.
template <typename Add>
__device__ __forceinline__ void test_records(const CanvasView &cv, uint32_t rec, double x, double y, Add &&add)
{
    while (true) {
        const Cand c0 = cv.cands[rec];
        const Cand c1 = cv.cands[rec + 1];
        if (cand_inside(cv, c0, x, y)) add(c0.poly);
        if (c0.meta & CAND_LAST) break;
        if (cand_inside(cv, c1, x, y)) add(c1.poly);
        if (c1.meta & CAND_LAST) break;
        rec += 2;
    }
}

// Counts accumulate in a context-owned accumulator `acc` that is all zero
// between calls: the last workgroup to finish (found with a counter, after a
// device-scope fence) copies acc into the caller's output and clears acc and
// the counter again, so a query needs no memset.  Each wavefront tests its
// queued boundary points itself whenever 64 have gathered.
//
// MODE: C_LDS counts in the LDS histogram; C_ATOMIC adds every match to acc
// (the path that needs no memory of its own); C_LABEL stores every point's
// polygon (NO_LABEL: none) in labels and adds only the further polygons of a
// point that lies in several to acc, the rest is k_label_hist's.  A global
// atomic per match is bound by the rate of scattered atomics, about 10 per ns:
// 30M points x 40,000 cells took 3.24 ms with them and 0.80 ms without.
enum { C_LDS = 0, C_ATOMIC = 1, C_LABEL = 2 };
constexpr uint32_t NO_LABEL = 0xffffu;

template <int MODE, int UNROLL>
__global__ __launch_bounds__(CNT_THREADS) void k_count(CanvasView cv, int64_t n, const double *X,
                                                       const double *Y, unsigned long long *acc,
                                                       unsigned int *done, unsigned long long *out, uint16_t *labels)
{
    constexpr bool LDSHIST = MODE == C_LDS;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ bool s_last;
    const int M = (int)cv.M;
    const size_t coarse_bytes = ((size_t)cv.Wc * cv.Hc * (cv.cbyte ? 1 : 2) + 15) & ~(size_t)15;
    uint16_t *coarse = (uint16_t *)smem;
    uint32_t *hist = (uint32_t *)(smem + coarse_bytes);
    const size_t hist_bytes = LDSHIST ? (((size_t)M * 4 + 15) & ~(size_t)15) : 0;
    unsigned char *qbase = smem + coarse_bytes + hist_bytes;
    const int wv = threadIdx.x >> 6;
    double *qx = (double *)(qbase) + wv * QCAP;
    double *qy = (double *)(qbase) + (CNT_THREADS / 64) * QCAP + wv * QCAP;
    uint32_t *qr = (uint32_t *)((double *)(qbase) + 2 * (CNT_THREADS / 64) * QCAP) + wv * QCAP;
    uint32_t *qi = qr + (CNT_THREADS / 64) * QCAP;   // C_LABEL: the points' indices (below 2^32)

    load_coarse(cv, coarse, CNT_THREADS);
    if (LDSHIST)
        for (int k = threadIdx.x; k < M; k += CNT_THREADS) hist[k] = 0;
    __syncthreads();

    auto add = [&](uint32_t k) {
        if (LDSHIST) atomicAdd(&hist[k], 1u);
        else atomicAdd(&acc[k], 1ull);
    };
    const uint32_t lane = lane_id();
    uint32_t qn = 0;   // wave-uniform queue length
    // exact tests of the queued points lo .. qn-1
    auto drain = [&](uint32_t lo) {
        __builtin_amdgcn_wave_barrier();
        if (lane >= lo && lane < qn) {
            if (MODE == C_LABEL) {
                uint32_t first = NO_LABEL;
                test_records(cv, qr[lane], qx[lane], qy[lane], [&](uint32_t k) {
                    if (first == NO_LABEL) first = k;
                    else atomicAdd(&acc[k], 1ull);
                });
                labels[qi[lane]] = (uint16_t)first;
            } else {
                test_records(cv, qr[lane], qx[lane], qy[lane], add);
            }
        }
        __builtin_amdgcn_wave_barrier();
        qn = 0;
    };

    // software pipeline: the next iteration's points are in flight while the
    // current ones are classified
    const int64_t step = (int64_t)gridDim.x * CNT_THREADS * UNROLL;
    double xn[UNROLL], yn[UNROLL];
    auto fetch = [&](int64_t b) {
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            const int64_t i = b + (int64_t)u * CNT_THREADS + threadIdx.x;
            xn[u] = i < n ? __builtin_nontemporal_load(X + i) : NAN;
            yn[u] = i < n ? __builtin_nontemporal_load(Y + i) : NAN;
        }
    };
    int64_t base = (int64_t)blockIdx.x * CNT_THREADS * UNROLL;
    if (base < n) fetch(base);
    for (; base < n; base += step) {
        double xs[UNROLL], ys[UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) { xs[u] = xn[u]; ys[u] = yn[u]; }
        if (base + step < n) fetch(base + step);
        // the coarse words of all points of this iteration first, then
        // their full-canvas reads, all issued before any result is used
        Look lk[UNROLL];
        uint32_t ws[UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) lk[u] = look_coarse(cv, coarse, xs[u], ys[u]);
#pragma unroll
        for (int u = 0; u < UNROLL; ++u)
            ws[u] = lk[u].full ? ((gu32p)cv.cells)[lk[u].fidx] : lk[u].word;
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            const uint32_t w = ws[u];
            const bool bnd = (w & BFLAG) != 0;
            const int64_t i = base + (int64_t)u * CNT_THREADS + threadIdx.x;
            if (MODE == C_LABEL) {
                if (!bnd && i < n) labels[i] = w != 0u ? (uint16_t)(w - 1u) : (uint16_t)NO_LABEL;
            } else if (w != 0u && !bnd) {
                add(w - 1u);
            }
            const unsigned long long mask = __ballot(bnd);
            const uint32_t nnew = (uint32_t)__popcll(mask);
            if (nnew == 0) continue;
            if (qn + nnew > QCAP) drain(0);
            if (bnd) {
                const uint32_t slot = qn + (uint32_t)__popcll(mask & ((1ull << lane) - 1ull));
                qx[slot] = xs[u];
                qy[slot] = ys[u];
                qr[slot] = w & ~BFLAG;
                if (MODE == C_LABEL) qi[slot] = (uint32_t)i;
            }
            qn += nnew;
        }
    }
    if (qn) drain(0);
    if (MODE == C_LABEL) return;

    if (LDSHIST) {
        __syncthreads();
        for (int k = threadIdx.x; k < M; k += CNT_THREADS) {
            const uint32_t c = hist[k];
            if (c) atomicAdd(&acc[k], (unsigned long long)c);
        }
    }
    __threadfence();
    __syncthreads();
    if (threadIdx.x == 0) s_last = (atomicAdd(done, 1u) == gridDim.x - 1);
    __syncthreads();
    if (!s_last) return;
    __threadfence();
    for (int k = threadIdx.x; k < M; k += CNT_THREADS) {
        out[k] = __hip_atomic_load(&acc[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        acc[k] = 0ull;
    }
    if (threadIdx.x == 0) *done = 0u;
}

// Histogram of the labels.  Each workgroup counts its share (grid-stride) in
// 16-bit counters, two to an LDS word, and stores them as one slice; no global
// atomics.  A round adds at most LH_ROUND to a counter and the thread whose
// add takes one past 2^15 - 1 moves 2^15 of it to acc before the round's
// barrier, so a counter stays below 2^15 + LH_ROUND and never carries.
constexpr int LH_THREADS = 1024;
constexpr int LH_PER = 8;                        // labels per thread and round, one 16-byte load
constexpr int LH_ROUND = LH_THREADS * LH_PER;
constexpr int64_t LABEL_MAX_POLYS = 65535;       // labels below NO_LABEL; the counters take 128 KB of LDS

__global__ __launch_bounds__(LH_THREADS) void k_label_hist(int64_t n, const uint16_t *labels, int M,
                                                           unsigned long long *acc, uint32_t *slices)
{
    static_assert(LH_ROUND < 32768, "a round must not carry out of a counter");
    extern __shared__ uint32_t lh[];
    const int nw = (M + 1) / 2;
    for (int w = threadIdx.x; w < nw; w += LH_THREADS) lh[w] = 0u;
    __syncthreads();
    for (int64_t r = (int64_t)blockIdx.x * LH_ROUND; r < n; r += (int64_t)gridDim.x * LH_ROUND) {
        const int64_t i = r + (int64_t)threadIdx.x * LH_PER;
        uint4 v = make_uint4(~0u, ~0u, ~0u, ~0u);
        if (i < n) v = *(const uint4 *)(labels + i);   // the buffer is padded to whole rounds
        const uint32_t wv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int k = 0; k < LH_PER; ++k) {
            const uint32_t lab = (wv[k / 2] >> (16 * (k & 1))) & 0xffffu;
            if (i + k < n && lab != NO_LABEL) {
                const int sh = 16 * (int)(lab & 1u);
                const uint32_t old = (atomicAdd(&lh[lab >> 1], 1u << sh) >> sh) & 0xffffu;
                if (old == 0x7fffu) {
                    atomicSub(&lh[lab >> 1], 0x8000u << sh);
                    atomicAdd(&acc[lab], 0x8000ull);
                }
            }
        }
        __syncthreads();
    }
    uint32_t *sl = slices + (size_t)blockIdx.x * nw;
    for (int w = threadIdx.x; w < nw; w += LH_THREADS) sl[w] = lh[w];
}

// out = acc + the slices' counters; acc is left zero.  64 words by 16 groups
// of slices per workgroup.
__global__ __launch_bounds__(LH_THREADS) void k_label_sum(int M, int nslice, const uint32_t *slices,
                                                          unsigned long long *acc, unsigned long long *out)
{
    constexpr int G = LH_THREADS / 64;
    __shared__ uint2 s[G][64];
    const int nw = (M + 1) / 2, lane = threadIdx.x & 63, g = threadIdx.x >> 6;
    const int w = blockIdx.x * 64 + lane;
    uint32_t a = 0u, b = 0u;
    if (w < nw)
#pragma unroll 4
        for (int k = g; k < nslice; k += G) {
            const uint32_t v = slices[(size_t)k * nw + w];
            a += v & 0xffffu;
            b += v >> 16;
        }
    s[g][lane] = make_uint2(a, b);
    __syncthreads();
    if (g >= 2) return;
    unsigned long long t = 0ull;
#pragma unroll
    for (int k = 0; k < G; ++k) t += g == 0 ? s[k][lane].x : s[k][lane].y;
    const int p = 2 * w + g;
    if (p < M) {
        out[p] = acc[p] + t;
        acc[p] = 0ull;
    }
}

static int num_cus(spade_ctx *ctx)
{
    static int cached = 0;
    if (!cached) {
        int v = 0;
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, ctx->device) != hipSuccess || v <= 0)
            v = 256;
        cached = v;
    }
    return cached;
}

// The accumulator lives in a context scratch slot that is zeroed whenever it
// is (re)allocated; k_count leaves it zeroed.
static int count_acc(spade_ctx *ctx, int64_t M, unsigned long long **acc, unsigned int **done)
{
    DevBuf &b = ctx->scratch[S_PROBE];
    const size_t need = sizeof(unsigned long long) * (size_t)(M + 1);
    if (b.cap < need) {
        if (ensure(ctx, b, need)) return SPADE_E_NOMEM;
        SPADE_HIP(ctx, hipMemsetAsync(b.p, 0, b.cap, ctx->stream));
    }
    *acc = (unsigned long long *)b.p;
    *done = (unsigned int *)((unsigned long long *)b.p + M);
    return SPADE_OK;
}

static size_t coarse_bytes_of(const CanvasView &v)
{
    return ((size_t)v.Wc * v.Hc * (v.cbyte ? 1 : 2) + 15) & ~(size_t)15;
}

// Launches the count probe with the accumulator acc[M] and the finish
// counter *done, both zero on entry and left zero by the kernels.  With
// `scratch`, more polygons than the LDS histogram holds are counted through
// labels, as far as 16 bits name them and 32 the points' indices: faster than
// the atomics from 1,000 points (38 against 53 us a call with 40,000 cells) to
// 30M (3.24 -> 0.93 ms).
static int launch_count(spade_ctx *ctx, const spade_canvas *cv, const spade_points *pts, uint64_t *out_counts,
                        unsigned long long *acc, unsigned int *done, bool scratch)
{
    hipStream_t st = ctx->stream;
    const CanvasView &v = cv->view;
    const int64_t M = v.M, n = pts->n;
    const int cus = num_cus(ctx);
    const bool ldshist = M <= HIST_MAX;
    const int64_t need = std::max<int64_t>(1, (n + CNT_THREADS * CNT_UNROLL - 1) / (CNT_THREADS * CNT_UNROLL));
    // one workgroup per CU even where the LDS would hold two: a second one
    // slows the stream down (measured), so spare LDS goes to a finer coarse
    // level instead
    const int grid = (int)std::min<int64_t>(need, (int64_t)cus);
    unsigned long long *o = (unsigned long long *)out_counts;
    uint16_t *labels = nullptr;
    uint32_t *slices = nullptr;
    const int64_t rounds = (n + LH_ROUND - 1) / LH_ROUND;
    const int hgrid = (int)std::min<int64_t>(std::max<int64_t>(rounds, 1), cus);
    const int nw = (int)((M + 1) / 2);
    // not into a caller's graph, whose replays would outlive the buffers
    if (scratch && !ldshist && M <= LABEL_MAX_POLYS && n > 0 && n <= (int64_t)0xffffffffLL && !capturing(st)) {
        DevBuf &bl = ctx->scratch[S_BITS], &bs = ctx->scratch[S_LOOKBACK];
        if (ensure(ctx, bl, sizeof(uint16_t) * (size_t)(rounds * LH_ROUND)) == SPADE_OK &&
            ensure(ctx, bs, sizeof(uint32_t) * (size_t)nw * (size_t)hgrid) == SPADE_OK) {
            labels = (uint16_t *)bl.p;
            slices = (uint32_t *)bs.p;
        } else {
            ctx->err.clear();   // without the room: an atomic per match
        }
    }
    const size_t lds = coarse_bytes_of(v) + (ldshist ? (((size_t)M * 4 + 15) & ~(size_t)15) : 0) + QUEUE_BYTES +
                       (labels ? sizeof(uint32_t) * (CNT_THREADS / 64) * QCAP : 0);
    if (lds + LDS_RESERVE > LDS_TOTAL) return set_error(ctx, SPADE_E_HIP, "internal: probe LDS budget exceeded");
    auto go = [&](auto kern) -> int {
        SPADE_HIP(ctx, hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        hipLaunchKernelGGL(kern, dim3(grid), dim3(CNT_THREADS), lds, st, v, n, pts->x, pts->y, acc, done, o, labels);
        SPADE_HIP(ctx, hipGetLastError());
        return SPADE_OK;
    };
    if (ctx->timing) SPADE_HIP(ctx, hipEventRecord(ctx->ev[2], st));
    int rc = ldshist ? go(k_count<C_LDS, CNT_UNROLL>)
                     : labels ? go(k_count<C_LABEL, CNT_UNROLL>) : go(k_count<C_ATOMIC, CNT_UNROLL>);
    if (rc) return rc;
    if (labels) {
        const size_t hl = sizeof(uint32_t) * (size_t)nw;
        SPADE_HIP(ctx, hipFuncSetAttribute((const void *)k_label_hist, hipFuncAttributeMaxDynamicSharedMemorySize, (int)hl));
        hipLaunchKernelGGL(k_label_hist, dim3(hgrid), dim3(LH_THREADS), hl, st, n, (const uint16_t *)labels, (int)M, acc,
                           slices);
        hipLaunchKernelGGL(k_label_sum, dim3((nw + 63) / 64), dim3(LH_THREADS), 0, st, (int)M, hgrid,
                           (const uint32_t *)slices, acc, o);
        SPADE_HIP(ctx, hipGetLastError());
    }
    if (ctx->timing) SPADE_HIP(ctx, hipEventRecord(ctx->ev[3], st));
    return SPADE_OK;
}

int probe_count(spade_ctx *ctx, const spade_canvas *cv, const spade_points *pts, uint64_t *out_counts)
{
    const int64_t M = cv->view.M;
    if (M == 0) return SPADE_OK;
    unsigned long long *acc = nullptr;
    unsigned int *done = nullptr;
    int rc = count_acc(ctx, M, &acc, &done);
    if (rc) return rc;
    return launch_count(ctx, cv, pts, out_counts, acc, done, true);
}

// ------------------------------------------------- stream-read reference

// Reads every point's two coordinates once (the probe's algorithmic bytes)
// and sums them, nothing else: the ceiling a point stream can reach.
// Shape 0 is the count probe's (one 1024-thread workgroup per CU, UNROLL
// points per thread in flight); shape 1 uses 256-thread workgroups, eight
// per CU.
template <int THREADS, int UNROLL>
__global__ __launch_bounds__(THREADS) void k_stream(int64_t n, const double *X, const double *Y, double *out)
{
    __shared__ double part[THREADS / 64];
    double acc = 0.0;
    const int64_t step = (int64_t)gridDim.x * THREADS * UNROLL;
    for (int64_t b = (int64_t)blockIdx.x * THREADS * UNROLL; b < n; b += step) {
        double xs[UNROLL], ys[UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            const int64_t i = b + (int64_t)u * THREADS + threadIdx.x;
            xs[u] = i < n ? __builtin_nontemporal_load(X + i) : 0.0;
            ys[u] = i < n ? __builtin_nontemporal_load(Y + i) : 0.0;
        }
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) acc += xs[u] + ys[u];
    }
    for (int d = 32; d > 0; d >>= 1) acc += __shfl_xor(acc, d, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int w = 0; w < THREADS / 64; ++w) t += part[w];
        atomicAdd(out, t);
    }
}

int stream_read(spade_ctx *ctx, const spade_points *pts, int shape, double *out)
{
    hipStream_t st = ctx->stream;
    const int cus = num_cus(ctx);
    if (ctx->timing) SPADE_HIP(ctx, hipEventRecord(ctx->ev[2], st));
    if (shape == 0) {
        const int64_t need = std::max<int64_t>(1, (pts->n + 1024 * 8 - 1) / (1024 * 8));
        hipLaunchKernelGGL((k_stream<1024, 8>), dim3((int)std::min<int64_t>(need, cus)), dim3(1024), 0, st, pts->n,
                           pts->x, pts->y, out);
    } else {
        const int64_t need = std::max<int64_t>(1, (pts->n + 256 * 8 - 1) / (256 * 8));
        hipLaunchKernelGGL((k_stream<256, 8>), dim3((int)std::min<int64_t>(need, (int64_t)cus * 8)), dim3(256), 0,
                           st, pts->n, pts->x, pts->y, out);
    }
    SPADE_HIP(ctx, hipGetLastError());
    if (ctx->timing) SPADE_HIP(ctx, hipEventRecord(ctx->ev[3], st));
    return SPADE_OK;
}

// ------------------------------------------------- join-count without allocation
//
// The count probe's only scratch is its accumulator (one u64 per polygon)
// and finish counter.  For callers that cannot allocate device memory they
// live in a fixed array of this source file instead of a context slot.  Its
// device address differs per GPU and is looked up once per device when a
// context is created there; host code passes that address, never the
// array's own name.  Calls that overlap on one GPU share the array and race.
constexpr int64_t NOALLOC_MAX_POLYS = 65536;
static __device__ __align__(256) unsigned long long scratch[NOALLOC_MAX_POLYS + 1];
constexpr int MAX_DEVICES = 64;
static void *g_scratch_ptr[MAX_DEVICES];
static std::mutex g_scratch_mu;

int noalloc_init(spade_ctx *ctx)
{
    if (ctx->device < 0 || ctx->device >= MAX_DEVICES)
        return set_error(ctx, SPADE_E_UNSUPPORTED, "device index beyond the library's table");
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (g_scratch_ptr[ctx->device]) return SPADE_OK;
    void *p = nullptr;
    hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) {
        (void)hipGetLastError();
        return set_error(ctx, SPADE_E_HIP, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
    }
    g_scratch_ptr[ctx->device] = p;
    return SPADE_OK;
}

__global__ void k_fill_u64(int64_t n, unsigned long long *p)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0ull;
}

int probe_count_noalloc(spade_ctx *ctx, const spade_canvas *cv, const spade_points *pts, uint64_t *out_counts)
{
    const int64_t M = cv->view.M;
    if (M > NOALLOC_MAX_POLYS)
        return set_error(ctx, SPADE_E_UNSUPPORTED,
                         "join-count without allocation supports at most 65536 polygons");
    if (M == 0) return SPADE_OK;
    void *base = nullptr;
    {
        std::lock_guard<std::mutex> lk(g_scratch_mu);
        base = g_scratch_ptr[ctx->device];
    }
    if (!base) return set_error(ctx, SPADE_E_HIP, "scratch address of the device was not looked up");
    unsigned long long *acc = (unsigned long long *)base;
    unsigned int *done = (unsigned int *)(acc + M);
    // the array keeps the last call's contents: clear what must start at
    // zero with a kernel (no memset node, so the call can be captured)
    hipLaunchKernelGGL(k_fill_u64, dim3((unsigned)std::min<int64_t>((M + 256) / 256, 256)), dim3(256), 0,
                       ctx->stream, M + 1, acc);
    SPADE_HIP(ctx, hipGetLastError());
    return launch_count(ctx, cv, pts, out_counts, acc, done, false);
}

// ------------------------------------------------------------ ordered emit

// Write pass that probes again, for canvases in which the count pass met a
// point in several polygons.  Every wavefront owns segments of EMIT_SEG consecutive points
// (grid-stride over segments), EMIT_WGROUP points per lane in flight at a
// time.  The boundary points of a group are queued in LDS and tested a full
// wavefront at a time (as in k_count); each lane then takes the results of
// its own queued points back with a shuffle.  The entries of segment s are
// written in point order (ascending polygon order for a point in several
// polygons) from position offs[s] on; positions at or beyond cap are not
// written.  No barriers after the coarse canvas is loaded.
__global__ __launch_bounds__(EMIT_THREADS) void k_emit(CanvasView cv, int64_t n, const double *X,
                                                       const double *Y, int64_t nseg,
                                                       const unsigned long long *offs, uint32_t *out_pt,
                                                       uint32_t *out_poly, int64_t cap, const unsigned *multi)
{
    static_assert(EMIT_THREADS == CNT_THREADS, "the queue area is sized for CNT_THREADS");
    if (*multi == 0u) return;   // k_emit_labels has written the pairs
    extern __shared__ __align__(16) unsigned char smem[];
    uint16_t *coarse = (uint16_t *)smem;
    const size_t coarse_bytes = ((size_t)cv.Wc * cv.Hc * (cv.cbyte ? 1 : 2) + 15) & ~(size_t)15;
    unsigned char *qbase = smem + coarse_bytes;
    const int wv = threadIdx.x >> 6;
    double *qx = (double *)(qbase) + wv * QCAP;
    double *qy = (double *)(qbase) + (EMIT_THREADS / 64) * QCAP + wv * QCAP;
    uint32_t *qr = (uint32_t *)((double *)(qbase) + 2 * (EMIT_THREADS / 64) * QCAP) + wv * QCAP;
    load_coarse(cv, coarse, EMIT_THREADS);
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const unsigned long long below = (1ull << lane) - 1ull;
    const int64_t nwave = ((int64_t)gridDim.x * EMIT_THREADS) >> 6;
    for (int64_t sg = ((int64_t)blockIdx.x * EMIT_THREADS + threadIdx.x) >> 6; sg < nseg; sg += nwave) {
        const int64_t i0 = sg * EMIT_SEG + lane;
        unsigned long long pos = offs[sg];
        // EMIT_WDRAIN words share one boundary queue (drained when full and
        // at their end); their points are loaded EMIT_WGROUP words at a time
        for (int g0 = 0; g0 < EMIT_SEG / 64; g0 += EMIT_WDRAIN) {
            // per word: the entry count (the queue slot while its boundary
            // point waits in the queue) and the label or first record
            uint32_t cs[EMIT_WDRAIN], lab[EMIT_WDRAIN];
            uint32_t qn = 0, pend = 0;   // wave-uniform: queue length, words queued
            uint32_t mine = 0;           // words whose point of this lane is queued
            auto drain = [&]() {
                __builtin_amdgcn_wave_barrier();
                uint32_t m = 0, first = 0, rec0 = 0;
                if (lane < (int)qn) {
                    const double x = qx[lane], y = qy[lane];
                    rec0 = qr[lane];
                    uint32_t rec = rec0;
                    while (true) {   // two records at a time (the slot after the last exists)
                        const Cand c0 = cv.cands[rec];
                        const Cand c1 = cv.cands[rec + 1];
                        if (cand_inside(cv, c0, x, y)) { if (m == 0) first = c0.poly; ++m; }
                        if (c0.meta & CAND_LAST) break;
                        if (cand_inside(cv, c1, x, y)) { if (m == 0) first = c1.poly; ++m; }
                        if (c1.meta & CAND_LAST) break;
                        rec += 2;
                    }
                }
                __builtin_amdgcn_wave_barrier();
                const uint32_t rl = m == 1 ? first : (m > 1 ? rec0 : 0u);
#pragma unroll
                for (int k = 0; k < EMIT_WDRAIN; ++k) {
                    if (!(pend & (1u << k))) continue;
                    const int from = (mine & (1u << k)) ? (int)cs[k] : 0;
                    const uint32_t c = (uint32_t)__shfl((int)m, from, 64);
                    const uint32_t l = (uint32_t)__shfl((int)rl, from, 64);
                    if (mine & (1u << k)) { cs[k] = c; lab[k] = l; }
                }
                pend = 0;
                mine = 0;
                qn = 0;
            };
#pragma unroll
            for (int g = 0; g < EMIT_WDRAIN; g += EMIT_WGROUP) {
                // the group's points, then their canvas words, level by level
                double xs[EMIT_WGROUP], ys[EMIT_WGROUP];
#pragma unroll
                for (int k = 0; k < EMIT_WGROUP; ++k) {
                    const int64_t i = i0 + 64 * (g0 + g + k);
                    xs[k] = i < n ? __builtin_nontemporal_load(X + i) : NAN;   // NaN: outside
                    ys[k] = i < n ? __builtin_nontemporal_load(Y + i) : NAN;
                }
                uint32_t ws[EMIT_WGROUP];
#pragma unroll
                for (int k = 0; k < EMIT_WGROUP; ++k) {
                    const Look lk = look_coarse(cv, coarse, xs[k], ys[k]);
                    ws[k] = lk.full ? ((gu32p)cv.cells)[lk.fidx] : lk.word;
                }
                // matches of every point: interior words at once, boundary
                // points through the queue
#pragma unroll
                for (int k = 0; k < EMIT_WGROUP; ++k) {
                    const int kk = g + k;
                    const uint32_t w = ws[k];
                    const bool bnd = (w & BFLAG) != 0;
                    cs[kk] = (w != 0u && !bnd) ? 1u : 0u;
                    lab[kk] = (w != 0u && !bnd) ? w - 1u : 0u;
                    const unsigned long long mask = __ballot(bnd);
                    const uint32_t nnew = (uint32_t)__popcll(mask);
                    if (nnew == 0) continue;
                    if (qn + nnew > QCAP) drain();
                    if (bnd) {
                        const uint32_t sl = qn + (uint32_t)__popcll(mask & below);
                        qx[sl] = xs[k];
                        qy[sl] = ys[k];
                        qr[sl] = w & ~BFLAG;
                        cs[kk] = sl;
                        mine |= 1u << kk;
                    }
                    qn += nnew;
                    pend |= 1u << kk;
                }
            }
            if (qn) drain();
#pragma unroll
            for (int k = 0; k < EMIT_WDRAIN; ++k) {
                // inclusive scan of the entry counts across the wavefront
                const uint32_t cnt = cs[k];
                uint32_t inc = cnt;
#pragma unroll
                for (int d = 1; d < 64; d <<= 1) {
                    const uint32_t t = __shfl_up(inc, d, 64);
                    if (lane >= d) inc += t;
                }
                const uint32_t tot = __shfl(inc, 63, 64);
                if (cnt) {
                    const int64_t i = i0 + 64 * (g0 + k);
                    const uint32_t pt = (uint32_t)i;
                    unsigned long long p = pos + (inc - cnt);
                    if (cnt == 1) {
                        if ((int64_t)p < cap) {
                            out_pt[p] = pt;
                            if (out_poly) out_poly[p] = lab[k];
                        }
                    } else if ((int64_t)p < cap) {
                        // several polygons: the smallest L of them (all when
                        // below cap), ascending, kept in out_poly[p, p + L)
                        // by insertion during one pass over the pixel's
                        // records (this lane's own range, read back by this
                        // lane only)
                        const uint32_t L = (int64_t)(p + cnt) <= cap ? cnt : (uint32_t)(cap - (int64_t)p);
                        if (out_poly) {
                            const double x = X[i], y = Y[i];
                            uint32_t rec = lab[k], j = 0;
                            while (true) {
                                const Cand cd = cv.cands[rec];
                                if (cand_inside(cv, cd, x, y)) {
                                    const uint32_t v = cd.poly;
                                    uint32_t at = j;
                                    if (j < L) ++j;
                                    else at = out_poly[p + L - 1] > v ? L - 1 : L;   // L: v is not kept
                                    if (at < L) {
                                        while (at > 0) {
                                            const uint32_t u = out_poly[p + at - 1];
                                            if (u < v) break;
                                            out_poly[p + at] = u;
                                            --at;
                                        }
                                        out_poly[p + at] = v;
                                    }
                                }
                                if (cd.meta & CAND_LAST) break;
                                ++rec;
                            }
                        }
                        for (uint32_t t = 0; t < L; ++t) out_pt[p + t] = pt;
                    }
                }
                pos += tot;
            }
        }
    }
}

// The labels of a group of 64 * EMIT_GROUP points lie lane by lane, so that a
// lane's EMIT_GROUP labels are one store of the count pass (128-byte stores of
// a word's labels had the pass wait for its stores: 477 us for 50M points)
// and one load of the write pass.
template <typename T>
struct alignas(16) LabelVec {
    T l[EMIT_GROUP];
};

// Count pass with the boundary points of a wavefront queued in LDS and
// tested a full wavefront at a time (as in k_count): counts[s] = output
// entries of segment s.  The same records and the same test as k_emit,
// so the counts match what the write pass writes.  While *multi is clear,
// labels keeps every point's polygon (all ones: none), so that the write pass
// reads 2 or 4 bytes per point instead of the points and the canvas again; a
// point in several polygons sets *multi, and the labels are not used.  Bound
// by the latency of the points and their cells, as k_count: 100M points, 64
// polygons on a 2048 canvas, 0.37 ms (0.31 without the labels, whose 0.2 GB
// save the write pass 0.38 ms).
template <typename T, bool LABELS>
__global__ __launch_bounds__(EMIT_THREADS) void k_emit_count(CanvasView cv, int64_t n, const double *X,
                                                             const double *Y, int64_t nseg,
                                                             unsigned long long *counts, unsigned *multi, T *labels,
                                                             const unsigned *skip)
{
    static_assert(EMIT_THREADS == CNT_THREADS, "the queue area is sized for CNT_THREADS");
    static_assert(EMIT_SEG <= 65536 && EMIT_INDEX_BYTES <= LDS_RESERVE, "the queued points' places fit the reserve");
    if (LABELS == (*skip != 0u)) return;
    extern __shared__ __align__(16) unsigned char smem[];
    uint16_t *coarse = (uint16_t *)smem;
    const size_t coarse_bytes = ((size_t)cv.Wc * cv.Hc * (cv.cbyte ? 1 : 2) + 15) & ~(size_t)15;
    unsigned char *qbase = smem + coarse_bytes;
    const int wv = threadIdx.x >> 6;
    double *qx = (double *)(qbase) + wv * QCAP;
    double *qy = (double *)(qbase) + (EMIT_THREADS / 64) * QCAP + wv * QCAP;
    uint32_t *qr = (uint32_t *)((double *)(qbase) + 2 * (EMIT_THREADS / 64) * QCAP) + wv * QCAP;
    uint16_t *qi = (uint16_t *)(qbase + QUEUE_BYTES) + wv * QCAP;   // the points' places in the segment
    load_coarse(cv, coarse, EMIT_THREADS);
    __syncthreads();
    const uint32_t lane = lane_id();
    const unsigned long long below = (1ull << lane) - 1ull;
    const int64_t nwave = ((int64_t)gridDim.x * EMIT_THREADS) >> 6;
    bool several = false;   // a point lies in several polygons
    for (int64_t sg = ((int64_t)blockIdx.x * EMIT_THREADS + threadIdx.x) >> 6; sg < nseg; sg += nwave) {
        const int64_t i0 = sg * EMIT_SEG + lane;
        // whole segments: no bounds to check; none once the labels are known
        // not to be used
        if (LABELS) several = several || __hip_atomic_load(multi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u;
        T *seg = !LABELS || several ? nullptr : labels + sg * EMIT_SEG;
        unsigned long long total = 0;   // wave-uniform
        uint32_t qn = 0;                // wave-uniform queue length
        auto drain = [&]() {
            __builtin_amdgcn_wave_barrier();
            uint32_t m = 0;
            if (lane < qn) {
                const double x = qx[lane], y = qy[lane];
                uint32_t rec = qr[lane], first = ~0u;
                if (LABELS) {   // one record at a time: two spill registers
                    while (true) {
                        const Cand c0 = cv.cands[rec];
                        if (cand_inside(cv, c0, x, y)) { ++m; first = c0.poly; }
                        if (c0.meta & CAND_LAST) break;
                        ++rec;
                    }
                } else {
                    test_records(cv, rec, x, y, [&](uint32_t) { ++m; });
                }
                // after the group's own store: one wavefront's stores to
                // an address keep their order under the fence
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
                if (LABELS && seg) seg[qi[lane]] = (T)first;
            }
            __builtin_amdgcn_wave_barrier();
            // a point in several polygons: the write pass probes again (told
            // once per wavefront: the stores of all of them meet in one place)
            if (LABELS && !several && __ballot(m > 1u)) {
                several = true;
                if (lane == 0) __hip_atomic_store(multi, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) m += __shfl_xor(m, d, 64);
            total += m;
            qn = 0;
        };
        for (int g = 0; g < EMIT_SEG / 64; g += EMIT_GROUP) {
            double xs[EMIT_GROUP], ys[EMIT_GROUP];
#pragma unroll
            for (int k = 0; k < EMIT_GROUP; ++k) {
                const int64_t i = i0 + 64 * (g + k);
                xs[k] = i < n ? __builtin_nontemporal_load(X + i) : NAN;   // NaN: outside
                ys[k] = i < n ? __builtin_nontemporal_load(Y + i) : NAN;
            }
            uint32_t ws[EMIT_GROUP];
#pragma unroll
            for (int k = 0; k < EMIT_GROUP; ++k) {
                const Look lk = look_coarse(cv, coarse, xs[k], ys[k]);
                ws[k] = lk.full ? ((gu32p)cv.cells)[lk.fidx] : lk.word;
            }
            if (LABELS && seg) {   // a boundary point's label is stored by its drain
                LabelVec<T> v;
#pragma unroll
                for (int k = 0; k < EMIT_GROUP; ++k) v.l[k] = (T)(ws[k] - 1u);   // word 0: all ones
                *(LabelVec<T> *)(seg + 64 * g + EMIT_GROUP * lane) = v;
            }
#pragma unroll
            for (int k = 0; k < EMIT_GROUP; ++k) {
                const uint32_t w = ws[k];
                const bool bnd = (w & BFLAG) != 0;
                total += (unsigned long long)__popcll(__ballot(w != 0u && !bnd));
                const unsigned long long mask = __ballot(bnd);
                const uint32_t nnew = (uint32_t)__popcll(mask);
                if (nnew == 0) continue;
                if (qn + nnew > QCAP) drain();
                if (bnd) {
                    const uint32_t slot = qn + (uint32_t)__popcll(mask & below);
                    qx[slot] = xs[k];
                    qy[slot] = ys[k];
                    qr[slot] = w & ~BFLAG;
                    if (LABELS) qi[slot] = (uint16_t)(64 * g + EMIT_GROUP * lane + k);
                }
                qn += nnew;
            }
        }
        if (qn) drain();
        if (lane == 0) counts[sg] = total;
    }
}

// Write pass from the count pass's labels, when no point lies in several
// polygons: a wavefront takes a segment, all its labels in flight, and stores
// the pairs of a word to consecutive positions from offs[segment] on (below
// cap).  Bound by HBM: 50M pairs (0.1 GB read, 0.4 GB written) in 0.10 ms,
// where the pass that read the points and the canvas again took 0.48 ms.
template <typename T>
__global__ __launch_bounds__(256) void k_emit_labels(int64_t nseg, const unsigned long long *offs, const T *labels,
                                                     const unsigned *multi, uint32_t *out_pt, uint32_t *out_poly,
                                                     int64_t cap)
{
    if (*multi != 0u) return;   // k_emit writes the pairs
    constexpr int NW = EMIT_SEG / 64;
    const int lane = threadIdx.x & 63;
    const unsigned long long below = (1ull << lane) - 1ull;
    const int64_t nwave = ((int64_t)gridDim.x * blockDim.x) >> 6;
    for (int64_t sg = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6; sg < nseg; sg += nwave) {
        LabelVec<T> v[NW / EMIT_GROUP];
#pragma unroll
        for (int j = 0; j < NW / EMIT_GROUP; ++j)
            v[j] = *(const LabelVec<T> *)(labels + sg * EMIT_SEG + EMIT_GROUP * (64 * j + lane));
        int64_t pos = (int64_t)offs[sg];
#pragma unroll
        for (int j = 0; j < NW; ++j) {
            const T lab = v[j / EMIT_GROUP].l[j % EMIT_GROUP];
            const bool on = lab != (T)~(T)0;
            const unsigned long long m = __ballot(on);
            const int64_t p = pos + __popcll(m & below);
            if (on && p < cap) {
                out_pt[p] = (uint32_t)(sg * EMIT_SEG + 64 * j + lane);
                if (out_poly) out_poly[p] = (uint32_t)lab;
            }
            pos += __popcll(m);
        }
    }
}

// Count pass for a canvas of one polygon (a point matches at most once)
// that also keeps every point's result, so that the write pass reads bits
// instead of the points: bits[sg * (EMIT_SEG / 64) + j] holds the matches of
// points sg * EMIT_SEG + 64 j + lane (bit = lane).  Boundary points are
// queued and tested a wavefront at a time as in k_emit; each lane takes its
// own points' results back with a shuffle.
__global__ __launch_bounds__(EMIT_THREADS) void k_emit_count_bits(CanvasView cv, int64_t n, const double *X,
                                                                  const double *Y, int64_t nseg,
                                                                  unsigned long long *counts,
                                                                  unsigned long long *bits)
{
    static_assert(EMIT_THREADS == CNT_THREADS, "the queue area is sized for CNT_THREADS");
    static_assert(EMIT_SEG / 64 <= 64, "a segment's words are held one per lane");
    extern __shared__ __align__(16) unsigned char smem[];
    uint16_t *coarse = (uint16_t *)smem;
    const size_t coarse_bytes = ((size_t)cv.Wc * cv.Hc * (cv.cbyte ? 1 : 2) + 15) & ~(size_t)15;
    unsigned char *qbase = smem + coarse_bytes;
    const int wv = threadIdx.x >> 6;
    double *qx = (double *)(qbase) + wv * QCAP;
    double *qy = (double *)(qbase) + (EMIT_THREADS / 64) * QCAP + wv * QCAP;
    uint32_t *qr = (uint32_t *)((double *)(qbase) + 2 * (EMIT_THREADS / 64) * QCAP) + wv * QCAP;
    load_coarse(cv, coarse, EMIT_THREADS);
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const unsigned long long below = (1ull << lane) - 1ull;
    const int64_t nwave = ((int64_t)gridDim.x * EMIT_THREADS) >> 6;
    for (int64_t sg = ((int64_t)blockIdx.x * EMIT_THREADS + threadIdx.x) >> 6; sg < nseg; sg += nwave) {
        const int64_t i0 = sg * EMIT_SEG + lane;
        unsigned long long total = 0;   // wave-uniform
        unsigned long long segw = 0;    // lane j < EMIT_SEG / 64: the word of points 64 j ..
        // the segment's words share one boundary queue (drained when full
        // and at the segment's end); points are loaded EMIT_WGROUP words at
        // a time
        constexpr int NW = EMIT_SEG / 64;
        uint32_t hit = 0, slot[NW];   // hit: bit k for this lane's point of word k
        uint32_t qn = 0, pend = 0, mine = 0;
        auto drain = [&]() {
            __builtin_amdgcn_wave_barrier();
            uint32_t m = 0;
            if (lane < (int)qn) {
                const double x = qx[lane], y = qy[lane];
                uint32_t rec = qr[lane];
                while (true) {
                    const Cand c0 = cv.cands[rec];
                    if (cand_inside(cv, c0, x, y)) m = 1u;
                    if (c0.meta & CAND_LAST) break;
                    ++rec;
                }
            }
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int k = 0; k < NW; ++k) {
                if (!(pend & (1u << k))) continue;
                const uint32_t c = (uint32_t)__shfl((int)m, (int)slot[k], 64);
                if ((mine & (1u << k)) && c) hit |= 1u << k;
            }
            pend = 0;
            mine = 0;
            qn = 0;
        };
#pragma unroll
        for (int g = 0; g < NW; g += EMIT_WGROUP) {
            double xs[EMIT_WGROUP], ys[EMIT_WGROUP];
#pragma unroll
            for (int k = 0; k < EMIT_WGROUP; ++k) {
                const int64_t i = i0 + 64 * (g + k);
                xs[k] = i < n ? __builtin_nontemporal_load(X + i) : NAN;   // NaN: outside
                ys[k] = i < n ? __builtin_nontemporal_load(Y + i) : NAN;
            }
            uint32_t ws[EMIT_WGROUP];
#pragma unroll
            for (int k = 0; k < EMIT_WGROUP; ++k) {
                const Look lk = look_coarse(cv, coarse, xs[k], ys[k]);
                ws[k] = lk.full ? ((gu32p)cv.cells)[lk.fidx] : lk.word;
            }
#pragma unroll
            for (int k = 0; k < EMIT_WGROUP; ++k) {
                const int kk = g + k;
                const uint32_t w = ws[k];
                const bool bnd = (w & BFLAG) != 0;
                if (w != 0u && !bnd) hit |= 1u << kk;
                slot[kk] = 0;
                const unsigned long long mask = __ballot(bnd);
                const uint32_t nnew = (uint32_t)__popcll(mask);
                if (nnew == 0) continue;
                if (qn + nnew > QCAP) drain();
                if (bnd) {
                    const uint32_t sl = qn + (uint32_t)__popcll(mask & below);
                    qx[sl] = xs[k];
                    qy[sl] = ys[k];
                    qr[sl] = w & ~BFLAG;
                    slot[kk] = sl;
                    mine |= 1u << kk;
                }
                qn += nnew;
                pend |= 1u << kk;
            }
        }
        if (qn) drain();
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            const unsigned long long word = __ballot((hit >> k) & 1u);
            total += (unsigned long long)__popcll(word);
            if (lane == k) segw = word;
        }
        if (lane < EMIT_SEG / 64) bits[sg * (EMIT_SEG / 64) + lane] = segw;
        if (lane == 0) counts[sg] = total;
    }
}

// Write pass from the count pass's bits: each wavefront takes segments and
// walks a segment's words in point order; lane l writes point 64 j + l of
// word j, so the ids of a word are stored to consecutive positions (below
// cap; polygon 0 into out_poly), from offs[segment] on.
__global__ __launch_bounds__(256) void k_emit_bits(int64_t nseg, const unsigned long long *offs,
                                                   const unsigned long long *bits, uint32_t *out_pt,
                                                   uint32_t *out_poly, int64_t cap)
{
    const int lane = threadIdx.x & 63;
    const unsigned long long below = (1ull << lane) - 1ull;
    const int64_t nwave = ((int64_t)gridDim.x * blockDim.x) >> 6;
    for (int64_t sg = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6; sg < nseg; sg += nwave) {
        int64_t pos = (int64_t)offs[sg];
        const unsigned long long mine = lane < EMIT_SEG / 64 ? bits[sg * (EMIT_SEG / 64) + lane] : 0ull;
        for (int j = 0; j < EMIT_SEG / 64; ++j) {
            const unsigned long long word = (unsigned long long)__shfl((long long)mine, j, 64);
            if (!word) continue;   // uniform over the wavefront
            if ((word >> lane) & 1ull) {
                const int64_t p = pos + __popcll(word & below);
                if (p < cap) {
                    out_pt[p] = (uint32_t)(sg * EMIT_SEG + 64 * j + lane);
                    if (out_poly) out_poly[p] = 0u;
                }
            }
            pos += __popcll(word);
        }
    }
}

// Clears the count behind the last segment, whose scan is the total, and says
// whether the pairs' count pass keeps labels: p[0], set later by a point in
// several polygons, and p[1] start at 0 if so, else at 1.  No labels where the
// pixels that the raster found inside several polygons would hold one of n
// evenly spread points: the write pass would have to probe again, and the count
// pass without labels is the faster one (12 overlapping polygons, 30M points:
// 224 us, with labels 344; the call 940 us and 1,055).  Everywhere else they
// pay, however many of the pixels are boundary ones (calls of 30M points: 260
// zones, 5 % of the pixels, 660 us with labels and 930 probing twice; 29 %, 2.1
// and 4.0 ms; 40,000 cells, 14 %, 7.1 and 13.2 ms; 40,000 rectangles of a pixel
// each, 1.9 and 3.1 ms).  One wavefront; over: the counters of a build not read
// yet, else null.
__global__ __launch_bounds__(64) void k_emit_start(unsigned long long *end, unsigned *p, int labelled,
                                                   const unsigned long long *over, int shards, int stride,
                                                   unsigned long long known, unsigned long long n,
                                                   unsigned long long pixels)
{
    if (over) {
        known = 0ull;
        for (int k = threadIdx.x; k < shards; k += 64) known += over[k * stride];
        for (int d = 32; d > 0; d >>= 1) known += (unsigned long long)__shfl_xor((long long)known, d, 64);
    }
    if (threadIdx.x != 0) return;
    *end = 0ull;
    if (p) p[0] = p[1] = labelled && known * n < pixels ? 0u : 1u;
}

int probe_emit(spade_ctx *ctx, const spade_canvas *cv, const spade_points *pts, uint32_t *out_pt,
               uint32_t *out_poly, int64_t cap, int64_t *n_out)
{
    hipStream_t st = ctx->stream;
    const int64_t n = pts->n;
    *n_out = 0;
    if (n == 0 || cv->view.M == 0) return SPADE_OK;
    const int64_t nseg = (n + EMIT_SEG - 1) / EMIT_SEG;
    DevBuf &lb = ctx->scratch[S_LOOKBACK];
    if (ensure(ctx, lb, sizeof(unsigned long long) * (2 * (size_t)(nseg + 1) + 1))) return SPADE_E_NOMEM;
    unsigned long long *counts = (unsigned long long *)lb.p;
    unsigned long long *offs = counts + (nseg + 1);
    unsigned *multi = (unsigned *)(offs + (nseg + 1));   // set by the count pass: a point in several polygons
    const size_t lds = coarse_bytes_of(cv->view);
    if (lds + QUEUE_BYTES + LDS_RESERVE > LDS_TOTAL)
        return set_error(ctx, SPADE_E_HIP, "internal: emit probe LDS budget exceeded");
    const int per_cu = std::max<int>(1, (int)(LDS_TOTAL / (lds + LDS_RESERVE)));
    const int cus = num_cus(ctx);
    const int64_t wpb = EMIT_THREADS / 64;
    const int grid = (int)std::max<int64_t>(1, std::min<int64_t>((nseg + wpb - 1) / wpb, (int64_t)cus * std::min(per_cu, 2)));
    // a canvas of one polygon keeps every point's result in the count pass
    // (one bit per point), so that the write pass need not read the points
    unsigned long long *bits = nullptr;
    if (cv->view.M == 1 && cap > 0) {
        DevBuf &bb = ctx->scratch[S_BITS];
        if (ensure(ctx, bb, sizeof(unsigned long long) * (EMIT_SEG / 64) * (size_t)nseg) == SPADE_OK)
            bits = (unsigned long long *)bb.p;
        else
            ctx->err.clear();   // read the points twice instead
    }
    // other canvases keep every point's polygon, in 16 bits where they name it
    uint16_t *lab16 = nullptr;
    uint32_t *lab32 = nullptr;
    if (!bits && cap > 0) {
        DevBuf &bb = ctx->scratch[S_BITS];
        const bool narrow = cv->view.M < 65536;
        if (ensure(ctx, bb, (narrow ? 2 : 4) * (size_t)EMIT_SEG * (size_t)nseg) == SPADE_OK) {
            if (narrow) lab16 = (uint16_t *)bb.p;
            else lab32 = (uint32_t *)bb.p;
        } else {
            ctx->err.clear();   // probe twice instead
        }
    }
    const bool labelled = lab16 || lab32;
    auto launch = [&](auto kern, size_t bytes, auto... args) -> int {
        SPADE_HIP(ctx, hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes));
        hipLaunchKernelGGL(kern, dim3(grid), dim3(EMIT_THREADS), bytes, st, cv->view, n, pts->x, pts->y, nseg, args...);
        SPADE_HIP(ctx, hipGetLastError());
        return SPADE_OK;
    };
    int rc = SPADE_OK, shards = 0, stride = 0;
    if (ctx->timing) SPADE_HIP(ctx, hipEventRecord(ctx->ev[2], st));
    const unsigned long long *over = bits ? nullptr : build_overlap(cv, &shards, &stride);
    hipLaunchKernelGGL(k_emit_start, dim3(1), dim3(64), 0, st, counts + nseg, bits ? nullptr : multi, labelled ? 1 : 0, over,
                       shards, stride, (unsigned long long)cv->n_overlap, (unsigned long long)n,
                       (unsigned long long)cv->view.W * (unsigned long long)cv->view.H);
    SPADE_HIP(ctx, hipGetLastError());
    if (bits) {
        rc = launch(k_emit_count_bits, lds + QUEUE_BYTES, counts, bits);
    } else {   // the pass that is not chosen returns at once
        const size_t qb = lds + QUEUE_BYTES;
        const unsigned *skip = multi + 1;
        if (lab16) rc = launch(k_emit_count<uint16_t, true>, qb + EMIT_INDEX_BYTES, counts, multi, lab16, skip);
        if (lab32) rc = launch(k_emit_count<uint32_t, true>, qb + EMIT_INDEX_BYTES, counts, multi, lab32, skip);
        if (!rc) rc = launch(k_emit_count<uint16_t, false>, qb, counts, multi, lab16, skip);
    }
    if (rc) return rc;
    DevBuf &cub = ctx->scratch[S_CUBTMP];
    size_t tb = 0;
    SPADE_HIP(ctx, hipcub::DeviceScan::ExclusiveSum(nullptr, tb, counts, offs, (int)(nseg + 1), st));
    if (ensure(ctx, cub, std::max<size_t>(tb, 1))) return SPADE_E_NOMEM;
    SPADE_HIP(ctx, hipcub::DeviceScan::ExclusiveSum(cub.p, tb, counts, offs, (int)(nseg + 1), st));
    if (cap > 0 && bits) {
        const int bg = (int)std::max<int64_t>(1, std::min<int64_t>((nseg + 3) / 4, (int64_t)cus * 16));
        hipLaunchKernelGGL(k_emit_bits, dim3(bg), dim3(256), 0, st, nseg, offs, bits, out_pt, out_poly, cap);
        SPADE_HIP(ctx, hipGetLastError());
    } else if (cap > 0) {
        const int bg = (int)std::max<int64_t>(1, std::min<int64_t>((nseg + 3) / 4, (int64_t)cus * 16));
        if (lab16)
            hipLaunchKernelGGL(k_emit_labels<uint16_t>, dim3(bg), dim3(256), 0, st, nseg, (const unsigned long long *)offs,
                               (const uint16_t *)lab16, (const unsigned *)multi, out_pt, out_poly, cap);
        if (lab32)
            hipLaunchKernelGGL(k_emit_labels<uint32_t>, dim3(bg), dim3(256), 0, st, nseg, (const unsigned long long *)offs,
                               (const uint32_t *)lab32, (const unsigned *)multi, out_pt, out_poly, cap);
        if ((rc = launch(k_emit, lds + QUEUE_BYTES, (const unsigned long long *)offs, out_pt, out_poly, cap,
                         (const unsigned *)multi)))
            return rc;
    }
    if (ctx->timing) SPADE_HIP(ctx, hipEventRecord(ctx->ev[3], st));
    unsigned long long *h = (unsigned long long *)ensure_pinned(ctx, 64);
    if (!h) return set_error(ctx, SPADE_E_NOMEM, "pinned staging allocation failed");
    SPADE_HIP(ctx, hipMemcpyAsync(h, offs + nseg, sizeof(unsigned long long), hipMemcpyDeviceToHost, st));
    SPADE_HIP(ctx, hipStreamSynchronize(st));
    *n_out = (int64_t)h[0];
    if (*n_out > cap) return set_error(ctx, SPADE_E_CAPACITY, "output capacity too small");
    return SPADE_OK;
}

}  // namespace spade
