// Distance selection from lines and from a polygon: the rounded rectangles
// of Sec. 4.2 (every position within distance r of a segment) drawn around
// every segment of a set of polylines, or around every edge of a polygon
// together with the polygon itself, and the distance selection of Sec. 5.2
// over that shape.
//
// Instead of rasterising the rounded rectangles, the segments are binned
// into a uniform grid over their box widened by r: a cell that lies wholly
// within r of a segment is full, any other lists every segment that may be
// within r of one of its points (count, scan, fill).  One pass over the
// points then keeps, per 1024-point segment of the stream, one result bit
// per point: for a polygon, the canvas of the polygon answers first (coarse
// level in LDS, full canvas, exact records, as the selection probe does);
// a point not yet kept that lies in the grid's box is kept in a full cell, and
// tested exactly against the segments that another cell lists, until one is
// within r.  The tests of a
// wavefront's 64 points are spread over its lanes (buf_wave_walk), so that a
// wavefront takes about as many rounds as its points have candidates in
// total / 64 rather than as many as its longest list.  The ordered ids are
// then written from the bits (the two-step Map of the selection).
#include "common.h"
#include "lookup.h"
#include "segdist.h"
#include "wavewalk.h"

#include <hipcub/hipcub.hpp>
#include <rocprim/rocprim.hpp>

#include <algorithm>
#include <cmath>
#include <cstring>

namespace spade {

constexpr int BUF_GRID_MAX = 4096;            // cells per side
constexpr double BUF_FINE = 2.0;              // finest cell: the distance over this
constexpr double BUF_PER_CELL = 4.0;          // points per cell of a fine grid, at least
constexpr double BUF_PER_ENTRY = 8.0;         // points per list entry of a fine grid, at least
constexpr int64_t BUF_FILTER_MIN = 1 << 20;   // points from which a pass without exact tests pays for its launch (5 us)
constexpr int BUF_THREADS = 1024;
constexpr int BUF_WORDS = EMIT_SEG / 64;      // bit words per point segment

// Order-preserving 64-bit key of a double (minima by atomicMin).
__device__ __forceinline__ unsigned long long buf_key(double v)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    return (b & 0x8000000000000000ull) ? ~b : (b | 0x8000000000000000ull);
}

static double buf_from_key(unsigned long long k)
{
    const unsigned long long b = (k & 0x8000000000000000ull) ? (k & 0x7fffffffffffffffull) : ~k;
    double d;
    std::memcpy(&d, &b, sizeof d);
    return d;
}

// The grid: cells of side `cell` (1 / inv) from (X0, Y0); (X1, Y1) closes
// the box.
struct BufGrid {
    double X0, Y0, X1, Y1, inv, cell;
    int gx, gy;
};

__device__ __forceinline__ int buf_cell(double v, double v0, double inv, int g)
{
    const double u = __dmul_rn(__dsub_rn(v, v0), inv);
    return (int)fmin(fmax(floor(u), 0.0), (double)(g - 1));
}

// The box's keys at all ones, the flags, the entry total and the length zero.
__global__ void k_buf_init(unsigned long long *bb)
{
    if (threadIdx.x < 8) bb[threadIdx.x] = threadIdx.x < 4 ? ~0ull : 0ull;
}

// One segment slot per vertex: vertex v of its ring to the next one (the
// ring's first vertex after the last when `closed`; a one-vertex ring is a
// point).  Validates the offsets and the vertices on the way (err bit 1:
// offsets, bit 2: a non-finite vertex) and reduces the segments' box into
// bb (min x, -max x, min y, -max y as ordered keys); sums the segments'
// lengths (an FP64 estimate, only for the grid's cell size) into *len.
__global__ __launch_bounds__(256) void k_buf_segs(int64_t R, const int64_t *rvo, int64_t V, const double *vx, const double *vy,
                           int closed, Seg *segs, uint8_t *valid, unsigned long long *bb, unsigned *err,
                           double *len)
{
    const int64_t nth = (int64_t)gridDim.x * blockDim.x;
    const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (int64_t k = gid; k <= R; k += nth) {
        const int64_t o = rvo[k];
        if ((k == 0 && o != 0) || (k == R && o != V) || (k < R && rvo[k + 1] < o)) atomicOr(err, 1u);
    }
    unsigned long long k0 = ~0ull, k1 = ~0ull, k2 = ~0ull, k3 = ~0ull;
    double lsum = 0.0;
    for (int64_t v = gid; v < V; v += nth) {
        valid[v] = 0;
        // ring of v: the last ring whose first vertex is <= v
        int64_t lo = 0, hi = R - 1;
        while (lo < hi) {
            const int64_t mid = (lo + hi + 1) >> 1;
            if (rvo[mid] <= v) lo = mid; else hi = mid - 1;
        }
        const int64_t o = rvo[lo], e = rvo[lo + 1];
        if (!(o >= 0 && o <= v && v < e && e <= V)) {
            atomicOr(err, 1u);
            continue;
        }
        int64_t w;
        if (e - o == 1) w = v;
        else if (v + 1 < e) w = v + 1;
        else if (closed) w = o;
        else continue;
        const double ax = vx[v], ay = vy[v], bx = vx[w], by = vy[w];
        if (!(isfinite(ax) && isfinite(ay) && isfinite(bx) && isfinite(by))) {
            atomicOr(err, 2u);
            continue;
        }
        segs[v] = Seg{ax, ay, bx, by};
        valid[v] = 1;
        lsum += hypot(bx - ax, by - ay);
        k0 = min(k0, min(buf_key(ax), buf_key(bx))); k1 = min(k1, min(buf_key(-ax), buf_key(-bx)));
        k2 = min(k2, min(buf_key(ay), buf_key(by))); k3 = min(k3, min(buf_key(-ay), buf_key(-by)));
    }
    for (int d = 32; d > 0; d >>= 1) {
        k0 = min(k0, (unsigned long long)__shfl_xor((long long)k0, d, 64));
        k1 = min(k1, (unsigned long long)__shfl_xor((long long)k1, d, 64));
        k2 = min(k2, (unsigned long long)__shfl_xor((long long)k2, d, 64));
        k3 = min(k3, (unsigned long long)__shfl_xor((long long)k3, d, 64));
    }
    for (int d = 32; d > 0; d >>= 1) lsum += __shfl_xor(lsum, d, 64);
    // one set of atomics per workgroup of 256 (all meet in one line)
    __shared__ unsigned long long part[4][4];
    __shared__ double plen[4];
    const int wv = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        part[wv][0] = k0;
        part[wv][1] = k1;
        part[wv][2] = k2;
        part[wv][3] = k3;
        plen[wv] = lsum;
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        const int k = threadIdx.x;
        const unsigned long long m = min(min(part[0][k], part[1][k]), min(part[2][k], part[3][k]));
        if (m != ~0ull) atomicMin(&bb[k], m);
    }
    if (threadIdx.x == 0) atomicAdd(len, plen[0] + plen[1] + plen[2] + plen[3]);
}

// Cells that may hold a point within r of each valid segment: the cells
// whose centre lies within r + half the cell diagonal of it (FP64 distance,
// with a relative margin of 1e-9 and the absolute part of pad, far above its
// rounding and that of the point-to-cell mapping).  A cell whose centre lies
// so near to one segment that its whole square is within r (fin: r less half
// the diagonal and the same margins; any point of the segment bounds the
// distance from above, so rounding of the nearest one cannot make it too
// small) is full: its points are results without a test, and it lists
// nothing.  FILL false: cnt[c] counts the entries, or has its top bit set
// when full, and the entries of all cells are summed into *tot.  FILL true:
// a copy of the segment goes in a per-cell slot from off[] claimed with
// cursor[], so that a point reads its cell's candidates contiguously, with no
// index to follow.
//
// The rows of a segment's box are spread over 2^lsh lanes, and of a row only
// the columns near the part of the segment that the row can reach are
// visited: a long segment is the work of its own cells, not of its box's.
constexpr uint32_t BUF_FULL = 0x80000000u;

template <bool FILL>
__global__ __launch_bounds__(256) void k_buf_bin(int64_t V, const Seg *segs, const uint8_t *valid, BufGrid g,
                                                 double pad, double fin, int lsh, uint32_t *cnt,
                                                 const uint32_t *off, uint32_t *cursor, Seg *list, unsigned long long *tot)
{
#pragma clang fp contract(off)   // both passes decide alike
    const int64_t nth = (int64_t)gridDim.x * blockDim.x;
    const double reach = (pad + 0.7071067811865476 * g.cell) * (1.0 + 1e-9);
    const double reach2 = reach * reach, fin2 = fin > 0.0 ? fin * fin : -1.0;
    unsigned long long nlisted = 0;
    for (int64_t w = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; w < (V << lsh); w += nth) {
        const int64_t v = w >> lsh;
        if (!valid[v]) continue;
        const Seg s = segs[v];
        const int x0 = buf_cell(fmin(s.ax, s.bx) - pad, g.X0, g.inv, g.gx);
        const int x1 = buf_cell(fmax(s.ax, s.bx) + pad, g.X0, g.inv, g.gx);
        const int y0 = buf_cell(fmin(s.ay, s.by) - pad, g.Y0, g.inv, g.gy);
        const int y1 = buf_cell(fmax(s.ay, s.by) + pad, g.Y0, g.inv, g.gy);
        const double ex = s.bx - s.ax, ey = s.by - s.ay, l2 = ex * ex + ey * ey;
        for (int cy = y0 + (int)(w - (v << lsh)); cy <= y1; cy += 1 << lsh) {
            int c0 = x0, c1 = x1;
            const double py = g.Y0 + (cy + 0.5) * g.cell;
            if (ey != 0.0) {
                const double t0 = fmin(fmax((py - reach - s.ay) / ey, 0.0), 1.0);
                const double t1 = fmin(fmax((py + reach - s.ay) / ey, 0.0), 1.0);
                const double xa = s.ax + t0 * ex, xb = s.ax + t1 * ex;
                const double lo = fmin(xa, xb) - reach, hi = fmax(xa, xb) + reach;
                if (isfinite(lo) && isfinite(hi)) {
                    c0 = max(c0, buf_cell(lo, g.X0, g.inv, g.gx) - 1);
                    c1 = min(c1, buf_cell(hi, g.X0, g.inv, g.gx) + 1);
                }
            }
            for (int cx = c0; cx <= c1; ++cx) {
                const double px = g.X0 + (cx + 0.5) * g.cell;
                double t = l2 > 0.0 ? ((px - s.ax) * ex + (py - s.ay) * ey) / l2 : 0.0;
                t = fmin(fmax(t, 0.0), 1.0);
                const double dx = px - (s.ax + t * ex), dy = py - (s.ay + t * ey);
                const double d2 = dx * dx + dy * dy;
                if (d2 > reach2) continue;
                const int64_t c = (int64_t)cy * g.gx + cx;
                if (FILL) {
                    if (!(cnt[c] & BUF_FULL)) list[off[c] + atomicAdd(&cursor[c], 1u)] = s;
                } else {
                    if (d2 <= fin2) atomicOr(&cnt[c], BUF_FULL);
                    else atomicAdd(&cnt[c], 1u);
                    ++nlisted;
                }
            }
        }
    }
    if (!FILL) {
        __shared__ unsigned long long part[4];
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) nlisted += (unsigned long long)__shfl_xor((long long)nlisted, d, 64);
        if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = nlisted;
        __syncthreads();
        // (2,048 workgroups adding to one word take 20 us, and with few
        // segments most have nothing to add)
        const unsigned long long sum = part[0] + part[1] + part[2] + part[3];
        if (threadIdx.x == 0 && sum != 0ull) atomicAdd(tot, sum);
    }
}

// Entries that a cell lists: none when it is full.
struct BufListed {
    __host__ __device__ uint32_t operator()(uint32_t c) const { return (c & BUF_FULL) ? 0u : c; }
};

// Two bits per cell, 16 cells a word: no candidate (0), candidates (1), full
// (2).  The points read these, which stay in a chiplet's L2 (1.4 MB for 5.8M
// cells); a table of 4-byte offsets did not, and every point's read of it
// went past (558 us for 50M points near 24k segments, now 495).
// Also leaves the number of list entries in *listed and clears *end (the
// count behind the last segment of points, whose scan is the total).
__global__ void k_buf_class(int64_t G, const uint32_t *cnt, const uint32_t *off, uint32_t *cls,
                            unsigned long long *listed, unsigned long long *end)
{
    const int64_t w = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (w == 0) {
        *listed = off[G];
        *end = 0ull;
    }
    if (w * 16 >= G) return;
    uint32_t v = 0;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const uint32_t c = w * 16 + k < G ? cnt[w * 16 + k] : 0u;
        v |= (c & BUF_FULL ? 2u : c ? 1u : 0u) << (2 * k);
    }
    cls[w] = v;
}

// The candidate tests of one wavefront's points, balanced over its lanes
// (wave_round): lane i's point has the candidates list[k, k + rem) left, and
// a point any of whose candidates in a round was within r drops the rest.
// Returns whether this lane's point was hit.  Without EXACT, candidates that
// the filter leaves open set `open` (for the whole wavefront) and count as not
// within.  Called by every lane of the wavefront.
template <bool EXACT>
__device__ __forceinline__ bool buf_wave_walk(double x, double y, uint32_t k, uint32_t rem, const Seg *list,
                                              double r, double r2, double pad, int lane, bool &open)
{
    bool hit = false;
    while (__ballot(rem != 0u)) {
        const WaveRound w = wave_round(rem, lane);
        const uint32_t ok = __shfl(k, w.o, 64);
        const double ox = __shfl(x, w.o, 64), oy = __shfl(y, w.o, 64);
        int h = 0;
        if ((uint32_t)lane < w.ntake) {
            const Seg s = list[ok + ((uint32_t)lane - w.opre)];
            // outside the segment's box widened by pad: farther than r
            if (!(ox < fmin(s.ax, s.bx) - pad || ox > fmax(s.ax, s.bx) + pad || oy < fmin(s.ay, s.by) - pad ||
                  oy > fmax(s.ay, s.by) + pad))
                h = EXACT ? (seg_near(ox, oy, s, r, r2) ? 1 : 0) : seg_near_filter(ox, oy, s, r2);
        }
        const unsigned long long hm = __ballot(h > 0);
        if (!EXACT && __ballot(h < 0)) open = true;
        const uint32_t len = wave_round_len(w);
        if (hm & wave_round_mask(w)) {
            hit = true;
            rem = 0u;
        } else {
            k += len;
            rem -= len;
        }
    }
    return hit;
}

// One result bit per point (layout of the ordered emit: word j of segment sg
// holds points sg * EMIT_SEG + 64 j + lane) and the count per segment.
//
// Bound by the latency of a chain of three dependent loads (point, cell
// range, candidates) and by the tests of the candidates.  A wavefront loads
// the points and cell ranges of BUF_GROUP words together, and queues the few
// points that have candidates in LDS, so that the candidate walk runs with
// about 64 points rather than with those of one word.  50M points, 24k
// segments, 50 m: 1.70 ms with cells of 150 m (every point's candidates
// tested, one word at a time), 0.50 ms with cells of 25 m; what is left is
// the rate of L2 requests (71M, most of them the points' cell codes).
// The canvas's coarse level needs one workgroup per CU; without a canvas the
// workgroups are small, so that the registers alone limit their number, and
// the exact tests' are kept out: a first pass (EXACT false) decides by the
// filter and leaves BUF_OPEN as the count of a segment in which a candidate
// stayed open, a second one (EXACT and ONLY_OPEN) does those segments again.
constexpr int BUF_GROUP = 4;                  // words in flight
constexpr int BUF_QCAP = 64;                  // queued points per wavefront
constexpr int BUF_QWAVE = BUF_QCAP * 22;      // x, y, cell, place: bytes per wavefront

constexpr unsigned long long BUF_OPEN = ~0ull;

template <bool POLY, int TH, bool EXACT, bool ONLY_OPEN>
__global__ __launch_bounds__(TH, TH == 256 && !EXACT ? 5 : 1) void k_buf_bits(CanvasView cv, int64_t n, const double *X, const double *Y,
                                                 BufGrid g, const uint32_t *cls, const uint32_t *off,
                                                 const Seg *list, double r, double r2, double pad, int64_t nseg, unsigned long long *counts,
                                                 unsigned long long *bits)
{
    static_assert(BUF_WORDS % BUF_GROUP == 0 && BUF_WORDS <= BUF_QCAP, "words per segment");
    static_assert(BUF_QWAVE % 8 == 0 && EMIT_SEG <= 65536, "queue layout");
    extern __shared__ __align__(16) unsigned char smem[];
    uint16_t *coarse = (uint16_t *)smem;
    size_t cbytes = 0;
    if (POLY) {
        cbytes = ((size_t)cv.Wc * cv.Hc * (cv.cbyte ? 1 : 2) + 15) & ~(size_t)15;
        load_coarse(cv, coarse, TH);
        __syncthreads();
    }
    const int lane = threadIdx.x & 63;
    const unsigned long long below = (1ull << lane) - 1ull;
    unsigned char *q = smem + cbytes + (threadIdx.x >> 6) * BUF_QWAVE;
    double *qx = (double *)q, *qy = qx + BUF_QCAP;
    uint32_t *qc = (uint32_t *)(qy + BUF_QCAP);
    uint16_t *qi = (uint16_t *)(qc + BUF_QCAP);
    unsigned long long *qw = (unsigned long long *)q;   // a drain's result words, over the points it has read
    auto sync = [] {   // order this wavefront's LDS accesses
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    const int64_t nwave = ((int64_t)gridDim.x * TH) >> 6;
    for (int64_t sg = ((int64_t)blockIdx.x * TH + threadIdx.x) >> 6; sg < nseg; sg += nwave) {
        if (ONLY_OPEN && counts[sg] != BUF_OPEN) continue;
        unsigned long long segw = 0;   // lane j < BUF_WORDS: word j
        uint32_t qn = 0;               // wave-uniform
        bool open = false;             // wave-uniform
        auto drain = [&]() {
            sync();
            double x = NAN, y = NAN;
            uint32_t k = 0u, rem = 0u, id = 0u;
            if (lane < (int)qn) {
                x = qx[lane];
                y = qy[lane];
                id = qi[lane];
                const uint32_t c = qc[lane];
                k = off[c];
                rem = off[c + 1] - k;
            }
            const bool hit = buf_wave_walk<EXACT>(x, y, k, rem, list, r, r2, pad, lane, open);
            sync();
            if (lane < BUF_WORDS) qw[lane] = 0ull;
            sync();
            if (hit) atomicOr(&qw[id >> 6], 1ull << (id & 63u));
            sync();
            if (lane < BUF_WORDS) segw |= qw[lane];
            sync();
            qn = 0;
        };
#pragma nounroll
        for (int g0 = 0; g0 < BUF_WORDS; g0 += BUF_GROUP) {
            double xs[BUF_GROUP], ys[BUF_GROUP];
#pragma unroll
            for (int k = 0; k < BUF_GROUP; ++k) {
                const int64_t i = sg * EMIT_SEG + 64 * (g0 + k) + lane;
                xs[k] = i < n ? __builtin_nontemporal_load(X + i) : NAN;
                ys[k] = i < n ? __builtin_nontemporal_load(Y + i) : NAN;
            }
            uint32_t inside = 0;   // bit k: the polygon holds this lane's point of word k
            if (POLY) {
                uint32_t ws[BUF_GROUP];
#pragma unroll
                for (int k = 0; k < BUF_GROUP; ++k) ws[k] = lookup(cv, coarse, xs[k], ys[k]);
#pragma unroll
                for (int k = 0; k < BUF_GROUP; ++k) {
                    bool in = ws[k] != 0u && !(ws[k] & BFLAG);
                    if (ws[k] & BFLAG) {
                        uint32_t rec = ws[k] & ~BFLAG;
                        while (true) {
                            const Cand c = cv.cands[rec];
                            if (cand_inside(cv, c, xs[k], ys[k])) { in = true; break; }
                            if (c.meta & CAND_LAST) break;
                            ++rec;
                        }
                    }
                    const unsigned long long word = __ballot(in);
                    if (lane == g0 + k) segw |= word;
                    if (in) inside |= 1u << k;
                }
            }
            uint32_t cs[BUF_GROUP], code[BUF_GROUP];
#pragma unroll
            for (int k = 0; k < BUF_GROUP; ++k) {
                // NaN fails the box test
                const bool on = xs[k] >= g.X0 && xs[k] <= g.X1 && ys[k] >= g.Y0 && ys[k] <= g.Y1 &&
                                !(POLY && ((inside >> k) & 1u));
                cs[k] = on ? (uint32_t)buf_cell(ys[k], g.Y0, g.inv, g.gy) * (uint32_t)g.gx +
                                 (uint32_t)buf_cell(xs[k], g.X0, g.inv, g.gx)
                           : 0u;
                code[k] = on ? cls[cs[k] >> 4] >> (2u * (cs[k] & 15u)) & 3u : 0u;
            }
#pragma unroll
            for (int k = 0; k < BUF_GROUP; ++k) {
                const unsigned long long word = __ballot(code[k] == 2u);
                if (lane == g0 + k) segw |= word;
                const bool on = code[k] == 1u;
                const unsigned long long mask = __ballot(on);
                const uint32_t nnew = (uint32_t)__popcll(mask);
                if (nnew == 0) continue;
                if (qn + nnew > (uint32_t)BUF_QCAP) drain();
                if (on) {
                    const uint32_t slot = qn + (uint32_t)__popcll(mask & below);
                    qx[slot] = xs[k];
                    qy[slot] = ys[k];
                    qc[slot] = cs[k];
                    qi[slot] = (uint16_t)(64 * (g0 + k) + lane);
                }
                qn += nnew;
            }
        }
        if (qn) drain();
        uint32_t total = lane < BUF_WORDS ? (uint32_t)__popcll(segw) : 0u;
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) total += __shfl_xor(total, d, 64);
        if (lane < BUF_WORDS) bits[sg * BUF_WORDS + lane] = segw;
        if (lane == 0) counts[sg] = !EXACT && open ? BUF_OPEN : total;
    }
}

__global__ void k_buf_zero(unsigned long long *p) { *p = 0ull; }

int buffer_select(spade_ctx *ctx, const spade_canvas *cv, const spade_points *pts, const spade_polys *geom, double r,
                  bool closed, uint32_t *out_ids, int64_t cap, int64_t *n_out)
{
    hipStream_t st = ctx->stream;
    if (n_out) *n_out = 0;
    if (!(std::isfinite(r) && r >= 0.0)) return set_error(ctx, SPADE_E_INVALID, "the distance must be finite and >= 0");
    if (cap < 0) return set_error(ctx, SPADE_E_INVALID, "negative capacity");
    if (cap > 0 && !out_ids) return set_error(ctx, SPADE_E_INVALID, "out_ids is NULL");
    if (!geom) return set_error(ctx, SPADE_E_INVALID, "geometry is NULL");
    const int64_t R = geom->n_rings;
    if (R < 0) return set_error(ctx, SPADE_E_INVALID, "negative ring count");
    if (R > 0 && (!geom->ring_vtx_off || !geom->vx || !geom->vy))
        return set_error(ctx, SPADE_E_INVALID, "geometry array is NULL");
    // vertex count: given, else read back
    int64_t V = 0;
    if (R > 0) {
        if (geom->n_vertices > 0) {
            V = geom->n_vertices;
        } else {
            int64_t *h = (int64_t *)ensure_pinned(ctx, 64);
            if (!h) return set_error(ctx, SPADE_E_NOMEM, "pinned staging allocation failed");
            SPADE_HIP(ctx, hipMemcpyAsync(h, geom->ring_vtx_off + R, sizeof(int64_t), hipMemcpyDeviceToHost, st));
            SPADE_HIP(ctx, hipStreamSynchronize(st));
            V = h[0];
        }
        if (V < 0 || V >= (int64_t)0xffffffffLL) return set_error(ctx, SPADE_E_INVALID, "bad vertex count");
    }
    const int64_t n = pts->n;
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, ctx->device) != hipSuccess || cus <= 0)
        cus = 256;

    // segments, their box, validation
    DevBuf &bs = ctx->scratch[S_BUF_SEGS], &bg = ctx->scratch[S_BUF_GRID];
    if (ensure(ctx, bs, sizeof(Seg) * (size_t)std::max<int64_t>(V, 1) + (size_t)V + 16) || ensure(ctx, bg, 256))
        return SPADE_E_NOMEM;
    Seg *segs = (Seg *)bs.p;
    uint8_t *valid = (uint8_t *)(segs + std::max<int64_t>(V, 1));
    unsigned long long *bb = (unsigned long long *)bg.p;
    unsigned *err = (unsigned *)(bb + 4);
    double *dlen = (double *)(bb + 6);
    hipLaunchKernelGGL(k_buf_init, dim3(1), dim3(64), 0, st, bb);
    SPADE_HIP(ctx, hipGetLastError());
    if (R > 0) {
        const int sgrid = (int)std::max<int64_t>(1, std::min<int64_t>((std::max(V, R + 1) + 255) / 256, (int64_t)cus * 8));
        hipLaunchKernelGGL(k_buf_segs, dim3(sgrid), dim3(256), 0, st, R, geom->ring_vtx_off, V, geom->vx, geom->vy,
                           closed ? 1 : 0, segs, valid, bb, err, dlen);
        SPADE_HIP(ctx, hipGetLastError());
    }
    unsigned long long *h = (unsigned long long *)ensure_pinned(ctx, 64);
    if (!h) return set_error(ctx, SPADE_E_NOMEM, "pinned staging allocation failed");
    SPADE_HIP(ctx, hipMemcpyAsync(h, bb, 7 * sizeof(unsigned long long), hipMemcpyDeviceToHost, st));
    SPADE_HIP(ctx, hipStreamSynchronize(st));
    const unsigned ef = (unsigned)(h[4] & 0xffffffffu);
    if (ef & 1u) return set_error(ctx, SPADE_E_INVALID, "ring offsets are not a valid CSR array");
    if (ef & 2u) return set_error(ctx, SPADE_E_INVALID, "a vertex coordinate is not finite");
    const bool any = h[0] != ~0ull;
    double len_sum;
    std::memcpy(&len_sum, &h[6], sizeof len_sum);
    if (n == 0) return SPADE_OK;

    const int64_t nseg = (n + EMIT_SEG - 1) / EMIT_SEG;
    DevBuf &lb = ctx->scratch[S_LOOKBACK], &bbits = ctx->scratch[S_BITS];
    if (ensure(ctx, lb, sizeof(unsigned long long) * 2 * (size_t)(nseg + 1)) ||
        ensure(ctx, bbits, sizeof(unsigned long long) * BUF_WORDS * (size_t)nseg))
        return SPADE_E_NOMEM;
    unsigned long long *counts = (unsigned long long *)lb.p;
    unsigned long long *offs = counts + (nseg + 1);
    unsigned long long *bits = (unsigned long long *)bbits.p;

    // the grid over the segments' box widened by r (and a relative margin,
    // so that rounding never drops a position within r)
    BufGrid grid{0.0, 0.0, -1.0, -1.0, 1.0, 1.0, 1, 1};   // empty box: no point is tested
    double pad = 0.0;
    uint32_t *off = nullptr, *cls = nullptr;
    Seg *list = nullptr;
    if (any) {
        const double x0 = buf_from_key(h[0]), x1 = -buf_from_key(h[1]);
        const double y0 = buf_from_key(h[2]), y1 = -buf_from_key(h[3]);
        const double mag = std::fabs(x0) + std::fabs(x1) + std::fabs(y0) + std::fabs(y1);
        pad = r * (1.0 + 0x1p-40) + mag * 0x1p-40 + 1e-300;
        const double X0 = x0 - pad, X1 = x1 + pad, Y0 = y0 - pad, Y1 = y1 + pad;
        const double w = X1 - X0, hgt = Y1 - Y0;
        // Cells as wide as r or the mean segment length, whichever is
        // larger (a segment then meets a few cells, a cell a few segments),
        // at most BUF_GRID_MAX per side.  With many points, finer ones, down
        // to r / BUF_FINE, of which those inside the distance need no test:
        // as many as leaves the lists and the cell table small beside the
        // points (the entries a segment makes are about the area it reaches
        // over that of a cell).  50M points, 24k segments, 50 m: r / 2 takes
        // 0.85 ms, r / 3 1.18 (lists and table twice as large), r 1.9.
        const double lmean = std::isfinite(len_sum) ? len_sum / (double)std::max<int64_t>(V, 1) : 0.0;
        double cell = std::max(r, std::min(lmean, std::sqrt(w * hgt / (2.0 * (double)std::max<int64_t>(V, 1)))));
        cell = std::max(cell, std::max(w, hgt) / BUF_GRID_MAX);
        if (!(cell > 1e-290)) cell = 1.0;
        const double most = std::min((double)n / BUF_PER_ENTRY, 16777216.0);
        double fine = std::max({r / BUF_FINE, std::sqrt(w) * std::sqrt(hgt) / std::sqrt((double)n / BUF_PER_CELL),
                                std::max(w, hgt) / BUF_GRID_MAX});
        auto entries = [&](double c) {
            const double reach = pad + 0.75 * c;
            return (double)V * (2.0 * reach * lmean + 3.15 * reach * reach) / (c * c);
        };
        while (fine < cell && !(entries(fine) <= most)) fine *= 1.19;
        const double coarse_cell = cell;
        if (fine > 1e-290 && fine < cell && std::isfinite(len_sum)) cell = fine;
        uint32_t *cnt, *cursor;
        int64_t G;
        int lsh, bgrid;
        double fin;
        while (true) {
            grid.X0 = X0; grid.Y0 = Y0; grid.X1 = X1; grid.Y1 = Y1;
            grid.inv = 1.0 / cell;
            grid.cell = cell;
            grid.gx = (int)std::min<double>(BUF_GRID_MAX, std::max(1.0, std::ceil(w * grid.inv)));
            grid.gy = (int)std::min<double>(BUF_GRID_MAX, std::max(1.0, std::ceil(hgt * grid.inv)));
            G = (int64_t)grid.gx * grid.gy;
            // within r whatever the rounding: half a diagonal and the margins less
            const double eps = mag * 0x1p-40 + 1e-300;
            fin = r * (1.0 - 0x1p-40) - 4.0 * eps - 0.7071067811865476 * cell * (1.0 + 0x1p-19);
            // lanes per segment: enough that few segments still fill the chip
            lsh = 0;
            while (lsh < 12 && (V << lsh) < (int64_t)cus * 2048) ++lsh;
            DevBuf &bt = ctx->scratch[S_BUF_TMP];
            if (ensure(ctx, bg, 256 + sizeof(uint32_t) * (3 * (size_t)(G + 1) + (size_t)(G / 16 + 1))))
                return SPADE_E_NOMEM;
            bb = (unsigned long long *)bg.p;
            cnt = (uint32_t *)((unsigned char *)bg.p + 256);
            cursor = cnt + (G + 1);
            off = cursor + (G + 1);
            cls = off + (G + 1);
            unsigned long long *tot = bb + 5;   // cleared with the counters behind it
            SPADE_HIP(ctx, hipMemsetAsync(tot, 0, (size_t)((unsigned char *)off - (unsigned char *)tot), st));
            bgrid = (int)std::max<int64_t>(1, std::min<int64_t>(((V << lsh) + 255) / 256, (int64_t)cus * 8));
            hipLaunchKernelGGL(k_buf_bin<false>, dim3(bgrid), dim3(256), 0, st, V, (const Seg *)segs,
                               (const uint8_t *)valid, grid, pad, fin, lsh, cnt, (const uint32_t *)nullptr,
                               (uint32_t *)nullptr, (Seg *)nullptr, tot);
            SPADE_HIP(ctx, hipGetLastError());
            rocprim::transform_iterator<const uint32_t *, BufListed, uint32_t> listed(cnt, BufListed{});
            size_t tb = 0;
            SPADE_HIP(ctx, rocprim::exclusive_scan(nullptr, tb, listed, off, 0u, (size_t)(G + 1),
                                                   rocprim::plus<uint32_t>(), st));
            if (ensure(ctx, bt, std::max<size_t>(tb, 1))) return SPADE_E_NOMEM;
            SPADE_HIP(ctx, rocprim::exclusive_scan(bt.p, tb, listed, off, 0u, (size_t)(G + 1),
                                                   rocprim::plus<uint32_t>(), st));
            // the 64-bit entry count first: the cell lists (32 bytes an entry)
            // stay below 2^28 entries, so their 32-bit offsets are exact
            hipLaunchKernelGGL(k_buf_class, dim3((unsigned)((G + 4095) / 4096)), dim3(256), 0, st, G,
                               (const uint32_t *)cnt, (const uint32_t *)off, cls, tot + 1, counts + nseg);
            SPADE_HIP(ctx, hipGetLastError());
            SPADE_HIP(ctx, hipMemcpyAsync(h, tot, 2 * sizeof(unsigned long long), hipMemcpyDeviceToHost, st));
            SPADE_HIP(ctx, hipStreamSynchronize(st));
            if (h[0] < ((unsigned long long)1 << 28)) break;
            if (cell == coarse_cell)
                return set_error(ctx, SPADE_E_TOO_LARGE, "too many (segment, cell) entries: the distance is too large "
                                                         "for the segments' spread");
            cell = coarse_cell;   // the estimate was too low
        }
        const uint64_t total = h[1];
        DevBuf &bl = ctx->scratch[S_BUF_LIST];
        if (ensure(ctx, bl, sizeof(Seg) * (size_t)std::max<uint64_t>(total, 1))) return SPADE_E_NOMEM;
        list = (Seg *)bl.p;
        hipLaunchKernelGGL(k_buf_bin<true>, dim3(bgrid), dim3(256), 0, st, V, (const Seg *)segs,
                           (const uint8_t *)valid, grid, pad, fin, lsh, cnt, (const uint32_t *)off, cursor, list,
                           (unsigned long long *)nullptr);
        SPADE_HIP(ctx, hipGetLastError());
    }

    // result bits and per-segment counts, then the ordered write pass
    const double r2 = r * r;
    auto bits_pass = [&](auto kern, int threads, int per_cu, size_t lds, const CanvasView &v) -> int {
        const int64_t wpb = threads / 64;
        const int grid_b = (int)std::max<int64_t>(1, std::min<int64_t>((nseg + wpb - 1) / wpb, (int64_t)cus * per_cu));
        lds += (size_t)wpb * BUF_QWAVE;
        SPADE_HIP(ctx, hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        hipLaunchKernelGGL(kern, dim3(grid_b), dim3(threads), lds, st, v, n, pts->x, pts->y, grid,
                           (const uint32_t *)cls, (const uint32_t *)off, (const Seg *)list, r, r2, pad, nseg, counts,
                           bits);
        SPADE_HIP(ctx, hipGetLastError());
        return SPADE_OK;
    };
    if (ctx->timing) SPADE_HIP(ctx, hipEventRecord(ctx->ev[2], st));
    if (cv) {
        const CanvasView &v = cv->view;
        const size_t lds = ((size_t)v.Wc * v.Hc * (v.cbyte ? 1 : 2) + 15) & ~(size_t)15;
        if (lds + BUF_THREADS / 64 * BUF_QWAVE > 160 * 1024)
            return set_error(ctx, SPADE_E_HIP, "internal: coarse level exceeds the LDS");
        if (const int rc = bits_pass(k_buf_bits<true, BUF_THREADS, true, false>, BUF_THREADS, 1, lds, v)) return rc;
    } else if (n < BUF_FILTER_MIN) {
        if (const int rc = bits_pass(k_buf_bits<false, 256, true, false>, 256, 4, 0, CanvasView{})) return rc;
    } else {
        if (const int rc = bits_pass(k_buf_bits<false, 256, false, false>, 256, 5, 0, CanvasView{})) return rc;
        if (const int rc = bits_pass(k_buf_bits<false, 256, true, true>, 256, 4, 0, CanvasView{})) return rc;
    }
    if (!any) hipLaunchKernelGGL(k_buf_zero, dim3(1), dim3(1), 0, st, counts + nseg);
    SPADE_HIP(ctx, hipGetLastError());
    DevBuf &bt = ctx->scratch[S_BUF_TMP];
    size_t tb = 0;
    SPADE_HIP(ctx, hipcub::DeviceScan::ExclusiveSum(nullptr, tb, counts, offs, (int)(nseg + 1), st));
    if (ensure(ctx, bt, std::max<size_t>(tb, 1))) return SPADE_E_NOMEM;
    SPADE_HIP(ctx, hipcub::DeviceScan::ExclusiveSum(bt.p, tb, counts, offs, (int)(nseg + 1), st));
    if (cap > 0) {
        const int eg = (int)std::max<int64_t>(1, std::min<int64_t>((nseg + 3) / 4, (int64_t)cus * 16));
        hipLaunchKernelGGL(k_emit_bits, dim3(eg), dim3(256), 0, st, nseg, (const unsigned long long *)offs,
                           (const unsigned long long *)bits, out_ids, (uint32_t *)nullptr, cap);
        SPADE_HIP(ctx, hipGetLastError());
    }
    if (ctx->timing) SPADE_HIP(ctx, hipEventRecord(ctx->ev[3], st));
    SPADE_HIP(ctx, hipMemcpyAsync(h, offs + nseg, sizeof(unsigned long long), hipMemcpyDeviceToHost, st));
    SPADE_HIP(ctx, hipStreamSynchronize(st));
    if (n_out) *n_out = (int64_t)h[0];
    if ((int64_t)h[0] > cap) return set_error(ctx, SPADE_E_CAPACITY, "output capacity too small");
    return SPADE_OK;
}


// ------------------------------------------------------------ distance join with lines
//
// Sec. 5.2's distance joins of types (1) and (2) with lines as the
// constraint dataset: every ring of the line set is one line object j (an
// open polyline) with its distance r_j (type 2) or one distance for all
// (type 1), and the join returns the pairs (point, line) of the points within
// r_j of line j.  The segments, each with its line and distance, are binned
// as for the selection; each cell's list is then sorted by segment id, so
// that a line's segments are consecutive in it and a point meets each of its
// lines once, in ascending line order: the first segment of a line within
// that line's distance emits the pair, the rest of the line is skipped.

struct JSeg {
    double ax, ay, bx, by, r;
    uint32_t line, pad_;
};

// Segment slot v of a set of open polylines: its line (ring) and far end,
// or false (last vertex of a ring, or malformed offsets: err bit 1).
__device__ __forceinline__ bool line_seg_of(int64_t R, const int64_t *rvo, int64_t V, int64_t v, int64_t &ring,
                                            int64_t &w, unsigned *err)
{
    int64_t lo = 0, hi = R - 1;
    while (lo < hi) {
        const int64_t mid = (lo + hi + 1) >> 1;
        if (rvo[mid] <= v) lo = mid; else hi = mid - 1;
    }
    const int64_t o = rvo[lo], e = rvo[lo + 1];
    if (!(o >= 0 && o <= v && v < e && e <= V)) {
        atomicOr(err, 1u);
        return false;
    }
    ring = lo;
    if (e - o == 1) w = v;
    else if (v + 1 < e) w = v + 1;
    else return false;
    return true;
}

// Segments with their line and distance; validates offsets (err bit 1),
// vertices (bit 2) and distances (bit 4); reduces the segments' box into bb
// and the largest distance into bb[7] (as the ordered key of -r).
__global__ void k_bufj_segs(int64_t R, const int64_t *rvo, int64_t V, const double *vx, const double *vy,
                            const double *rline, double r_all, JSeg *segs, uint8_t *valid,
                            unsigned long long *bb, unsigned *err, double *len)
{
    const int64_t nth = (int64_t)gridDim.x * blockDim.x;
    const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (int64_t k = gid; k <= R; k += nth) {
        const int64_t o = rvo[k];
        if ((k == 0 && o != 0) || (k == R && o != V) || (k < R && rvo[k + 1] < o)) atomicOr(err, 1u);
        if (k < R && rline && !(isfinite(rline[k]) && rline[k] >= 0.0)) atomicOr(err, 4u);
    }
    unsigned long long k0 = ~0ull, k1 = ~0ull, k2 = ~0ull, k3 = ~0ull, kr = ~0ull;
    double lsum = 0.0;
    for (int64_t v = gid; v < V; v += nth) {
        valid[v] = 0;
        int64_t ring, w;
        if (!line_seg_of(R, rvo, V, v, ring, w, err)) continue;
        const double ax = vx[v], ay = vy[v], bx = vx[w], by = vy[w];
        const double r = rline ? rline[ring] : r_all;
        if (!(isfinite(ax) && isfinite(ay) && isfinite(bx) && isfinite(by))) {
            atomicOr(err, 2u);
            continue;
        }
        if (!(isfinite(r) && r >= 0.0)) continue;   // reported through bit 4
        segs[v] = JSeg{ax, ay, bx, by, r, (uint32_t)ring, 0u};
        valid[v] = 1;
        lsum += hypot(bx - ax, by - ay);
        k0 = min(k0, min(buf_key(ax), buf_key(bx))); k1 = min(k1, min(buf_key(-ax), buf_key(-bx)));
        k2 = min(k2, min(buf_key(ay), buf_key(by))); k3 = min(k3, min(buf_key(-ay), buf_key(-by)));
        kr = min(kr, buf_key(-r));
    }
    for (int d = 32; d > 0; d >>= 1) {
        k0 = min(k0, (unsigned long long)__shfl_xor((long long)k0, d, 64));
        k1 = min(k1, (unsigned long long)__shfl_xor((long long)k1, d, 64));
        k2 = min(k2, (unsigned long long)__shfl_xor((long long)k2, d, 64));
        k3 = min(k3, (unsigned long long)__shfl_xor((long long)k3, d, 64));
        kr = min(kr, (unsigned long long)__shfl_xor((long long)kr, d, 64));
        lsum += __shfl_xor(lsum, d, 64);
    }
    if ((threadIdx.x & 63) == 0 && k0 != ~0ull) {
        atomicMin(&bb[0], k0); atomicMin(&bb[1], k1); atomicMin(&bb[2], k2); atomicMin(&bb[3], k3);
        atomicMin(&bb[7], kr);
        atomicAdd(len, lsum);
    }
}

// Cells that may hold a point within a segment's own distance of it (as
// k_buf_bin, with the segment's pad r (1 + 2^-40) + magpad): counted
// (FILL false, entries summed into *tot) or listed as sort keys
// (cell << 32 | segment) with the segment as value.
template <bool FILL>
__global__ void k_bufj_bin(int64_t V, const JSeg *segs, const uint8_t *valid, BufGrid g, double magpad,
                           uint32_t *cnt, const uint32_t *off, unsigned long long *keys, uint32_t *vals,
                           unsigned long long *tot)
{
    const int64_t nth = (int64_t)gridDim.x * blockDim.x;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < V; v += nth) {
        if (!valid[v]) continue;
        const JSeg s = segs[v];
        const double pad = s.r * (1.0 + 0x1p-40) + magpad;
        const int x0 = buf_cell(fmin(s.ax, s.bx) - pad, g.X0, g.inv, g.gx);
        const int x1 = buf_cell(fmax(s.ax, s.bx) + pad, g.X0, g.inv, g.gx);
        const int y0 = buf_cell(fmin(s.ay, s.by) - pad, g.Y0, g.inv, g.gy);
        const int y1 = buf_cell(fmax(s.ay, s.by) + pad, g.Y0, g.inv, g.gy);
        const double ex = s.bx - s.ax, ey = s.by - s.ay, l2 = ex * ex + ey * ey;
        const double reach = (pad + 0.7071067811865476 * g.cell) * (1.0 + 1e-9);
        const double reach2 = reach * reach;
        unsigned long long nlisted = 0;
        for (int cy = y0; cy <= y1; ++cy)
            for (int cx = x0; cx <= x1; ++cx) {
                const double px = g.X0 + (cx + 0.5) * g.cell, py = g.Y0 + (cy + 0.5) * g.cell;
                double t = l2 > 0.0 ? ((px - s.ax) * ex + (py - s.ay) * ey) / l2 : 0.0;
                t = fmin(fmax(t, 0.0), 1.0);
                const double dx = px - (s.ax + t * ex), dy = py - (s.ay + t * ey);
                if (dx * dx + dy * dy > reach2) continue;
                const int64_t c = (int64_t)cy * g.gx + cx;
                if (FILL) {
                    const uint32_t at = off[c] + atomicAdd(&cnt[c], 1u);
                    keys[at] = ((unsigned long long)c << 32) | (unsigned long long)v;
                    vals[at] = (uint32_t)v;
                } else {
                    atomicAdd(&cnt[c], 1u);
                }
                ++nlisted;
            }
        if (!FILL) atomicAdd(tot, nlisted);
    }
}

// Cell lists in sorted order: copies of the segments.
__global__ void k_bufj_gather(int64_t ntot, const uint32_t *vals, const JSeg *segs, JSeg *list)
{
    const int64_t nth = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < ntot; i += nth) list[i] = segs[vals[i]];
}

// The cell's candidates of a point: list[k, k + rem), or none outside the
// grid's box (NaN fails the test too).
__device__ __forceinline__ void bufj_range(double x, double y, const BufGrid &g, const uint32_t *off, uint32_t &k,
                                           uint32_t &rem)
{
    k = 0u;
    rem = 0u;
    if (x >= g.X0 && x <= g.X1 && y >= g.Y0 && y <= g.Y1) {
        const int64_t c = (int64_t)buf_cell(y, g.Y0, g.inv, g.gy) * g.gx + buf_cell(x, g.X0, g.inv, g.gx);
        k = off[c];
        rem = off[c + 1] - k;
    }
}

// The (point, line) pairs of a wavefront's points, with the candidate tests
// balanced over the lanes (wave_round).  A cell's list is sorted by segment,
// so a line's segments are consecutive in it, and a hit repeats its point's
// previous hit exactly when it has the same line: the previous hit is found
// among the round's earlier positions of the same point, else it is the last
// line the point met in earlier rounds.  A repeated line is not tested again
// once its point has met it in an earlier round.  For each new pair the
// testing lane calls pair(o, slot, line) with o the point's lane and slot =
// base of lane o + the pair's rank among the point's pairs (ascending line
// order); on return cnt holds the number of pairs of this lane's point.
// Called by every lane of the wavefront.
template <typename Pair>
__device__ __forceinline__ void bufj_wave_walk(double x, double y, uint32_t k, uint32_t rem, const JSeg *list,
                                               double magpad, uint32_t base, int lane, uint32_t &cnt, Pair &&pair)
{
    uint32_t last = 0xffffffffu;
    cnt = 0u;
    while (__ballot(rem != 0u)) {
        const WaveRound w = wave_round(rem, lane);
        const uint32_t ok = __shfl(k, w.o, 64);
        const uint32_t olast = __shfl(last, w.o, 64);
        const uint32_t ocnt = __shfl(cnt, w.o, 64);
        const uint32_t obase = __shfl(base, w.o, 64);
        const double ox = __shfl(x, w.o, 64), oy = __shfl(y, w.o, 64);
        bool h = false;
        uint32_t line = 0xffffffffu;
        if ((uint32_t)lane < w.ntake) {
            const JSeg sg = list[ok + ((uint32_t)lane - w.opre)];
            line = sg.line;
            if (line != olast) {
                const double pad = sg.r * (1.0 + 0x1p-40) + magpad;
                if (!(ox < fmin(sg.ax, sg.bx) - pad || ox > fmax(sg.ax, sg.bx) + pad ||
                      oy < fmin(sg.ay, sg.by) - pad || oy > fmax(sg.ay, sg.by) + pad))
                    h = seg_near(ox, oy, Seg{sg.ax, sg.ay, sg.bx, sg.by}, sg.r, sg.r * sg.r);
            }
        }
        const unsigned long long hm = __ballot(h);
        // the previous hit of the same point in this round, if any
        const unsigned long long own = wave_round_before(w, lane);
        const unsigned long long ph = hm & own;
        const uint32_t pline = __shfl(line, ph ? 63 - __clzll((long long)ph) : lane, 64);
        const bool fresh = h && line != (ph ? pline : olast);
        const unsigned long long nm = __ballot(fresh);
        if (fresh) pair(w.o, obase + ocnt + (uint32_t)__popcll(nm & own), line);
        // this point's pairs of the round, and its last hit line
        const unsigned long long mine = wave_round_mask(w);
        const unsigned long long myh = hm & mine;
        const uint32_t hline = __shfl(line, myh ? 63 - __clzll((long long)myh) : lane, 64);
        if (myh) last = hline;
        cnt += (uint32_t)__popcll(nm & mine);
        const uint32_t len = wave_round_len(w);
        k += len;
        rem -= len;
    }
}

// MODE 0: pairs per 1024-point segment (counts[sg]; with pcount, also the
// pairs of every point, so that the write pass walks once); MODE 1: the pairs, from
// offs[sg] on (below cap; the first cap in (point, line) order); MODE 2:
// pairs per line added into lcount (an LDS histogram when nlines <= hist).
template <int MODE>
__global__ __launch_bounds__(BUF_THREADS) void k_bufj_pairs(int64_t n, const double *X, const double *Y, BufGrid g,
                                                            const uint32_t *off, const JSeg *list, double magpad,
                                                            int64_t nseg, unsigned long long *counts,
                                                            const unsigned long long *offs, uint32_t *out_pt,
                                                            uint32_t *out_line, int64_t cap,
                                                            unsigned long long *lcount, int nlines, int hist,
                                                            uint32_t *pcount)
{
    extern __shared__ __align__(16) unsigned char smem[];
    uint32_t *h = (uint32_t *)smem;
    const bool lds = MODE == 2 && nlines <= hist;
    if (lds) {
        for (int k = threadIdx.x; k < nlines; k += BUF_THREADS) h[k] = 0u;
        __syncthreads();
    }
    const int lane = threadIdx.x & 63;
    const int64_t nwave = ((int64_t)gridDim.x * BUF_THREADS) >> 6;
    for (int64_t sg = ((int64_t)blockIdx.x * BUF_THREADS + threadIdx.x) >> 6; sg < nseg; sg += nwave) {
        unsigned long long total = 0;
        int64_t pos = MODE == 1 ? (int64_t)offs[sg] : 0;
        for (int j = 0; j < BUF_WORDS; ++j) {
            const int64_t i = sg * EMIT_SEG + 64 * j + lane;
            const double x = i < n ? __builtin_nontemporal_load(X + i) : NAN;
            const double y = i < n ? __builtin_nontemporal_load(Y + i) : NAN;
            uint32_t k, rem, cnt;
            bufj_range(x, y, g, off, k, rem);
            if (MODE == 2) {
                bufj_wave_walk(x, y, k, rem, list, magpad, 0u, lane, cnt, [&](int, uint32_t, uint32_t line) {
                    if (lds) atomicAdd(&h[line], 1u);
                    else atomicAdd(&lcount[line], 1ull);
                });
                continue;
            }
            if (MODE == 1 && pcount) {
                cnt = i < n ? pcount[i] : 0u;   // the count pass's pairs of this point
            } else {
                bufj_wave_walk(x, y, k, rem, list, magpad, 0u, lane, cnt, [](int, uint32_t, uint32_t) {});
                if (MODE == 0 && pcount && i < n) pcount[i] = cnt;
            }
            // the wavefront's pairs of this word, in lane order
            uint32_t pre = cnt;
            for (int d = 1; d < 64; d <<= 1) {
                const uint32_t t = (uint32_t)__shfl_up((int)pre, d, 64);
                if (lane >= d) pre += t;
            }
            const uint32_t wsum = (uint32_t)__shfl((int)pre, 63, 64);
            if (MODE == 1 && wsum) {
                // again, writing each pair at pos + (pairs of earlier lanes) + rank
                const int64_t w0 = sg * EMIT_SEG + 64 * j;
                uint32_t c2;
                bufj_wave_walk(x, y, k, cnt ? rem : 0u, list, magpad, pre - cnt, lane, c2,
                               [&](int o, uint32_t slot, uint32_t line) {
                                   const int64_t p = pos + (int64_t)slot;
                                   if (p < cap) {
                                       out_pt[p] = (uint32_t)(w0 + o);
                                       out_line[p] = line;
                                   }
                               });
            }
            pos += wsum;
            total += wsum;
        }
        if (MODE == 0 && lane == 0) counts[sg] = total;
    }
    if (lds) {
        __syncthreads();
        for (int k = threadIdx.x; k < nlines; k += BUF_THREADS)
            if (h[k]) atomicAdd(&lcount[k], (unsigned long long)h[k]);
    }
}

__global__ void k_bufj_zero(int64_t n, unsigned long long *p)
{
    const int64_t nth = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += nth) p[i] = 0ull;
}

int buffer_join_lines(spade_ctx *ctx, const spade_points *pts, const spade_polys *lines, const double *r,
                      double r_all, uint32_t *out_pt, uint32_t *out_line, int64_t cap, int64_t *n_out,
                      uint64_t *out_counts)
{
    hipStream_t st = ctx->stream;
    if (n_out) *n_out = 0;
    const bool counting = out_counts != nullptr;
    if (!r && !(std::isfinite(r_all) && r_all >= 0.0))
        return set_error(ctx, SPADE_E_INVALID, "the distance must be finite and >= 0");
    if (!counting) {
        if (cap < 0) return set_error(ctx, SPADE_E_INVALID, "negative capacity");
        if (cap > 0 && (!out_pt || !out_line)) return set_error(ctx, SPADE_E_INVALID, "output array is NULL");
    }
    if (!lines) return set_error(ctx, SPADE_E_INVALID, "line set is NULL");
    const int64_t R = lines->n_rings;
    if (R < 0) return set_error(ctx, SPADE_E_INVALID, "negative ring count");
    if (R >= 0x7fffffffLL) return set_error(ctx, SPADE_E_TOO_LARGE, "line ids must be < 2^31 - 1");
    if (R > 0 && (!lines->ring_vtx_off || !lines->vx || !lines->vy))
        return set_error(ctx, SPADE_E_INVALID, "line array is NULL");
    int64_t V = 0;
    if (R > 0) {
        if (lines->n_vertices > 0) {
            V = lines->n_vertices;
        } else {
            int64_t *hv = (int64_t *)ensure_pinned(ctx, 64);
            if (!hv) return set_error(ctx, SPADE_E_NOMEM, "pinned staging allocation failed");
            SPADE_HIP(ctx, hipMemcpyAsync(hv, lines->ring_vtx_off + R, sizeof(int64_t), hipMemcpyDeviceToHost, st));
            SPADE_HIP(ctx, hipStreamSynchronize(st));
            V = hv[0];
        }
        if (V < 0 || V >= (int64_t)0xffffffffLL) return set_error(ctx, SPADE_E_INVALID, "bad vertex count");
    }
    const int64_t n = pts->n;
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, ctx->device) != hipSuccess || cus <= 0)
        cus = 256;
    if (counting && R > 0)
        hipLaunchKernelGGL(k_bufj_zero, dim3((unsigned)std::min<int64_t>((R + 255) / 256, 4096)), dim3(256), 0, st, R,
                           (unsigned long long *)out_counts);

    DevBuf &bs = ctx->scratch[S_BUF_SEGS], &bg = ctx->scratch[S_BUF_GRID];
    if (ensure(ctx, bs, sizeof(JSeg) * (size_t)std::max<int64_t>(V, 1) + (size_t)V + 16) || ensure(ctx, bg, 256))
        return SPADE_E_NOMEM;
    JSeg *segs = (JSeg *)bs.p;
    uint8_t *valid = (uint8_t *)(segs + std::max<int64_t>(V, 1));
    unsigned long long *bb = (unsigned long long *)bg.p;
    unsigned *err = (unsigned *)(bb + 4);
    double *dlen = (double *)(bb + 6);
    SPADE_HIP(ctx, hipMemsetAsync(bb, 0xff, 8 * sizeof(unsigned long long), st));
    SPADE_HIP(ctx, hipMemsetAsync(bb + 4, 0, 3 * sizeof(unsigned long long), st));
    if (R > 0) {
        const int sgrid = (int)std::max<int64_t>(1, std::min<int64_t>((std::max(V, R + 1) + 255) / 256, (int64_t)cus * 8));
        hipLaunchKernelGGL(k_bufj_segs, dim3(sgrid), dim3(256), 0, st, R, lines->ring_vtx_off, V, lines->vx, lines->vy,
                           r, r_all, segs, valid, bb, err, dlen);
        SPADE_HIP(ctx, hipGetLastError());
    }
    unsigned long long *h = (unsigned long long *)ensure_pinned(ctx, 64);
    if (!h) return set_error(ctx, SPADE_E_NOMEM, "pinned staging allocation failed");
    SPADE_HIP(ctx, hipMemcpyAsync(h, bb, 8 * sizeof(unsigned long long), hipMemcpyDeviceToHost, st));
    SPADE_HIP(ctx, hipStreamSynchronize(st));
    const unsigned ef = (unsigned)(h[4] & 0xffffffffu);
    if (ef & 1u) return set_error(ctx, SPADE_E_INVALID, "ring offsets are not a valid CSR array");
    if (ef & 2u) return set_error(ctx, SPADE_E_INVALID, "a vertex coordinate is not finite");
    if (ef & 4u) return set_error(ctx, SPADE_E_INVALID, "a line's distance is not finite and >= 0");
    const bool any = h[0] != ~0ull;
    double len_sum;
    std::memcpy(&len_sum, &h[6], sizeof len_sum);
    const double rmax = any ? -buf_from_key(h[7]) : 0.0;
    if (n == 0) return SPADE_OK;

    BufGrid grid{0.0, 0.0, -1.0, -1.0, 1.0, 1.0, 1, 1};   // empty box: no point is tested
    double magpad = 0.0;
    uint32_t *off = nullptr;
    JSeg *list = nullptr;
    if (any) {
        const double x0 = buf_from_key(h[0]), x1 = -buf_from_key(h[1]);
        const double y0 = buf_from_key(h[2]), y1 = -buf_from_key(h[3]);
        const double mag = std::fabs(x0) + std::fabs(x1) + std::fabs(y0) + std::fabs(y1);
        magpad = mag * 0x1p-40 + 1e-300;
        const double pad = rmax * (1.0 + 0x1p-40) + magpad;
        const double X0 = x0 - pad, X1 = x1 + pad, Y0 = y0 - pad, Y1 = y1 + pad;
        const double w = X1 - X0, hgt = Y1 - Y0;
        const double lmean = std::isfinite(len_sum) ? len_sum / (double)std::max<int64_t>(V, 1) : 0.0;
        double cell = std::max(rmax, std::min(lmean, std::sqrt(w * hgt / (2.0 * (double)std::max<int64_t>(V, 1)))));
        cell = std::max(cell, std::max(w, hgt) / BUF_GRID_MAX);
        if (!(cell > 1e-290)) cell = 1.0;
        grid.X0 = X0; grid.Y0 = Y0; grid.X1 = X1; grid.Y1 = Y1;
        grid.inv = 1.0 / cell;
        grid.cell = cell;
        grid.gx = (int)std::min<double>(BUF_GRID_MAX, std::max(1.0, std::ceil(w * grid.inv)));
        grid.gy = (int)std::min<double>(BUF_GRID_MAX, std::max(1.0, std::ceil(hgt * grid.inv)));
        const int64_t G = (int64_t)grid.gx * grid.gy;
        if (ensure(ctx, bg, 256 + sizeof(uint32_t) * 3 * (size_t)(G + 1))) return SPADE_E_NOMEM;
        bb = (unsigned long long *)bg.p;
        uint32_t *cnt = (uint32_t *)((unsigned char *)bg.p + 256);
        off = cnt + (G + 1);
        uint32_t *cursor = off + (G + 1);
        unsigned long long *tot = bb + 5;
        SPADE_HIP(ctx, hipMemsetAsync(cnt, 0, sizeof(uint32_t) * (size_t)(G + 1), st));
        SPADE_HIP(ctx, hipMemsetAsync(tot, 0, sizeof(unsigned long long), st));
        const int bgrid = (int)std::max<int64_t>(1, std::min<int64_t>((V + 255) / 256, (int64_t)cus * 8));
        hipLaunchKernelGGL(k_bufj_bin<false>, dim3(bgrid), dim3(256), 0, st, V, (const JSeg *)segs,
                           (const uint8_t *)valid, grid, magpad, cnt, (const uint32_t *)nullptr,
                           (unsigned long long *)nullptr, (uint32_t *)nullptr, tot);
        SPADE_HIP(ctx, hipGetLastError());
        DevBuf &bt = ctx->scratch[S_BUF_TMP];
        size_t tb = 0;
        SPADE_HIP(ctx, hipcub::DeviceScan::ExclusiveSum(nullptr, tb, cnt, off, (int)(G + 1), st));
        if (ensure(ctx, bt, std::max<size_t>(tb, 1))) return SPADE_E_NOMEM;
        SPADE_HIP(ctx, hipcub::DeviceScan::ExclusiveSum(bt.p, tb, cnt, off, (int)(G + 1), st));
        SPADE_HIP(ctx, hipMemcpyAsync(h, tot, sizeof(unsigned long long), hipMemcpyDeviceToHost, st));
        SPADE_HIP(ctx, hipStreamSynchronize(st));
        if (h[0] >= ((unsigned long long)1 << 26))
            return set_error(ctx, SPADE_E_TOO_LARGE, "too many (segment, cell) entries: the distances are too "
                                                     "large for the segments' spread");
        const int64_t total = (int64_t)h[0];
        // cell lists: sort keys and values, sorted copies of the segments
        DevBuf &bl = ctx->scratch[S_BUF_LIST];
        const size_t keyb = sizeof(unsigned long long) * (size_t)std::max<int64_t>(total, 1);
        const size_t valb = sizeof(uint32_t) * (size_t)std::max<int64_t>(total, 1);
        const size_t listb = sizeof(JSeg) * (size_t)std::max<int64_t>(total, 1);
        if (ensure(ctx, bl, 2 * keyb + 2 * valb + listb + 64)) return SPADE_E_NOMEM;
        unsigned long long *k1 = (unsigned long long *)bl.p, *k2 = k1 + std::max<int64_t>(total, 1);
        uint32_t *v1 = (uint32_t *)(k2 + std::max<int64_t>(total, 1)), *v2 = v1 + std::max<int64_t>(total, 1);
        list = (JSeg *)(((uintptr_t)(v2 + std::max<int64_t>(total, 1)) + 15) & ~(uintptr_t)15);
        SPADE_HIP(ctx, hipMemsetAsync(cursor, 0, sizeof(uint32_t) * (size_t)(G + 1), st));
        hipLaunchKernelGGL(k_bufj_bin<true>, dim3(bgrid), dim3(256), 0, st, V, (const JSeg *)segs,
                           (const uint8_t *)valid, grid, magpad, cursor, (const uint32_t *)off, k1, v1,
                           (unsigned long long *)nullptr);
        SPADE_HIP(ctx, hipGetLastError());
        if (total > 0) {
            int cb = 1;
            while (cb < 40 && ((uint64_t)(G - 1) >> cb) != 0) ++cb;
            size_t sb = 0;
            SPADE_HIP(ctx, hipcub::DeviceRadixSort::SortPairs(nullptr, sb, (const unsigned long long *)k1, k2,
                                                              (const uint32_t *)v1, v2, (int)total, 0, 32 + cb, st));
            if (ensure(ctx, bt, std::max<size_t>(sb, 1))) return SPADE_E_NOMEM;
            SPADE_HIP(ctx, hipcub::DeviceRadixSort::SortPairs(bt.p, sb, (const unsigned long long *)k1, k2,
                                                              (const uint32_t *)v1, v2, (int)total, 0, 32 + cb, st));
            const int ggrid = (int)std::max<int64_t>(1, std::min<int64_t>((total + 255) / 256, (int64_t)cus * 8));
            hipLaunchKernelGGL(k_bufj_gather, dim3(ggrid), dim3(256), 0, st, (int64_t)total, (const uint32_t *)v2,
                               (const JSeg *)segs, list);
            SPADE_HIP(ctx, hipGetLastError());
        }
    }

    const int64_t nseg = (n + EMIT_SEG - 1) / EMIT_SEG;
    const int64_t wpb = BUF_THREADS / 64;
    const int gridp = (int)std::max<int64_t>(1, std::min<int64_t>((nseg + wpb - 1) / wpb, (int64_t)cus * 2));
    if (ctx->timing) SPADE_HIP(ctx, hipEventRecord(ctx->ev[2], st));
    if (counting) {
        constexpr int HIST = 16384;
        const size_t lds = R <= HIST ? sizeof(uint32_t) * (size_t)std::max<int64_t>(R, 1) : 0;
        SPADE_HIP(ctx, hipFuncSetAttribute((const void *)k_bufj_pairs<2>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)std::max<size_t>(lds, 4)));
        hipLaunchKernelGGL(k_bufj_pairs<2>, dim3(gridp), dim3(BUF_THREADS), lds, st, n, pts->x, pts->y, grid,
                           (const uint32_t *)off, (const JSeg *)list, magpad, nseg, (unsigned long long *)nullptr,
                           (const unsigned long long *)nullptr, (uint32_t *)nullptr, (uint32_t *)nullptr, (int64_t)0,
                           (unsigned long long *)out_counts, (int)R, HIST, (uint32_t *)nullptr);
        SPADE_HIP(ctx, hipGetLastError());
        if (ctx->timing) SPADE_HIP(ctx, hipEventRecord(ctx->ev[3], st));
        SPADE_HIP(ctx, hipStreamSynchronize(st));
        return SPADE_OK;
    }
    DevBuf &lb = ctx->scratch[S_LOOKBACK];
    if (ensure(ctx, lb, sizeof(unsigned long long) * 2 * (size_t)(nseg + 1))) return SPADE_E_NOMEM;
    unsigned long long *counts = (unsigned long long *)lb.p;
    unsigned long long *offs = counts + (nseg + 1);
    // pairs per point, kept by the count pass for the write pass (without the
    // room, the write pass counts again)
    DevBuf &pb = ctx->scratch[S_BITS];
    uint32_t *pcount = nullptr;
    if (cap > 0) {
        if (ensure(ctx, pb, sizeof(uint32_t) * (size_t)n) == SPADE_OK) pcount = (uint32_t *)pb.p;
        else ctx->err.clear();
    }
    hipLaunchKernelGGL(k_bufj_pairs<0>, dim3(gridp), dim3(BUF_THREADS), 0, st, n, pts->x, pts->y, grid,
                       (const uint32_t *)off, (const JSeg *)list, magpad, nseg, counts,
                       (const unsigned long long *)nullptr, (uint32_t *)nullptr, (uint32_t *)nullptr, (int64_t)0,
                       (unsigned long long *)nullptr, (int)R, 0, pcount);
    hipLaunchKernelGGL(k_buf_zero, dim3(1), dim3(1), 0, st, counts + nseg);
    SPADE_HIP(ctx, hipGetLastError());
    DevBuf &bt = ctx->scratch[S_BUF_TMP];
    size_t tb = 0;
    SPADE_HIP(ctx, hipcub::DeviceScan::ExclusiveSum(nullptr, tb, counts, offs, (int)(nseg + 1), st));
    if (ensure(ctx, bt, std::max<size_t>(tb, 1))) return SPADE_E_NOMEM;
    SPADE_HIP(ctx, hipcub::DeviceScan::ExclusiveSum(bt.p, tb, counts, offs, (int)(nseg + 1), st));
    if (cap > 0) {
        hipLaunchKernelGGL(k_bufj_pairs<1>, dim3(gridp), dim3(BUF_THREADS), 0, st, n, pts->x, pts->y, grid,
                           (const uint32_t *)off, (const JSeg *)list, magpad, nseg, (unsigned long long *)nullptr,
                           (const unsigned long long *)offs, out_pt, out_line, cap, (unsigned long long *)nullptr,
                           (int)R, 0, pcount);
        SPADE_HIP(ctx, hipGetLastError());
    }
    if (ctx->timing) SPADE_HIP(ctx, hipEventRecord(ctx->ev[3], st));
    SPADE_HIP(ctx, hipMemcpyAsync(h, offs + nseg, sizeof(unsigned long long), hipMemcpyDeviceToHost, st));
    SPADE_HIP(ctx, hipStreamSynchronize(st));
    if (n_out) *n_out = (int64_t)h[0];
    if ((int64_t)h[0] > cap) return set_error(ctx, SPADE_E_CAPACITY, "output capacity too small");
    return SPADE_OK;
}

}  // namespace spade
