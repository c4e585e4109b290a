// Distance joins between a point set and a set of disks (Sec. 4.2,
// canvases for distance-based queries; Sec. 5.2, distance-based joins):
//   type (1): all pairs (point i, disk j) with |p_i - c_j| <= r (one radius);
//   type (2): the same with a radius r_j per disk.
// Counts per disk (the aggregation over the join) come from the same probe.
//
// The disks play the paper's constraint canvases: a grid of cells over the
// disks' union box whose cells list the disks that can reach them (the
// boundary index of the disk set, ascending disk ids), those that hold the
// whole cell marked.  A marked disk is a pair of every point of the cell, any
// other listed one gets the exact closed-disk predicate, so results are exact
// and independent of the grid.  Pairs come out ascending
// by (point id, disk id) from the paper's two-step Map (count pass per
// wavefront segment, scan, write pass), with no sort.  The disk tests of a
// wavefront's points are spread over its lanes (wave_round), so that a
// wavefront's rounds follow its candidates in total rather than its longest
// list.
#include "common.h"
#include "disk.h"
#include "wavewalk.h"

#include <hipcub/hipcub.hpp>
#include <rocprim/warp/warp_reduce.hpp>
#include <rocprim/warp/warp_scan.hpp>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

namespace spade {

constexpr int DJ_THREADS = 256;
constexpr int DJ_ROUNDS = 8;                  // 64-point rounds per wavefront segment
constexpr int64_t DJ_SEG = 64 * DJ_ROUNDS;
constexpr int DJ_GRID_MAX = 4096;             // cells per grid side
constexpr int DJ_HIST_MAX = 8192;             // disks counted in LDS
constexpr uint32_t DJ_FULL = 0x80000000u;     // in a cell's entry: the disk holds the whole cell
// With many points the cells are finer than the mean radius: down to this
// fraction of it, while the table has at most n / DJ_PER_CELL cells and the
// lists about n / DJ_PER_ENTRY entries (both cost a pass each, the points
// the tests that they save).
constexpr double DJ_COVER = 0.0625;           // disks over a position on average, at least, for that
constexpr double DJ_STACK = 32.0;             // and at most (longer lists have no masks)
constexpr double DJ_FINE = 4.0, DJ_PER_CELL = 8.0, DJ_PER_ENTRY = 8.0;
constexpr unsigned DJ_LIST_SORT = 16;         // longest list ordered by one lane
constexpr unsigned DJ_LIST_WAVE = 256;        // by a wavefront
constexpr unsigned DJ_LIST_WG = 2048;         // by a workgroup
constexpr int DJ_QCAP = 64;                   // queued points per wavefront
constexpr int DJ_QWAVE = DJ_QCAP * 28;        // x, y, entries, place: bytes per wavefront
constexpr uint32_t DJ_STAGE = 512;            // pairs listed per wavefront before they are stored
constexpr int DJ_GROUP = 4;                   // words of points in flight

struct DiskGrid {
    double X0, Y0, sx, sy;   // cell (floor((x - X0) * sx), floor((y - Y0) * sy))
    double bx0, by0, bx1, by1;   // closed box of all disks
    int W, H;
};

struct DiskArgs {
    const double *cx, *cy, *r;   // r: per-disk radii or NULL
    double r_all;
};

__device__ __forceinline__ double radius_of(const DiskArgs &D, int64_t j)
{
    return D.r ? D.r[j] : D.r_all;
}

// Validation and union box: flags bit 0 = a non-finite centre or radius or a
// negative radius; box as order keys (min x, -max x, min y, -max y) of the
// disks' extents, and the sums of the radii and of their squares.
__device__ __forceinline__ unsigned long long okey_d(double v)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    return (b & 0x8000000000000000ull) ? ~b : (b | 0x8000000000000000ull);
}

__global__ __launch_bounds__(256) void k_disks_box(int64_t n, DiskArgs D, unsigned long long *bb, unsigned *bad,
                                                   double *rsum)
{
    __shared__ unsigned long long s[4][256];
    __shared__ double sr[256], sq[256];
    unsigned long long k0 = ~0ull, k1 = ~0ull, k2 = ~0ull, k3 = ~0ull;
    double rs = 0.0, rq = 0.0;
    unsigned nb = 0;
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n; j += (int64_t)gridDim.x * blockDim.x) {
        const double cx = D.cx[j], cy = D.cy[j], r = radius_of(D, j);
        if (!(isfinite(cx) && isfinite(cy) && isfinite(r) && r >= 0.0)) { nb = 1; continue; }
        k0 = min(k0, okey_d(cx - r)); k1 = min(k1, okey_d(-(cx + r)));
        k2 = min(k2, okey_d(cy - r)); k3 = min(k3, okey_d(-(cy + r)));
        rs += r;
        rq += r * r;
    }
    if (nb) atomicOr(bad, 1u);
    s[0][threadIdx.x] = k0; s[1][threadIdx.x] = k1; s[2][threadIdx.x] = k2; s[3][threadIdx.x] = k3;
    sr[threadIdx.x] = rs;
    sq[threadIdx.x] = rq;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            for (int q = 0; q < 4; ++q) s[q][threadIdx.x] = min(s[q][threadIdx.x], s[q][threadIdx.x + w]);
            sr[threadIdx.x] += sr[threadIdx.x + w];
            sq[threadIdx.x] += sq[threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x < 4) atomicMin(&bb[threadIdx.x], s[threadIdx.x][0]);
    if (threadIdx.x == 0) {
        atomicAdd(rsum, sr[0]);
        atomicAdd(rsum + 1, sq[0]);
    }
}

// Cells a disk can reach: its box widened by one cell (so that rounding in a
// point's cell index never loses a candidate), without the cells whose
// (slightly enlarged) square lies entirely outside the disk.
__device__ __forceinline__ void disk_cells(const DiskGrid &g, double cx, double cy, double r, int &c0, int &c1,
                                           int &r0, int &r1)
{
    c0 = (int)fmax(0.0, floor((cx - r - g.X0) * g.sx) - 1.0);
    c1 = (int)fmin((double)(g.W - 1), floor((cx + r - g.X0) * g.sx) + 1.0);
    r0 = (int)fmax(0.0, floor((cy - r - g.Y0) * g.sy) - 1.0);
    r1 = (int)fmin((double)(g.H - 1), floor((cy + r - g.Y0) * g.sy) + 1.0);
}

// Whether the disk reaches the cell (0: no, 1: yes) or holds all of it (2).
// lim scales r^2 for the second: below 1 by far more than the rounding of the
// corners, or negative where a cell is too small beside its coordinates for
// the quarter cell to cover the rounding of a point's index.
__device__ __forceinline__ int cell_reached(const DiskGrid &g, double ux, double uy, double cx, double cy, double r,
                                            double lim, int c, int rr)
{
#pragma clang fp contract(off)   // the count and the fill pass decide alike
    // the cell's square enlarged by a quarter cell on every side
    const double x0 = g.X0 + ((double)c - 0.25) * ux, x1 = g.X0 + ((double)c + 1.25) * ux;
    const double y0 = g.Y0 + ((double)rr - 0.25) * uy, y1 = g.Y0 + ((double)rr + 1.25) * uy;
    const double dx = fmax(fmax(x0 - cx, cx - x1), 0.0), dy = fmax(fmax(y0 - cy, cy - y1), 0.0);
    if (!(dx * dx + dy * dy <= r * r * 1.0000001)) return 0;
    const double fx = fmax(x1 - cx, cx - x0), fy = fmax(y1 - cy, cy - y0);
    const double f2 = fx * fx + fy * fy, l2 = r * r * lim;
    return l2 > 1e-280 && f2 <= l2 && f2 < 1e280 ? 2 : 1;
}

// The cells of every disk, a wavefront per disk (the cells of its box are
// spread over the lanes, so that a disk much larger than the others is not
// one lane's loop).  CELL_COUNT: the entries of every cell, and of all in
// total's shards (2,048 workgroups adding to one word took 20 us of 28);
// CELL_LIST: the entries into the cells' lists, in any order; CELL_KEYS:
// the same as keys, cell << 32 | disk << 1 | the disk holds the whole cell.
// FEW: at most DJ_FEW_CELLS cells, where many disks meet in one; a workgroup
// counts its disks in LDS and adds to a cell once (500 disks on one spot: 8
// and 22 us for counts and lists with an atomic per entry, 6 and 8 so).
enum { CELL_COUNT, CELL_KEYS, CELL_LIST };
constexpr int DJ_SHARDS = 16, DJ_SHARD_WORDS = 16;
constexpr int DJ_FEW_CELLS = 4096;

template <int STEP, bool FEW>
__global__ __launch_bounds__(256) void k_disk_cells(int64_t n, DiskArgs D, DiskGrid g, double ux, double uy,
                                                    double lim, uint32_t *ccnt, unsigned long long *keys,
                                                    const uint2 *cells, uint32_t *cell_disk, double2 *centre,
                                                    unsigned long long *total)
{
    __shared__ uint32_t hist[FEW ? DJ_FEW_CELLS : 1], base[FEW ? DJ_FEW_CELLS : 1];
    const int lane = threadIdx.x & 63;
    const int64_t nwave = ((int64_t)gridDim.x * blockDim.x) >> 6;
    // fn(disk, cell, reached or held) for the cells of this wavefront's disks
    auto disks = [&](auto fn) {
        for (int64_t j = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6; j < n; j += nwave) {
            const double cx = D.cx[j], cy = D.cy[j], r = radius_of(D, j);
            if (STEP == CELL_COUNT && lane == 0) centre[j] = double2{cx, cy};
            int c0, c1, r0, r1;
            disk_cells(g, cx, cy, r, c0, c1, r0, r1);
            const int wide = c1 - c0 + 1;
            const int64_t all = wide > 0 && r1 >= r0 ? (int64_t)wide * (r1 - r0 + 1) : 0;
            for (int64_t t0 = 0; t0 < all; t0 += 64) {
                const int64_t t = t0 + lane;
                const int rr = r0 + (int)(t / wide), c = c0 + (int)(t % wide);
                const int in = t < all ? cell_reached(g, ux, uy, cx, cy, r, lim, c, rr) : 0;
                fn(j, (int64_t)rr * g.W + c, in);
            }
        }
    };
    auto put = [&](int64_t j, int64_t cell, int in, uint32_t p) {
        if (STEP == CELL_KEYS)
            keys[cells[cell].x + p] =
                ((unsigned long long)cell << 32) | ((unsigned long long)j << 1) | (in == 2 ? 1ull : 0ull);
        if (STEP == CELL_LIST) cell_disk[cells[cell].x + p] = (uint32_t)j | (in == 2 ? DJ_FULL : 0u);
    };
    unsigned long long sum = 0;   // wave-uniform
    if (FEW) {
        const int ncell = g.W * g.H;
        for (int c = threadIdx.x; c < ncell; c += 256) hist[c] = 0u;
        __syncthreads();
        disks([&](int64_t, int64_t cell, int in) {
            if (in) atomicAdd(&hist[cell], 1u);
            sum += __popcll(__ballot(in != 0));
        });
        __syncthreads();
        for (int c = threadIdx.x; c < ncell; c += 256) {
            const uint32_t h = hist[c];
            base[c] = h ? atomicAdd(&ccnt[c], h) : 0u;
            hist[c] = 0u;
        }
        __syncthreads();
        if (STEP != CELL_COUNT)
            disks([&](int64_t j, int64_t cell, int in) {
                if (in) put(j, cell, in, base[cell] + atomicAdd(&hist[cell], 1u));
            });
    } else {
        disks([&](int64_t j, int64_t cell, int in) {
            if (in) put(j, cell, in, atomicAdd(&ccnt[cell], 1u));
            sum += __popcll(__ballot(in != 0));
        });
    }
    if (STEP == CELL_COUNT) {
        __shared__ unsigned long long part[4];
        if (lane == 0) part[threadIdx.x >> 6] = sum;
        __syncthreads();
        if (threadIdx.x == 0)
            atomicAdd(&total[(blockIdx.x % DJ_SHARDS) * DJ_SHARD_WORDS], part[0] + part[1] + part[2] + part[3]);
    }
}

// cells[c].x = off[c] (c = 0 .. ncell), *longest = the most entries of a
// cell if that is more than DJ_LIST_SORT (nothing asks below; an atomic per
// wavefront took 50 us); clears the counters for the lists.  The cells of more than
// DJ_LIST_SORT entries are listed in longs, *nlong of them, in any order, and
// the entries of all cells summed from their shards.
__global__ __launch_bounds__(256) void k_dcell_start(int64_t ncell, const uint32_t *off, uint32_t *ccnt, uint2 *cells,
                                                     uint32_t *longs, unsigned *nlong, unsigned *longest,
                                                     const unsigned long long *shards, unsigned long long *total)
{
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int lane = threadIdx.x & 63;
    uint32_t m = 0;
    if (c < ncell) {
        m = ccnt[c];
        ccnt[c] = 0u;
    }
    if (c <= ncell) cells[c] = uint2{off[c], 0u};
    if (c == 0) {
        unsigned long long t = 0ull;
#pragma unroll
        for (int k = 0; k < DJ_SHARDS; ++k) t += shards[k * DJ_SHARD_WORDS];
        *total = t;
    }
    const unsigned long long big = __ballot(m > DJ_LIST_SORT);
    if (big) {
        unsigned at = 0;
        if (lane == 0) at = atomicAdd(nlong, (unsigned)__popcll(big));
        at = (unsigned)__shfl((int)at, 0, 64) + (unsigned)__popcll(big & ((1ull << lane) - 1ull));
        if (m > DJ_LIST_SORT) longs[at] = (uint32_t)c;
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, d, 64));
    if (lane == 0 && m > DJ_LIST_SORT && m > __hip_atomic_load(longest, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        atomicMax(longest, m);
}

// The entries of the listed cells (at most DJ_LIST_WG each) in order of their
// disks: an entry's place is the count of smaller ones, four to an LDS read.  A
// wavefront takes a cell, the workgroup together one of more than DJ_LIST_WAVE.
__global__ __launch_bounds__(256) void k_dcell_sort(const unsigned *nlong, const uint32_t *longs, const uint2 *cells,
                                                    uint32_t *cell_disk)
{
    static_assert(4 * DJ_LIST_WAVE <= DJ_LIST_WG && DJ_LIST_WAVE % 4 == 0, "the wavefronts' lists share the stage");
    __shared__ __align__(16) uint32_t e[DJ_LIST_WG];
    const unsigned nl = *nlong, wv = threadIdx.x >> 6;
    auto order = [&](uint32_t *s, uint32_t k, uint32_t n, uint32_t first, uint32_t step, auto sync) {
        const uint32_t n4 = (n + 3u) & ~3u;
        for (uint32_t i = first; i < n4; i += step) s[i] = i < n ? cell_disk[k + i] : ~0u;   // past every disk
        sync();
        for (uint32_t i = first; i < n; i += step) {
            const uint32_t v = s[i] & ~DJ_FULL;
            uint32_t at = 0u;
#pragma unroll 4
            for (uint32_t j = 0; j < n4; j += 4) {
                const uint4 q = *(const uint4 *)(s + j);
                at += ((q.x & ~DJ_FULL) < v) + ((q.y & ~DJ_FULL) < v) + ((q.z & ~DJ_FULL) < v) + ((q.w & ~DJ_FULL) < v);
            }
            cell_disk[k + at] = s[i];
        }
        sync();
    };
    auto wave_sync = [] {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    for (unsigned q = blockIdx.x * 4 + wv; q < nl; q += gridDim.x * 4) {
        const uint32_t c = longs[q], k = cells[c].x, n = cells[c + 1].x - k;
        if (n <= DJ_LIST_WAVE) order(e + wv * DJ_LIST_WAVE, k, n, threadIdx.x & 63u, 64u, wave_sync);
    }
    __syncthreads();
    for (unsigned q = blockIdx.x; q < nl; q += gridDim.x) {
        const uint32_t c = longs[q], k = cells[c].x, n = cells[c + 1].x - k;
        if (n > DJ_LIST_WAVE) order(e, k, n, threadIdx.x, 256u, [] { __syncthreads(); });
    }
}

// The entries of sorted keys.
__global__ void k_dcell_list(int64_t nk, const unsigned long long *skeys, uint32_t *cell_disk)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nk; i += (int64_t)gridDim.x * blockDim.x)
        cell_disk[i] = (uint32_t)(skeys[i] & 0xffffffffull) >> 1 | (skeys[i] & 1ull ? DJ_FULL : 0u);
}

// cells[c].y = which of the cell's entries hold all of it, for a cell of at
// most 32; first, with sort, the entries of a cell of at most DJ_LIST_SORT in
// order of their disks, a lane per cell, by insertion in LDS (in place, 51 us
// for lists of 24: a step waits for a load).
__global__ __launch_bounds__(128) void k_dcell_full(int64_t ncell, uint2 *cells, uint32_t *cell_disk, int sort)
{
    __shared__ uint32_t s[DJ_LIST_SORT][128];
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int t = threadIdx.x;
    if (c >= ncell) return;
    const uint32_t k = cells[c].x, have = cells[c + 1].x - k, m = have > 32u ? 0u : have;
    uint32_t full = 0;
    if (sort && have <= DJ_LIST_SORT) {
        bool moved = false;
        uint32_t last = 0;   // the entry before, in order
        for (uint32_t i0 = 0; i0 < have; i0 += 4) {
            uint32_t in[4];
#pragma unroll
            for (uint32_t u = 0; u < 4; ++u) in[u] = i0 + u < have ? cell_disk[k + i0 + u] : 0u;
#pragma unroll
            for (uint32_t u = 0; u < 4; ++u) {
                if (i0 + u >= have) break;
                const uint32_t e = in[u];
                uint32_t p = i0 + u;
                if (p == 0 || (last & ~DJ_FULL) < (e & ~DJ_FULL)) {
                    last = e;
                } else {
                    moved = true;
                    for (; p > 0 && (s[p - 1][t] & ~DJ_FULL) > (e & ~DJ_FULL); --p) s[p][t] = s[p - 1][t];
                }
                s[p][t] = e;
            }
        }
        for (uint32_t i = 0; i < have; ++i) {
            const uint32_t e = s[i][t];
            if (moved) cell_disk[k + i] = e;
            full |= (e >> 31) << i;
        }
    } else {
#pragma unroll 8
        for (uint32_t i = 0; i < m; ++i) full |= (cell_disk[k + i] >> 31) << i;
    }
    if (full) cells[c].y = full;
}

struct DiskCanvas {
    DiskGrid g;
    const uint32_t *off;         // the cells' first entries; one past the last cell
    const uint2 *cells;          // the same, and which of the first 32 entries hold the cell
    const uint32_t *cell_disk;   // the cells' entries: disk ids ascending, DJ_FULL
    const double2 *centre;       // the disks' centres, one load each
    unsigned longest;            // most entries of a cell (0: at most DJ_LIST_SORT)
    bool together;               // points of short and long lists are walked together
    DiskArgs D;
};

// The cell of a point, or -1 outside the disks' box (NaN fails the test too).
__device__ __forceinline__ int disk_cell(const DiskCanvas &K, double x, double y)
{
    if (!(K.g.bx0 <= x && x <= K.g.bx1 && K.g.by0 <= y && y <= K.g.by1)) return -1;
    const int c = min((int)((x - K.g.X0) * K.g.sx), K.g.W - 1);
    const int r = min((int)((y - K.g.Y0) * K.g.sy), K.g.H - 1);
    return max(r, 0) * K.g.W + max(c, 0);   // at most DJ_GRID_MAX^2 cells
}

// A cell's record and its neighbour's in one load.
struct alignas(8) CellPair {
    uint2 a, b;
};

// The candidates of point (x, y): its cell's disks cell_disk[k, k + rem).
// From the offsets alone, half the table: counts of 100 disks over 30M points
// 212 us, 255 from the cells' records.
__device__ __forceinline__ void disk_range(const DiskCanvas &K, double x, double y, uint32_t &k, uint32_t &rem)
{
    const int cell = disk_cell(K, x, y);
    k = rem = 0u;
    if (cell < 0) return;
    k = K.off[cell];
    rem = K.off[cell + 1] - k;
}

// The (point, disk) pairs of a wavefront's points with the disk tests
// balanced over the lanes: for each pair the testing lane calls pair(o,
// slot, j) with o the point's lane and slot = base of lane o + the pair's
// rank among the point's pairs (ascending disk id, the order of the cell
// lists); on return cnt holds the number of pairs of this lane's point.
// Called by every lane of the wavefront.
template <typename Pair>
__device__ __forceinline__ void disk_wave_walk(const DiskCanvas &K, double x, double y, uint32_t k, uint32_t rem,
                                               uint32_t base, int lane, uint32_t &cnt, Pair &&pair)
{
    cnt = 0u;
    while (__ballot(rem != 0u)) {
        const WaveRound w = wave_round(rem, lane);
        const uint32_t ok = __shfl(k, w.o, 64);
        const uint32_t ocnt = __shfl(cnt, w.o, 64);
        const uint32_t obase = __shfl(base, w.o, 64);
        const double ox = __shfl(x, w.o, 64), oy = __shfl(y, w.o, 64);
        bool h = false;
        uint32_t j = 0u;
        if ((uint32_t)lane < w.ntake) {
            j = K.cell_disk[ok + ((uint32_t)lane - w.opre)];
            h = (j & DJ_FULL) != 0u;
            j &= ~DJ_FULL;
            if (!h) {
                const double rj = radius_of(K.D, j);
                h = in_disk(ox, oy, K.D.cx[j], K.D.cy[j], rj, rj * rj);
            }
        }
        const unsigned long long hm = __ballot(h);
        if (h) pair(w.o, obase + ocnt + (uint32_t)__popcll(hm & wave_round_before(w, lane)), j);
        cnt += (uint32_t)__popcll(hm & wave_round_mask(w));
        const uint32_t len = wave_round_len(w);
        k += len;
        rem -= len;
    }
}

// Which of the first 32 entries of this lane's cell (from k on) whose bits are
// in pm hold its point, the tests balanced over the lanes (wave_round).
// Without EXACT, a test that the floating-point filter leaves open sets `open`
// (for the whole wavefront) and counts as outside.  Called by every lane of
// the wavefront.
template <bool EXACT>
__device__ __forceinline__ uint32_t disk_mask_walk(const DiskCanvas &K, double x, double y, uint32_t k, uint32_t pm,
                                                   int lane, bool &open)
{
    uint32_t hits = 0u, rem = (uint32_t)__popc(pm), done = 0u;
    // without entries that hold the cell, the masks have no gaps
    const bool gaps = __ballot((pm & (pm + 1u)) != 0u) != 0ull;
    while (__ballot(rem != 0u)) {
        const WaveRound w = wave_round(rem, lane);
        const uint32_t ok = __shfl(k, w.o, 64);
        uint32_t opm = __shfl(gaps ? pm : done, w.o, 64);
        const double ox = __shfl(x, w.o, 64), oy = __shfl(y, w.o, 64);
        int h = 0;
        if ((uint32_t)lane < w.ntake) {
            uint32_t at = opm + (uint32_t)lane - w.opre;
            if (gaps) {   // few bits where disks hold cells
                for (uint32_t t = (uint32_t)lane - w.opre; t != 0u; --t) opm &= opm - 1u;
                at = (uint32_t)__ffs(opm) - 1u;
            }
            const uint32_t j = K.cell_disk[ok + at] & ~DJ_FULL;
            const double rj = radius_of(K.D, j);
            const double2 c = K.centre[j];
            h = EXACT ? (in_disk(ox, oy, c.x, c.y, rj, rj * rj) ? 1 : 0) : in_disk_filter(ox, oy, c.x, c.y, rj * rj);
        }
        const unsigned long long hm = __ballot(h > 0);
        if (!EXACT && __ballot(h < 0)) open = true;
        const uint32_t len = wave_round_len(w);
        uint32_t got = len ? (uint32_t)(hm >> w.pre) : 0u;
        if (gaps) {
            for (uint32_t t = 0; t < len; ++t) {
                const uint32_t low = pm & (0u - pm);
                if (got & 1u) hits |= low;
                got >>= 1;
                pm ^= low;
            }
        } else if (len) {
            hits |= (got & (~0u >> (32u - len))) << done;
            done += len;
        }
        rem -= len;
    }
    return hits;
}

// Count pass: pairs per wavefront segment, and with pm every point's pairs as
// (first entry of its cell, mask of the entries that hold it), or (all ones,
// number) for a cell of more than 32 entries and the points tested with such
// ones, so that the write pass reads 8 bytes per point and tests nothing else.
// A point's entries that hold its whole cell are pairs as they stand; points
// with others are queued in LDS and tested 64 at a time.  Bound by the rate of
// L2 requests (the cells, and an entry and a centre per test): 30M points,
// 10,000 disks of 300 m, 0.52 ms with cells of 75 m (0.95 with cells of 300 m
// and every candidate tested a word at a time).  The exact test costs registers
// (106 against 90), so a first pass (EXACT false) decides by the filter and
// leaves DJ_OPEN as the count of a segment in which a test stayed open, a second
// one (EXACT and ONLY_OPEN) does those segments again.
constexpr unsigned long long DJ_OPEN = ~0ull;
constexpr int64_t DJ_FILTER_MIN = 1 << 20;   // points from which the second launch (5 us) pays

template <bool EXACT, bool ONLY_OPEN>
__global__ __launch_bounds__(DJ_THREADS) void k_dj_count(DiskCanvas K, int64_t n, const double *X, const double *Y,
                                                         int64_t nseg, unsigned long long *counts, uint2 *pm)
{
    static_assert(DJ_ROUNDS % DJ_GROUP == 0 && DJ_SEG <= 65536 && DJ_QWAVE % 8 == 0, "queue layout");
    __shared__ __align__(16) unsigned char smem[DJ_THREADS / 64 * DJ_QWAVE];
    const int lane = threadIdx.x & 63;
    const unsigned long long below = (1ull << lane) - 1ull;
    unsigned char *q = smem + (threadIdx.x >> 6) * DJ_QWAVE;
    double *qx = (double *)q, *qy = qx + DJ_QCAP;
    uint32_t *qk = (uint32_t *)(qy + DJ_QCAP), *qf = qk + DJ_QCAP, *qi = qf + DJ_QCAP;
    const int64_t nwave = ((int64_t)gridDim.x * DJ_THREADS) >> 6;
    for (int64_t sg = ((int64_t)blockIdx.x * DJ_THREADS + threadIdx.x) >> 6; sg < nseg; sg += nwave) {
        if (ONLY_OPEN && counts[sg] != DJ_OPEN) continue;
        const int64_t i0 = sg * DJ_SEG;
        bool open = false;              // wave-uniform
        unsigned long long total = 0;   // this lane's pairs
        uint32_t qn = 0;                // wave-uniform
        auto drain = [&]() {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            double x = NAN, y = NAN;
            uint32_t k = 0u, rem = 0u, full = 0u, id = 0u;
            if (lane < (int)qn) {
                x = qx[lane];
                y = qy[lane];
                k = qk[lane];
                full = qf[lane];
                id = qi[lane] & 0xffffu;
                rem = qi[lane] >> 16;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            // Points of lists of more than 32 are walked and counted, and with
            // few points or no cells inside disks (whose masks save tests) the
            // others of the queue with them: 300,000 points near 2,000 disks,
            // lists of both kinds, 62 us, two walks 120; 30M points near disks
            // of all sizes, the call 1.56 ms and 1.43.
            const bool some = __ballot(rem > 32u) != 0ull;
            const bool many = some && (rem > 32u || K.together);
            const uint32_t all = rem >= 32u ? ~0u : (1u << rem) - 1u;
            uint32_t hits = full | disk_mask_walk<EXACT>(K, x, y, k, many ? 0u : all & ~full, lane, open);
            uint32_t m = (uint32_t)__popc(hits);
            if (!EXACT && some) open = true;
            if (EXACT && some) {
                uint32_t cnt;
                disk_range(K, x, y, k, rem);   // the queue holds no more than 33
                disk_wave_walk(K, x, y, k, many ? rem : 0u, 0u, lane, cnt, [](int, uint32_t, uint32_t) {});
                if (many) {
                    k = ~0u;
                    hits = m = cnt;
                }
            }
            if (lane < (int)qn) {
                total += m;
                if (pm) pm[i0 + id] = uint2{k, hits};
            }
            qn = 0;
        };
#pragma nounroll
        for (int g0 = 0; g0 < DJ_ROUNDS; g0 += DJ_GROUP) {
            double xs[DJ_GROUP], ys[DJ_GROUP];
#pragma unroll
            for (int k = 0; k < DJ_GROUP; ++k) {
                const int64_t i = i0 + 64 * (g0 + k) + lane;
                xs[k] = i < n ? __builtin_nontemporal_load(X + i) : NAN;
                ys[k] = i < n ? __builtin_nontemporal_load(Y + i) : NAN;
            }
            uint2 a[DJ_GROUP];
            uint32_t rem[DJ_GROUP];
#pragma unroll
            for (int k = 0; k < DJ_GROUP; ++k) {
                const int c = disk_cell(K, xs[k], ys[k]);
                const CellPair p = c >= 0 ? *(const CellPair *)(K.cells + c) : CellPair{{0u, 0u}, {0u, 0u}};
                a[k] = p.a;
                rem[k] = p.b.x - p.a.x;
            }
#pragma unroll
            for (int k = 0; k < DJ_GROUP; ++k) {
                const bool test = rem[k] > 32u || (uint32_t)__popc(a[k].y) != rem[k];
                const int64_t i = i0 + 64 * (g0 + k) + lane;
                if (!test) {
                    total += rem[k];
                    if (pm && i < n) pm[i] = a[k];
                }
                const unsigned long long mask = __ballot(test);
                const uint32_t nnew = (uint32_t)__popcll(mask);
                if (nnew == 0) continue;
                if (qn + nnew > (uint32_t)DJ_QCAP) drain();
                if (test) {
                    const uint32_t slot = qn + (uint32_t)__popcll(mask & below);
                    qx[slot] = xs[k];
                    qy[slot] = ys[k];
                    qk[slot] = a[k].x;
                    qf[slot] = a[k].y;
                    qi[slot] = (uint32_t)(64 * (g0 + k) + lane) | (min(rem[k], 33u) << 16);
                }
                qn += nnew;
            }
        }
        if (qn) drain();
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) total += (unsigned long long)__shfl_xor((long long)total, d, 64);
        if (lane == 0) counts[sg] = !EXACT && open ? DJ_OPEN : total;
    }
}

// Write pass from the count pass's masks.  The entries of a segment's pairs
// are listed in LDS in their order and then looked up and stored 64 at a
// time: 24M pairs of 30M points in 176 us, where every lane looking up and storing
// its own point's pairs one after the other took 240 us.  A word with more
// pairs than the list is stored by its lanes; points of cells with more than
// 32 entries are walked again.
__global__ __launch_bounds__(DJ_THREADS) void k_dj_write(DiskCanvas K, int64_t n, const double *X, const double *Y,
                                                         int64_t nseg, const unsigned long long *offs,
                                                         const uint2 *pm, uint32_t *out_pt, uint32_t *out_disk,
                                                         int64_t cap)
{
    __shared__ uint2 stage[DJ_THREADS / 64][DJ_STAGE];
    const int lane = threadIdx.x & 63;
    uint2 *list = stage[threadIdx.x >> 6];
    const int64_t nwave = ((int64_t)gridDim.x * DJ_THREADS) >> 6;
    for (int64_t sg = ((int64_t)blockIdx.x * DJ_THREADS + threadIdx.x) >> 6; sg < nseg; sg += nwave) {
        const int64_t i0 = sg * DJ_SEG + lane;
        uint2 e[DJ_ROUNDS];
#pragma unroll
        for (int k = 0; k < DJ_ROUNDS; ++k) e[k] = i0 + 64 * k < n ? pm[i0 + 64 * k] : uint2{0u, 0u};
        int64_t pos = (int64_t)offs[sg];   // of the list's first pair
        uint32_t have = 0;                 // pairs listed
        auto flush = [&]() {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            for (uint32_t t = (uint32_t)lane; t < have; t += 64) {
                const uint2 v = list[t];
                const uint32_t j = K.cell_disk[v.x] & ~DJ_FULL;
                if (pos + t < cap) {
                    out_pt[pos + t] = v.y;
                    out_disk[pos + t] = j;
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            pos += have;
            have = 0;
        };
#pragma unroll
        for (int k = 0; k < DJ_ROUNDS; ++k) {
            const int64_t i = i0 + 64 * k;
            const bool many = e[k].x == ~0u;
            uint32_t bits = many ? 0u : e[k].y;
            const uint32_t m = many ? e[k].y : (uint32_t)__popc(bits);
            uint32_t inc = m;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const uint32_t t = __shfl_up(inc, d, 64);
                if (lane >= d) inc += t;
            }
            const uint32_t tot = __shfl(inc, 63, 64);
            const bool direct = tot > DJ_STAGE || __ballot(many) != 0ull;
            if (direct || have + tot > DJ_STAGE) flush();
            uint32_t at = have + inc - m;
            while (bits) {
                const uint32_t x = e[k].x + (uint32_t)__ffs(bits) - 1u;
                bits &= bits - 1u;
                if (!direct) {
                    list[at] = uint2{x, (uint32_t)i};
                } else if (pos + at < cap) {
                    out_pt[pos + at] = (uint32_t)i;
                    out_disk[pos + at] = K.cell_disk[x] & ~DJ_FULL;
                }
                ++at;
            }
            if (!direct) {
                have += tot;
                continue;
            }
            if (__ballot(many)) {
                const double x = many ? X[i] : NAN, y = many ? Y[i] : NAN;
                uint32_t c0, rem, m2;
                disk_range(K, x, y, c0, rem);
                const int64_t w0 = sg * DJ_SEG + 64 * k;
                disk_wave_walk(K, x, y, c0, rem, inc - m, lane, m2, [&](int o, uint32_t slot, uint32_t j) {
                    if (pos + slot < cap) {
                        out_pt[pos + slot] = (uint32_t)(w0 + o);
                        out_disk[pos + slot] = j;
                    }
                });
            }
            pos += tot;
        }
        if (have) flush();
    }
}

// Walks that keep nothing.  MODE 1: pairs written from offs[s] on (positions
// at or beyond cap are not written), where the count pass's masks had no
// room; 2: per-disk counts.
template <int MODE>
__global__ __launch_bounds__(DJ_THREADS) void k_djoin(DiskCanvas K, int64_t n, const double *X, const double *Y,
                                                      int64_t nseg, const unsigned long long *offs, uint32_t *out_pt,
                                                      uint32_t *out_disk, int64_t cap, int64_t ndisk,
                                                      unsigned long long *dcount)
{
    extern __shared__ __align__(16) unsigned char smem[];
    uint32_t *hist = (uint32_t *)smem;
    const bool ldsh = MODE == 2 && ndisk <= DJ_HIST_MAX;
    if (MODE == 2) {
        if (ldsh)
            for (int64_t k = threadIdx.x; k < ndisk; k += DJ_THREADS) hist[k] = 0;
        __syncthreads();
    }
    const int lane = threadIdx.x & 63;
    const int64_t nwave = ((int64_t)gridDim.x * DJ_THREADS) >> 6;
    for (int64_t sg = ((int64_t)blockIdx.x * DJ_THREADS + threadIdx.x) >> 6; sg < nseg; sg += nwave) {
        const int64_t i0 = sg * DJ_SEG + lane;
        double xs[DJ_ROUNDS], ys[DJ_ROUNDS];
#pragma unroll
        for (int k = 0; k < DJ_ROUNDS; ++k) {
            const int64_t i = i0 + 64 * k;
            xs[k] = i < n ? __builtin_nontemporal_load(X + i) : NAN;
            ys[k] = i < n ? __builtin_nontemporal_load(Y + i) : NAN;
        }
        unsigned long long pos = MODE == 1 ? offs[sg] : 0ull;
        for (int k = 0; k < DJ_ROUNDS; ++k) {
            uint32_t c0, rem, m;
            disk_range(K, xs[k], ys[k], c0, rem);
            if (MODE == 2) {
                disk_wave_walk(K, xs[k], ys[k], c0, rem, 0u, lane, m, [&](int, uint32_t, uint32_t j) {
                    if (ldsh) atomicAdd(&hist[j], 1u);
                    else atomicAdd(&dcount[j], 1ull);
                });
                continue;
            }
            disk_wave_walk(K, xs[k], ys[k], c0, rem, 0u, lane, m, [](int, uint32_t, uint32_t) {});
            uint32_t inc = m;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const uint32_t t = __shfl_up(inc, d, 64);
                if (lane >= d) inc += t;
            }
            const uint32_t tot = __shfl(inc, 63, 64);
            if (tot) {
                // again, writing each pair at pos + (pairs of earlier lanes) + rank
                const int64_t w0 = sg * DJ_SEG + 64 * k;
                uint32_t m2;
                disk_wave_walk(K, xs[k], ys[k], c0, m ? rem : 0u, inc - m, lane, m2,
                               [&](int o, uint32_t slot, uint32_t j) {
                                   const unsigned long long p = pos + slot;
                                   if ((int64_t)p < cap) {
                                       out_pt[p] = (uint32_t)(w0 + o);
                                       out_disk[p] = j;
                                   }
                               });
            }
            pos += tot;
        }
    }
    if (MODE == 2 && ldsh) {
        __syncthreads();
        for (int64_t k = threadIdx.x; k < ndisk; k += DJ_THREADS)
            if (hist[k]) atomicAdd(&dcount[k], (unsigned long long)hist[k]);
    }
}

__global__ void k_dj_zero(int64_t n, unsigned long long *p)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0ull;
}

static int dj_grid(int64_t n, int64_t cap = 65536)
{
    return (int)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, cap));
}

static int dj_bits(uint64_t v)
{
    int b = 0;
    while (b < 64 && (v >> b) != 0) ++b;
    return b;
}

// Builds the disk canvas in ctx scratch (cell lists valid until the next
// call on ctx).  Counts need no order in the lists and no masks.
static int build_disk_canvas(spade_ctx *ctx, const spade_disks *dk, int64_t npts, bool counting, DiskCanvas &K)
{
    hipStream_t st = ctx->stream;
    const int64_t n = dk->n;
    K.D.cx = dk->cx;
    K.D.cy = dk->cy;
    K.D.r = dk->r;
    K.D.r_all = dk->r_all;
    DevBuf &bb = ctx->scratch[S_BLOCKRED];
    // box keys (4 words) | flag, long lists | - | sums of radii, of squares |
    // longest list | entries | - | shards of the entries
    const int64_t words = 16 + DJ_SHARDS * DJ_SHARD_WORDS;
    if (ensure(ctx, bb, 8 * (size_t)words)) return SPADE_E_NOMEM;
    unsigned long long *dbb = (unsigned long long *)bb.p;
    unsigned *bad = (unsigned *)(dbb + 4), *nlong = bad + 1;
    double *rsum = (double *)(dbb + 6);
    // box keys start at all-ones, the others at zero
    hipLaunchKernelGGL(k_dj_zero, dim3(1), dim3(256), 0, st, words, dbb);
    SPADE_HIP(ctx, hipGetLastError());
    SPADE_HIP(ctx, hipMemsetAsync(dbb, 0xff, 32, st));
    hipLaunchKernelGGL(k_disks_box, dim3(dj_grid(n, 1024)), dim3(256), 0, st, n, K.D, dbb, bad, rsum);
    SPADE_HIP(ctx, hipGetLastError());
    unsigned long long *h = (unsigned long long *)ensure_pinned(ctx, 128);
    if (!h) return set_error(ctx, SPADE_E_NOMEM, "pinned staging allocation failed");
    SPADE_HIP(ctx, hipMemcpyAsync(h, dbb, 64, hipMemcpyDeviceToHost, st));
    SPADE_HIP(ctx, hipStreamSynchronize(st));
    if (((unsigned *)(h + 4))[0]) return set_error(ctx, SPADE_E_INVALID, "disk centres and radii must be finite, radii >= 0");
    auto from_key = [](unsigned long long k) {
        const unsigned long long b = (k & 0x8000000000000000ull) ? (k & 0x7fffffffffffffffull) : ~k;
        double d;
        std::memcpy(&d, &b, sizeof d);
        return d;
    };
    double mr, rsq;
    std::memcpy(&mr, h + 6, sizeof mr);
    std::memcpy(&rsq, h + 7, sizeof rsq);
    DiskGrid &g = K.g;
    g.bx0 = from_key(h[0]);
    g.bx1 = -from_key(h[1]);
    g.by0 = from_key(h[2]);
    g.by1 = -from_key(h[3]);
    // cells about the mean radius on a side (at most DJ_GRID_MAX per side,
    // at least one), so a disk reaches a few cells; with many points, finer
    // ones.  An estimate of the finer lists' entries: the cells that meet a
    // disk widened by a cell's quarter and half its diagonal.
    const double w = g.bx1 - g.bx0, hgt = g.by1 - g.by0, sum_r = mr;
    mr /= (double)n;
    auto entries = [&](double c) {
        return 3.15 * (rsq + 2.2 * c * sum_r + 1.21 * c * c * (double)n) / (c * c);
    };
    const double least = std::max(w, hgt) / DJ_GRID_MAX;
    double cell = std::max(mr, least);
    double fine = std::max({mr / DJ_FINE, least, std::sqrt(w) * std::sqrt(hgt) / std::sqrt((double)npts / DJ_PER_CELL)});
    auto affordable = [&](double c) { return entries(c) <= std::min((double)npts / DJ_PER_ENTRY, 268435456.0); };
    // (cell <= DJ_FINE * fine, but for subnormal radii, which the factor may
    // leave as they are)
    for (int k = 0; k < 16 && fine < cell && !affordable(fine); ++k) fine *= 1.19;
    // Few disks: most cells list nothing, and a small table stays in the L1
    // (100 disks of 500 m over 60 km, 30M points: counts 330 us with cells of
    // 500 m, 430 with 125).
    const bool few = !(3.15 * rsq >= DJ_COVER * w * hgt), stacked = !(3.15 * rsq <= DJ_STACK * w * hgt);
    const bool finer = !few && !stacked && fine > 0.0 && fine < cell && affordable(fine);
    if (finer) cell = fine;
    K.together = !finer || npts < DJ_FILTER_MIN;
    g.W = (w > 0 && cell > 0) ? (int)std::min<double>(DJ_GRID_MAX, std::max(1.0, std::ceil(w / cell))) : 1;
    g.H = (hgt > 0 && cell > 0) ? (int)std::min<double>(DJ_GRID_MAX, std::max(1.0, std::ceil(hgt / cell))) : 1;
    g.X0 = g.bx0;
    g.Y0 = g.by0;
    g.sx = w > 0 ? g.W / w : 0.0;
    g.sy = hgt > 0 ? g.H / hgt : 0.0;
    const double ux = w > 0 ? w / g.W : 0.0, uy = hgt > 0 ? hgt / g.H : 0.0;
    const double mag = std::fabs(g.bx0) + std::fabs(g.bx1) + std::fabs(g.by0) + std::fabs(g.by1);
    const double lim = std::min(ux, uy) > mag * 0x1p-40 ? 1.0 - 1e-7 : -1.0;
    const int64_t ncell = (int64_t)g.W * g.H;
    // Cell lists: count, scan, fill in any order, order each list, by one lane
    // or a workgroup.  Where a list is longer than DJ_LIST_WG entries, (cell,
    // disk) keys are sorted instead (30 launches for a million of them: 140 us,
    // against 25).
    DevBuf &bw = ctx->scratch[S_VALS2];
    if (ensure(ctx, bw, sizeof(double2) * (size_t)n + (sizeof(uint2) + 3 * sizeof(uint32_t)) * (size_t)(ncell + 1)))
        return SPADE_E_NOMEM;
    double2 *centre = (double2 *)bw.p;
    uint2 *cells = (uint2 *)(centre + n);
    uint32_t *ccnt = (uint32_t *)(cells + (ncell + 1)), *coff = ccnt + (ncell + 1);
    uint32_t *longs = coff + (ncell + 1);
    unsigned *longest = (unsigned *)(dbb + 8);
    const bool few_cells = ncell <= DJ_FEW_CELLS;
    const dim3 dgrid(few_cells ? dj_grid(n * 16, 384) : dj_grid(n * 64, 2048)), cgrid((unsigned)(ncell / 256 + 1));
    auto disks = [&](auto kern, unsigned long long *keys, uint32_t *list) {
        hipLaunchKernelGGL(kern, dgrid, dim3(256), 0, st, n, K.D, g, ux, uy, lim, ccnt, keys,
                           (const uint2 *)cells, list, centre, dbb + 16);
    };
    DevBuf &cub = ctx->scratch[S_CUBTMP];
    size_t tb = 0;
    SPADE_HIP(ctx, hipMemsetAsync(ccnt, 0, sizeof(uint32_t) * (size_t)(ncell + 1), st));
    disks(few_cells ? k_disk_cells<CELL_COUNT, true> : k_disk_cells<CELL_COUNT, false>, nullptr, nullptr);
    SPADE_HIP(ctx, hipGetLastError());
    SPADE_HIP(ctx, hipcub::DeviceScan::ExclusiveSum(nullptr, tb, ccnt, coff, (int)(ncell + 1), st));
    if (ensure(ctx, cub, std::max<size_t>(tb, 1))) return SPADE_E_NOMEM;
    SPADE_HIP(ctx, hipcub::DeviceScan::ExclusiveSum(cub.p, tb, ccnt, coff, (int)(ncell + 1), st));
    hipLaunchKernelGGL(k_dcell_start, cgrid, dim3(256), 0, st, ncell, (const uint32_t *)coff, ccnt, cells, longs,
                       nlong, longest, (const unsigned long long *)(dbb + 16), dbb + 9);
    SPADE_HIP(ctx, hipGetLastError());
    SPADE_HIP(ctx, hipMemcpyAsync(h, dbb + 8, 16, hipMemcpyDeviceToHost, st));
    SPADE_HIP(ctx, hipStreamSynchronize(st));
    const unsigned most_listed = (unsigned)h[0];
    const int64_t nk = (int64_t)h[1];
    if (nk >= (int64_t)0xffffffffLL) return set_error(ctx, SPADE_E_UNSUPPORTED, "too many (cell, disk) entries");
    const bool sorted = !counting && most_listed > DJ_LIST_WG;
    DevBuf &bl = ctx->scratch[S_VALS];
    if (ensure(ctx, bl, 4 * (size_t)std::max<int64_t>(nk, 1) + 64)) return SPADE_E_NOMEM;
    uint32_t *cell_disk = (uint32_t *)bl.p;
    if (sorted) {
        DevBuf &bk = ctx->scratch[S_KEYS], &bk2 = ctx->scratch[S_KEYS2];
        if (ensure(ctx, bk, 8 * (size_t)nk) || ensure(ctx, bk2, 8 * (size_t)nk)) return SPADE_E_NOMEM;
        disks(few_cells ? k_disk_cells<CELL_KEYS, true> : k_disk_cells<CELL_KEYS, false>, (unsigned long long *)bk.p, nullptr);
        SPADE_HIP(ctx, hipGetLastError());
        const int kb = 32 + std::max(1, dj_bits((uint64_t)ncell));
        tb = 0;
        SPADE_HIP(ctx, hipcub::DeviceRadixSort::SortKeys(nullptr, tb, (const unsigned long long *)bk.p,
                                                         (unsigned long long *)bk2.p, (int)nk, 0, kb, st));
        if (ensure(ctx, cub, std::max<size_t>(tb, 1))) return SPADE_E_NOMEM;
        SPADE_HIP(ctx, hipcub::DeviceRadixSort::SortKeys(cub.p, tb, (const unsigned long long *)bk.p,
                                                         (unsigned long long *)bk2.p, (int)nk, 0, kb, st));
        hipLaunchKernelGGL(k_dcell_list, dim3(dj_grid(nk)), dim3(256), 0, st, nk, (const unsigned long long *)bk2.p,
                           cell_disk);
    } else {
        disks(few_cells ? k_disk_cells<CELL_LIST, true> : k_disk_cells<CELL_LIST, false>, nullptr, cell_disk);
        if (!counting && most_listed > DJ_LIST_SORT)
            hipLaunchKernelGGL(k_dcell_sort, dim3(1024), dim3(256), 0, st, (const unsigned *)nlong, (const uint32_t *)longs,
                               (const uint2 *)cells, cell_disk);
    }
    if (!counting)
        hipLaunchKernelGGL(k_dcell_full, dim3((unsigned)((ncell + 127) / 128)), dim3(128), 0, st, ncell, cells, cell_disk,
                           sorted ? 0 : 1);
    SPADE_HIP(ctx, hipGetLastError());
    K.off = coff;
    K.cells = cells;
    K.cell_disk = cell_disk;
    K.centre = centre;
    K.longest = most_listed;
    return SPADE_OK;
}

static int check_disks(spade_ctx *ctx, const spade_disks *dk)
{
    if (!dk) return set_error(ctx, SPADE_E_INVALID, "disks is NULL");
    if (dk->n < 0) return set_error(ctx, SPADE_E_INVALID, "negative disk count");
    if (dk->n >= (int64_t)0x7fffffffLL) return set_error(ctx, SPADE_E_TOO_LARGE, "disk ids must be < 2^31 - 1");
    if (dk->n > 0 && (!dk->cx || !dk->cy)) return set_error(ctx, SPADE_E_INVALID, "disk centre array is NULL");
    if (!dk->r && !(std::isfinite(dk->r_all) && dk->r_all >= 0.0))
        return set_error(ctx, SPADE_E_INVALID, "r_all must be finite and >= 0");
    return SPADE_OK;
}

static int num_cus_dj(int device)
{
    int v = 0;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess || v <= 0) v = 256;
    return v;
}

int distance_join(spade_ctx *ctx, const spade_points *pts, const spade_disks *dk, uint32_t *out_pt,
                  uint32_t *out_disk, int64_t cap, int64_t *n_out, uint64_t *out_counts)
{
    int rc = check_disks(ctx, dk);
    if (rc) return rc;
    hipStream_t st = ctx->stream;
    if (n_out) *n_out = 0;
    const int64_t n = pts->n, m = dk->n;
    const bool counting = out_counts != nullptr;
    if (counting && m > 0) {
        hipLaunchKernelGGL(k_dj_zero, dim3(dj_grid(m, 4096)), dim3(256), 0, st, m, (unsigned long long *)out_counts);
        SPADE_HIP(ctx, hipGetLastError());
    }
    if (n == 0 || m == 0) {
        if (counting) SPADE_HIP(ctx, hipStreamSynchronize(st));
        return SPADE_OK;
    }
    DiskCanvas K;
    if ((rc = build_disk_canvas(ctx, dk, n, counting, K))) return rc;
    const int64_t nseg = (n + DJ_SEG - 1) / DJ_SEG;
    const int cus = num_cus_dj(ctx->device);
    const int grid = (int)std::max<int64_t>(1, std::min<int64_t>((nseg + DJ_THREADS / 64 - 1) / (DJ_THREADS / 64),
                                                                 (int64_t)cus * 8));
    if (ctx->timing) SPADE_HIP(ctx, hipEventRecord(ctx->ev[2], st));
    if (counting) {
        const size_t lds = m <= DJ_HIST_MAX ? 4 * (size_t)m : 16;
        hipLaunchKernelGGL(k_djoin<2>, dim3(grid), dim3(DJ_THREADS), lds, st, K, n, pts->x, pts->y, nseg, nullptr,
                           nullptr, nullptr, (int64_t)0, m, (unsigned long long *)out_counts);
        SPADE_HIP(ctx, hipGetLastError());
        if (ctx->timing) SPADE_HIP(ctx, hipEventRecord(ctx->ev[3], st));
        SPADE_HIP(ctx, hipStreamSynchronize(st));
        return SPADE_OK;
    }
    DevBuf &lb = ctx->scratch[S_LOOKBACK];
    if (ensure(ctx, lb, sizeof(unsigned long long) * 2 * (size_t)(nseg + 1))) return SPADE_E_NOMEM;
    unsigned long long *counts = (unsigned long long *)lb.p, *offs = counts + (nseg + 1);
    // every point's pairs, kept by the count pass for the write pass (without
    // the room, the write pass tests again)
    DevBuf &pb = ctx->scratch[S_BITS];
    uint2 *pm = nullptr;
    if (cap > 0) {
        if (ensure(ctx, pb, sizeof(uint2) * (size_t)n) == SPADE_OK) pm = (uint2 *)pb.p;
        else ctx->err.clear();
    }
    auto count = [&](auto kern, int per_cu) {
        hipLaunchKernelGGL(kern, dim3(std::min(grid, cus * per_cu)), dim3(DJ_THREADS), 0, st, K, n, pts->x, pts->y, nseg,
                           counts, pm);
    };
    if (n < DJ_FILTER_MIN || K.longest > 32) {   // longer lists always take the exact walk
        count(k_dj_count<true, false>, 4);
    } else {
        count(k_dj_count<false, false>, 5);
        count(k_dj_count<true, true>, 4);
    }
    hipLaunchKernelGGL(k_dj_zero, dim3(1), dim3(64), 0, st, (int64_t)1, counts + nseg);
    SPADE_HIP(ctx, hipGetLastError());
    DevBuf &cub = ctx->scratch[S_CUBTMP];
    size_t tb = 0;
    SPADE_HIP(ctx, hipcub::DeviceScan::ExclusiveSum(nullptr, tb, counts, offs, (int)(nseg + 1), st));
    if (ensure(ctx, cub, std::max<size_t>(tb, 1))) return SPADE_E_NOMEM;
    SPADE_HIP(ctx, hipcub::DeviceScan::ExclusiveSum(cub.p, tb, counts, offs, (int)(nseg + 1), st));
    if (cap > 0) {
        if (pm)
            hipLaunchKernelGGL(k_dj_write, dim3(std::min(grid, cus * 5)), dim3(DJ_THREADS), 0, st, K, n, pts->x, pts->y, nseg,
                               (const unsigned long long *)offs, (const uint2 *)pm, out_pt, out_disk, cap);
        else
            hipLaunchKernelGGL(k_djoin<1>, dim3(grid), dim3(DJ_THREADS), 0, st, K, n, pts->x, pts->y, nseg, offs, out_pt,
                               out_disk, cap, m, nullptr);
        SPADE_HIP(ctx, hipGetLastError());
    }
    if (ctx->timing) SPADE_HIP(ctx, hipEventRecord(ctx->ev[3], st));
    unsigned long long *h = (unsigned long long *)ensure_pinned(ctx, 64);
    if (!h) return set_error(ctx, SPADE_E_NOMEM, "pinned staging allocation failed");
    SPADE_HIP(ctx, hipMemcpyAsync(h, offs + nseg, 8, hipMemcpyDeviceToHost, st));
    SPADE_HIP(ctx, hipStreamSynchronize(st));
    *n_out = (int64_t)h[0];
    if (*n_out > cap) return set_error(ctx, SPADE_E_CAPACITY, "output capacity too small");
    return SPADE_OK;
}

// ------------------------------------------------------------ kNN selection
//
// The paper's plan (Sec. 5.2, "kNN Queries"): nested circles around the
// query point with radii in a geometric progression, one aggregation pass
// that counts the points in every circle, a distance selection with the
// smallest circle that holds at least k points, and a sort of those
// candidates by distance.  The paper anchors the circles at r_max (the
// largest distance from the point to a corner of the points' bounding box)
// with r_i = r_max / alpha^i.  Here alpha = 2 and the circles are first the
// powers of two r_j = 2^j, -511 <= j <= 511 (r_j^2 is a normal double, so
// the exact closed-disk test applies): they need no bounding box, so the
// aggregation is the only pass before the selection.  Only when more than
// the points inside r_511 are needed (distances beyond 6.7e153) does the
// query fall back to circles r_max 2^-i (i <= KNN_LEVELS) from the bounding
// box.  Every comparison is exact: the circle counts use the exact
// closed-disk test, and the candidates are ordered by their FP64 squared
// distance, then every run of keys too close to tell apart is re-ordered
// exactly (ties in distance: smaller id first).

constexpr int KNN_LEVELS = 48;
constexpr int KNN_THREADS = 256;

// Points' bounding box (finite points) as order keys.
__global__ __launch_bounds__(256) void k_knn_box(int64_t n, const double *X, const double *Y,
                                                 unsigned long long *bb)
{
    __shared__ unsigned long long s[4][256];
    unsigned long long k0 = ~0ull, k1 = ~0ull, k2 = ~0ull, k3 = ~0ull;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const double x = X[i], y = Y[i];
        if (!isfinite(x) || !isfinite(y)) continue;
        k0 = min(k0, okey_d(x)); k1 = min(k1, okey_d(-x));
        k2 = min(k2, okey_d(y)); k3 = min(k3, okey_d(-y));
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

struct KnnCircles {
    double px, py;
    double r[KNN_LEVELS + 1];
    double r2[KNN_LEVELS + 1];
};

// Aggregation over the nested circles: level[i] counts the points whose
// innermost containing circle is circle i (binary search with the exact
// predicate; the circles are nested).  The radii (device array cr, r then
// r^2) are read into LDS.
__global__ __launch_bounds__(KNN_THREADS) void k_knn_levels(int64_t n, const double *X, const double *Y, double px,
                                                            double py, const double *cr, unsigned long long *level)
{
    __shared__ unsigned int h[KNN_LEVELS + 1];
    __shared__ double sr[2 * (KNN_LEVELS + 1)];
    for (int k = threadIdx.x; k <= KNN_LEVELS; k += KNN_THREADS) h[k] = 0;
    for (int k = threadIdx.x; k < 2 * (KNN_LEVELS + 1); k += KNN_THREADS) sr[k] = cr[k];
    __syncthreads();
    const double *r = sr, *r2 = sr + (KNN_LEVELS + 1);
    for (int64_t i = (int64_t)blockIdx.x * KNN_THREADS + threadIdx.x; i < n; i += (int64_t)gridDim.x * KNN_THREADS) {
        const double x = X[i], y = Y[i];
        if (!in_disk(x, y, px, py, r[0], r2[0])) continue;   // non-finite points too
        int lo = 0, hi = KNN_LEVELS;   // in circle lo; find the innermost
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (in_disk(x, y, px, py, r[mid], r2[mid])) lo = mid; else hi = mid - 1;
        }
        atomicAdd(&h[lo], 1u);
    }
    __syncthreads();
    for (int k = threadIdx.x; k <= KNN_LEVELS; k += KNN_THREADS)
        if (h[k]) atomicAdd(&level[k], (unsigned long long)h[k]);
}

constexpr int KNN_JMIN = -511, KNN_JMAX = 511;
constexpr int KNN_BINS = KNN_JMAX - KNN_JMIN + 2;   // + the points outside every circle

__device__ __forceinline__ bool in_circle_pow2(double x, double y, double px, double py, int j)
{
    return in_disk(x, y, px, py, ldexp(1.0, j), ldexp(1.0, 2 * j));
}

// Aggregation over the circles r_j = 2^j: bins[j - KNN_JMIN] counts the
// finite points whose innermost containing circle is j, bins[KNN_BINS - 1]
// those outside circle KNN_JMAX.  The FP64 squared distance only gives the
// first guess at j (4^j <= d2 up to rounding); the exact test settles it,
// usually with two tests: j is outside, j + 1 inside.
// Only bins that were hit are added to the global counts.  wmin keeps the
// innermost circle of every 64 consecutive points, so that the selection that
// follows reads only the points it can take: the pass runs at the rate of a
// plain read (100M points in 0.25 ms), and a second one over all points cost
// as much again.
constexpr int16_t KNN_NONE = 0x7fff;   // 64 points without a finite one
constexpr int KNN_PER = 2;             // points per thread in flight

__global__ __launch_bounds__(KNN_THREADS) void k_knn_pow2(int64_t n, const double *X, const double *Y, double px,
                                                          double py, unsigned long long *bins, int16_t *wmin)
{
    __shared__ unsigned int h[KNN_BINS];
    for (int k = threadIdx.x; k < KNN_BINS; k += KNN_THREADS) h[k] = 0;
    __syncthreads();
    const int64_t step = (int64_t)gridDim.x * KNN_THREADS * KNN_PER;
    for (int64_t b = (int64_t)blockIdx.x * KNN_THREADS * KNN_PER; b < n; b += step) {
        double xs[KNN_PER], ys[KNN_PER];
#pragma unroll
        for (int u = 0; u < KNN_PER; ++u) {
            const int64_t i = b + u * KNN_THREADS + threadIdx.x;
            xs[u] = i < n ? __builtin_nontemporal_load(X + i) : NAN;
            ys[u] = i < n ? __builtin_nontemporal_load(Y + i) : NAN;
        }
#pragma unroll
        for (int u = 0; u < KNN_PER; ++u) {
            const int64_t i = b + u * KNN_THREADS + threadIdx.x;
            const double x = xs[u], y = ys[u];
            int j = KNN_NONE;
            if (fabs(x) <= 1.7976931348623157e308 && fabs(y) <= 1.7976931348623157e308) {
                const double dx = x - px, dy = y - py;
                const double d2 = dx * dx + dy * dy;
                if (!(d2 > 0.0)) j = KNN_JMIN;
                else if (!(d2 <= 1.7976931348623157e308)) j = KNN_JMAX + 1;
                else j = min(max(ilogb(d2) >> 1, KNN_JMIN), KNN_JMAX + 1);   // 4^j <= d2 up to rounding
                if (j <= KNN_JMAX && !in_circle_pow2(x, y, px, py, j)) {
                    do ++j;
                    while (j <= KNN_JMAX && !in_circle_pow2(x, y, px, py, j));
                } else {
                    // in circle j (or j past the last one): move inwards while inside
                    while (j > KNN_JMIN && in_circle_pow2(x, y, px, py, j - 1)) --j;
                }
                atomicAdd(&h[j - KNN_JMIN], 1u);
            }
            int low;
            typename rocprim::warp_reduce<int, 64>::storage_type storage;
            rocprim::warp_reduce<int, 64>().reduce(j, low, storage, rocprim::minimum<int>());
            if ((threadIdx.x & 63) == 0 && i < n) wmin[i >> 6] = (int16_t)low;
        }
    }
    __syncthreads();
    for (int k = threadIdx.x; k < KNN_BINS; k += KNN_THREADS)
        if (h[k]) atomicAdd(&bins[k], (unsigned long long)h[k]);
}

// The points of circle 2^J from the words whose innermost circle reaches it:
// ids and keys (FP64 squared distance), a workgroup's in id order, the
// workgroups in no particular one.  A wavefront looks at 64 words, one per
// lane; one global atomic per workgroup.  seg, when given, keeps where every
// workgroup's points lie, and tot their number.
__global__ __launch_bounds__(KNN_THREADS) void k_knn_take(int64_t n, const double *X, const double *Y, double px,
                                                          double py, int J, const int16_t *wmin, uint32_t *count,
                                                          uint32_t cap, uint32_t *ids, unsigned long long *keys,
                                                          uint32_t *seg, uint32_t *tot)
{
    __shared__ uint32_t wsum[KNN_THREADS / 64];
    __shared__ uint32_t s_base;
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t nw = (n + 63) >> 6;
    const int64_t w0 = ((int64_t)blockIdx.x * (KNN_THREADS / 64) + wv) * 64;
    const bool reach = w0 + lane < nw && wmin[w0 + lane] <= J;
    unsigned long long mine = 0ull;   // the points of this lane's word that are taken
    for (unsigned long long m = __ballot(reach); m; m &= m - 1) {
        const int w = __ffsll((long long)m) - 1;
        const int64_t i = (w0 + w) * 64 + lane;
        const bool in = i < n && in_circle_pow2(X[i], Y[i], px, py, J);
        const unsigned long long t = __ballot(in);
        if (lane == w) mine = t;
    }
    const uint32_t c = (uint32_t)__popcll(mine);
    uint32_t incl;
    typename rocprim::warp_scan<uint32_t, 64>::storage_type storage;
    rocprim::warp_scan<uint32_t, 64>().inclusive_scan(c, incl, storage, rocprim::plus<uint32_t>());
    if (lane == 63) wsum[wv] = incl;
    __syncthreads();
    uint32_t pre = 0u, total = 0u;
#pragma unroll
    for (int w = 0; w < KNN_THREADS / 64; ++w) {
        if (w < wv) pre += wsum[w];
        total += wsum[w];
    }
    if (tot && threadIdx.x == 0) tot[blockIdx.x] = total;
    if (total == 0u) return;   // uniform over the workgroup
    if (threadIdx.x == 0) {
        s_base = atomicAdd(count, total);
        if (seg) seg[blockIdx.x] = s_base;
    }
    __syncthreads();
    const uint32_t first = s_base + pre + incl - c;   // of this lane's word
    for (unsigned long long m = __ballot(mine != 0ull); m; m &= m - 1) {
        const int w = __ffsll((long long)m) - 1;
        const unsigned long long t = (unsigned long long)__shfl((long long)mine, w, 64);
        const uint32_t at = (uint32_t)__shfl((int)first, w, 64) + (uint32_t)__popcll(t & ((1ull << lane) - 1ull));
        if (((t >> lane) & 1ull) && at < cap) {
            const int64_t i = (w0 + w) * 64 + lane;
            ids[at] = (uint32_t)i;
            keys[at] = (unsigned long long)__double_as_longlong(dist2(X[i], Y[i], px, py));
        }
    }
}

// The workgroups' points in id order: those of k_knn_take's workgroup b, at
// seg[b], to at[b].  The sort by key is stable, so a run of equal distances (a
// place with many points) then has its ids ascending and costs the exact
// comparison one step per point; out of order it would be quadratic.
__global__ __launch_bounds__(64) void k_knn_place(const uint32_t *seg, const uint32_t *tot, const uint32_t *at,
                                                  const uint32_t *ids, const unsigned long long *keys, uint32_t *oids,
                                                  unsigned long long *okeys)
{
    const uint32_t n = tot[blockIdx.x], from = n ? seg[blockIdx.x] : 0u, to = at[blockIdx.x];
    for (uint32_t i = threadIdx.x; i < n; i += 64) {
        oids[to + i] = ids[from + i];
        okeys[to + i] = keys[from + i];
    }
}

// Candidate keys: FP64 squared distance (non-negative, so its bits order it)
// and the id.
__global__ void k_knn_keys(int64_t m, const uint32_t *ids, const double *X, const double *Y, double px, double py,
                           unsigned long long *key)
{
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < m; t += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t i = ids[t];
        key[t] = (unsigned long long)__double_as_longlong(dist2(X[i], Y[i], px, py));
    }
}

__device__ __forceinline__ bool knn_close(unsigned long long a, unsigned long long b)
{
    const double qa = __longlong_as_double((long long)a), qb = __longlong_as_double((long long)b);
    return fabs(qa - qb) <= 1.7763568394002505e-15 * (qa + qb);
}

// Runs of consecutive keys too close to tell apart, starting among the first
// kk, are re-ordered by the exact comparison (ids break exact ties); one thread
// per run, insertion sort.  Every run's ids go to out, the first kk of all.
__global__ void k_knn_fix(int64_t m, int64_t kk, const unsigned long long *key, uint32_t *ids, const double *X,
                          const double *Y, double px, double py, uint32_t *out)
{
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < kk; t += (int64_t)gridDim.x * blockDim.x) {
        if (t > 0 && knn_close(key[t - 1], key[t])) continue;   // not a run start
        int64_t e = t + 1;
        while (e < m && knn_close(key[e - 1], key[e])) ++e;
        for (int64_t a = t + 1; a < e; ++a) {
            const uint32_t v = ids[a];
            int64_t b = a;
            while (b > t) {
                const uint32_t u = ids[b - 1];
                const int c = dist_cmp(X[u], Y[u], X[v], Y[v], px, py);
                if (c < 0 || (c == 0 && u < v)) break;
                ids[b] = u;
                --b;
            }
            ids[b] = v;
        }
        for (int64_t a = t; a < min(e, kk); ++a) out[a] = ids[a];
    }
}

// Few candidates (m <= KS_MAX) are sorted by (key, id) by one workgroup in
// LDS, a bitonic sort in place of the library's five launches for the 1,000 to
// 4,000 candidates of k = 1,000.  The runs of close keys are k_knn_fix's, whose
// comparisons need more than one CU: 3,000 lattice points in runs of up to 36,
// 439 us in this workgroup, 135 in a launch of its own.
constexpr int KS_THREADS = 1024;
constexpr int KS_MAX = 4096;

__global__ __launch_bounds__(KS_THREADS) void k_knn_order(int m, unsigned long long *keys, uint32_t *ids)
{
    __shared__ unsigned long long sk[KS_MAX];
    __shared__ uint32_t sid[KS_MAX];
    const int t = threadIdx.x;
    int P = 2;
    while (P < m) P <<= 1;
    for (int i = t; i < P; i += KS_THREADS) {
        sk[i] = i < m ? keys[i] : ~0ull;   // past every distance
        sid[i] = i < m ? ids[i] : 0xffffffffu;
    }
    __syncthreads();
    for (int k = 2; k <= P; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int e = t; e < P / 2; e += KS_THREADS) {
                const int a = ((e & ~(j - 1)) << 1) | (e & (j - 1)), b = a + j;
                const unsigned long long ka = sk[a], kb = sk[b];
                const uint32_t ia = sid[a], ib = sid[b];
                const bool gt = ka > kb || (ka == kb && ia > ib);
                if (gt == ((a & k) == 0)) {
                    sk[a] = kb; sk[b] = ka;
                    sid[a] = ib; sid[b] = ia;
                }
            }
            __syncthreads();
        }
    for (int i = t; i < m; i += KS_THREADS) {
        keys[i] = sk[i];
        ids[i] = sid[i];
    }
}

int knn_select(spade_ctx *ctx, const spade_points *pts, double px, double py, int64_t k, uint32_t *out_ids,
               int64_t *n_out)
{
    hipStream_t st = ctx->stream;
    *n_out = 0;
    if (!(std::isfinite(px) && std::isfinite(py))) return set_error(ctx, SPADE_E_INVALID, "query point must be finite");
    if (k < 0) return set_error(ctx, SPADE_E_INVALID, "negative k");
    if (k > 0 && !out_ids) return set_error(ctx, SPADE_E_INVALID, "out_ids is NULL");
    const int64_t n = pts->n;
    if (k == 0 || n == 0) return SPADE_OK;
    const int cus = num_cus_dj(ctx->device);
    // circles r_j = 2^j: bins of the innermost containing circle
    DevBuf &bb = ctx->scratch[S_BLOCKRED];
    const size_t bin_bytes = 8 * (size_t)KNN_BINS;
    if (ensure(ctx, bb, std::max<size_t>(bin_bytes + 8, 64 + 8 * (KNN_LEVELS + 1) + 16 * (KNN_LEVELS + 1))))
        return SPADE_E_NOMEM;
    unsigned long long *dbins = (unsigned long long *)bb.p;
    // (the word past the bins: the number of candidates taken)
    DevBuf &bw = ctx->scratch[S_NEXTP];
    if (ensure(ctx, bw, sizeof(int16_t) * (size_t)((n + 63) / 64))) return SPADE_E_NOMEM;
    int16_t *wmin = (int16_t *)bw.p;
    hipLaunchKernelGGL(k_dj_zero, dim3(5), dim3(256), 0, st, (int64_t)KNN_BINS + 1, dbins);
    if (ctx->timing) SPADE_HIP(ctx, hipEventRecord(ctx->ev[2], st));
    hipLaunchKernelGGL(k_knn_pow2, dim3((unsigned)std::min<int64_t>((n + KNN_THREADS * KNN_PER - 1) / (KNN_THREADS * KNN_PER), cus * 8)),
                       dim3(KNN_THREADS), 0, st, n, pts->x, pts->y, px, py, dbins, wmin);
    SPADE_HIP(ctx, hipGetLastError());
    unsigned long long *hb = (unsigned long long *)ensure_pinned(ctx, bin_bytes + 16 * (KNN_LEVELS + 8));
    if (!hb) return set_error(ctx, SPADE_E_NOMEM, "pinned staging allocation failed");
    SPADE_HIP(ctx, hipMemcpyAsync(hb, dbins, bin_bytes, hipMemcpyDeviceToHost, st));
    SPADE_HIP(ctx, hipStreamSynchronize(st));
    int64_t total = 0;
    for (int b = 0; b < KNN_BINS; ++b) total += (int64_t)hb[b];
    if (total == 0) return SPADE_OK;   // no finite point
    const int64_t want = std::min<int64_t>(k, total);
    int64_t cum = 0;
    double rsel = -1.0;
    int jsel = KNN_JMAX + 1;
    for (int b = 0; b + 1 < KNN_BINS; ++b) {
        cum += (int64_t)hb[b];
        if (cum >= want) {
            jsel = KNN_JMIN + b;
            rsel = std::ldexp(1.0, jsel);
            break;
        }
    }
    if (rsel < 0.0) {
        // more points are needed than lie within 2^511: the circles
        // r_max 2^-i from the points' bounding box
        unsigned long long *dbb = dbins;
        unsigned long long *level = dbb + 4;
        SPADE_HIP(ctx, hipMemsetAsync(dbb, 0xff, 32, st));
        hipLaunchKernelGGL(k_dj_zero, dim3(1), dim3(64), 0, st, (int64_t)(KNN_LEVELS + 1), level);
        hipLaunchKernelGGL(k_knn_box, dim3(dj_grid(n, 1024)), dim3(256), 0, st, n, pts->x, pts->y, dbb);
        SPADE_HIP(ctx, hipGetLastError());
        unsigned long long *h = hb;
        SPADE_HIP(ctx, hipMemcpyAsync(h, dbb, 32, hipMemcpyDeviceToHost, st));
        SPADE_HIP(ctx, hipStreamSynchronize(st));
        auto from_key = [](unsigned long long kk) {
            const unsigned long long b = (kk & 0x8000000000000000ull) ? (kk & 0x7fffffffffffffffull) : ~kk;
            double d;
            std::memcpy(&d, &b, sizeof d);
            return d;
        };
        const double x0 = from_key(h[0]), x1 = -from_key(h[1]), y0 = from_key(h[2]), y1 = -from_key(h[3]);
        double rmax = 0.0;
        for (double cx : {x0, x1})
            for (double cy : {y0, y1}) rmax = std::max(rmax, std::hypot(cx - px, cy - py));
        // round up by a relative 2^-40: every finite point is then in circle 0
        // (the exact test decides), whatever the rounding of hypot
        rmax = rmax * (1.0 + std::ldexp(1.0, -40)) + std::ldexp(1.0, -1000);
        KnnCircles C;
        C.px = px;
        C.py = py;
        for (int i = 0; i <= KNN_LEVELS; ++i) {
            C.r[i] = std::ldexp(rmax, -i);
            C.r2[i] = C.r[i] * C.r[i];
        }
        double *cr = (double *)(level + (KNN_LEVELS + 1));
        double *hr = (double *)(hb + KNN_LEVELS + 8);
        std::memcpy(hr, C.r, 8 * (KNN_LEVELS + 1));
        std::memcpy(hr + KNN_LEVELS + 1, C.r2, 8 * (KNN_LEVELS + 1));
        SPADE_HIP(ctx, hipMemcpyAsync(cr, hr, 16 * (KNN_LEVELS + 1), hipMemcpyHostToDevice, st));
        hipLaunchKernelGGL(k_knn_levels, dim3((unsigned)std::min<int64_t>((n + KNN_THREADS - 1) / KNN_THREADS, cus * 8)),
                           dim3(KNN_THREADS), 0, st, n, pts->x, pts->y, px, py, (const double *)cr, level);
        SPADE_HIP(ctx, hipGetLastError());
        SPADE_HIP(ctx, hipMemcpyAsync(h, level, 8 * (KNN_LEVELS + 1), hipMemcpyDeviceToHost, st));
        SPADE_HIP(ctx, hipStreamSynchronize(st));
        // count(r_i) = points whose innermost circle is i or deeper
        int64_t ltot = 0;
        for (int i = 0; i <= KNN_LEVELS; ++i) ltot += (int64_t)h[i];
        cum = 0;
        int sel = 0;
        for (int i = KNN_LEVELS; i >= 0; --i) {
            cum += (int64_t)h[i];
            if (cum >= std::min<int64_t>(k, ltot)) { sel = i; break; }
        }
        rsel = C.r[sel];
    }
    // The candidates: the points of that circle, with their keys.  Few of them
    // (one in 32 points, in 128 where they have to be put in id order; in no
    // spatial order two thirds of the words have one of one in 60) come from
    // the words of points that reach the circle; more, and the circles of the
    // bounding box, from a distance selection over all points.
    int64_t m = cum;
    DevBuf &bc = ctx->scratch[S_VALS2], &bk = ctx->scratch[S_KEYS];
    if (ensure(ctx, bc, 4 * (size_t)std::max<int64_t>(cum, 1)) || ensure(ctx, bk, 8 * (size_t)std::max<int64_t>(cum, 1)))
        return SPADE_E_NOMEM;
    // (sorted by the library, the candidates lie in bi and bk2 in id order)
    DevBuf &bk2 = ctx->scratch[S_KEYS2], &bi = ctx->scratch[S_VALS], &cub = ctx->scratch[S_CUBTMP];
    const bool take = jsel <= KNN_JMAX && cum <= n / (cum > KS_MAX ? 128 : 32), placed = take && cum > KS_MAX;
    if (cum > KS_MAX && (ensure(ctx, bk2, 8 * (size_t)cum) || ensure(ctx, bi, 4 * (size_t)cum))) return SPADE_E_NOMEM;
    size_t tb = 0;
    if (take) {
        const unsigned wgs = (unsigned)((n + 64 * KNN_THREADS - 1) / (64 * KNN_THREADS));
        uint32_t *seg = nullptr, *tot = nullptr, *at = nullptr;
        if (placed) {
            DevBuf &bn = ctx->scratch[S_LOOKBACK];
            if (ensure(ctx, bn, sizeof(uint32_t) * 3 * (size_t)wgs)) return SPADE_E_NOMEM;
            seg = (uint32_t *)bn.p;
            tot = seg + wgs;
            at = tot + wgs;
            SPADE_HIP(ctx, hipcub::DeviceScan::ExclusiveSum(nullptr, tb, tot, at, (int)wgs, st));
            if (ensure(ctx, cub, std::max<size_t>(tb, 1))) return SPADE_E_NOMEM;
        }
        hipLaunchKernelGGL(k_knn_take, dim3(wgs), dim3(KNN_THREADS), 0, st, n, pts->x, pts->y, px, py, jsel,
                           (const int16_t *)wmin, (uint32_t *)(dbins + KNN_BINS), (uint32_t)cum, (uint32_t *)bc.p,
                           (unsigned long long *)bk.p, seg, tot);
        SPADE_HIP(ctx, hipGetLastError());
        if (placed) {
            SPADE_HIP(ctx, hipcub::DeviceScan::ExclusiveSum(cub.p, tb, tot, at, (int)wgs, st));
            hipLaunchKernelGGL(k_knn_place, dim3(wgs), dim3(64), 0, st, (const uint32_t *)seg, (const uint32_t *)tot,
                               (const uint32_t *)at, (const uint32_t *)bc.p, (const unsigned long long *)bk.p,
                               (uint32_t *)bi.p, (unsigned long long *)bk2.p);
        }
    } else {
        int rc = select_disk(ctx, pts, px, py, rsel, (uint32_t *)bc.p, cum, &m);
        if (rc) return rc;
        if (m != cum) return set_error(ctx, SPADE_E_HIP, "internal: circle count and selection disagree");
        hipLaunchKernelGGL(k_knn_keys, dim3(dj_grid(m)), dim3(256), 0, st, m, (const uint32_t *)bc.p, pts->x, pts->y, px,
                           py, (unsigned long long *)bk.p);
    }
    SPADE_HIP(ctx, hipGetLastError());
    // order by distance, exactly; the first k are the result
    const int64_t kk = std::min<int64_t>(k, m);
    unsigned long long *sorted = (unsigned long long *)bk.p;
    uint32_t *sids = (uint32_t *)bc.p;
    if (m <= KS_MAX) {
        hipLaunchKernelGGL(k_knn_order, dim3(1), dim3(KS_THREADS), 0, st, (int)m, sorted, sids);
    } else {
        const unsigned long long *keys = (const unsigned long long *)(placed ? bk2.p : bk.p);
        const uint32_t *ids = (const uint32_t *)(placed ? bi.p : bc.p);
        sorted = (unsigned long long *)(placed ? bk.p : bk2.p);
        sids = (uint32_t *)(placed ? bc.p : bi.p);
        tb = 0;
        SPADE_HIP(ctx, hipcub::DeviceRadixSort::SortPairs(nullptr, tb, keys, sorted, ids, sids, (int)m, 0, 64, st));
        if (ensure(ctx, cub, std::max<size_t>(tb, 1))) return SPADE_E_NOMEM;
        SPADE_HIP(ctx, hipcub::DeviceRadixSort::SortPairs(cub.p, tb, keys, sorted, ids, sids, (int)m, 0, 64, st));
    }
    SPADE_HIP(ctx, hipGetLastError());
    hipLaunchKernelGGL(k_knn_fix, dim3(dj_grid(kk)), dim3(256), 0, st, m, kk, (const unsigned long long *)sorted, sids,
                       pts->x, pts->y, px, py, out_ids);
    SPADE_HIP(ctx, hipGetLastError());
    if (ctx->timing) SPADE_HIP(ctx, hipEventRecord(ctx->ev[3], st));
    SPADE_HIP(ctx, hipStreamSynchronize(st));
    *n_out = kk;
    return SPADE_OK;
}

}  // namespace spade
