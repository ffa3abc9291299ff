// rbf_knn: exact k-nearest-neighbour stencils on the GPU.
//
// Sec. 2.2 builds row r of D^(alpha,beta) from the n nearest beta-nodes of
// the alpha-node r.  The stencil is defined as the first k beta-nodes in the
// order of the key (d^2, index), with d^2 = dx*dx + dy*dy evaluated with
// separately rounded products (this file is compiled with
// -ffp-contract=off), so the result is unique even on lattices with ties.
//
// Method: a uniform cell grid over the source bounding box (counting sort of
// the sources by cell), then one thread per query (k_query): the cells that
// cover a square of half-width R around it, R from the density of the 5 x 5
// cells there, are scanned row by row (the sources of neighbouring cells of a
// row are contiguous), R being raised until they hold k; when the k-th distance
// exceeds R, again with R raised to it, which is then final.
#include <algorithm>
#include <climits>
#include <cmath>
#include <mutex>

#include "common.h"

namespace {

// Cell grid, made on the device (k_grid).  err: 1 non-finite sources, 2
// non-finite queries (nothing is searched then).
struct Grid {
    double x0, y0, c, inv_c;
    int gx, gy, err;
};

__device__ __forceinline__ int cell_coord(double v, double v0, double inv_c, int g) {
    const double t = floor((v - v0) * inv_c);
    return (t >= 1.0) ? (t >= (double)g ? g - 1 : (int)t) : 0;  // 0 for NaN too
}

// Per-block bounding box of the sources (blockIdx.y = 0) and queries (1) plus a
// non-finite flag: part[5 b + 0..3] = min x, max x, min y, max y over the finite
// points, part[5 b + 4] = 1 if any coordinate is NaN or infinite (fmin/fmax
// alone would skip a NaN).  Clears the cells' counts as well.
__global__ void k_bbox_partial(const double *__restrict__ xs, int64_t ns,
                               const double *__restrict__ xq, int64_t nq, double *__restrict__ part,
                               int *__restrict__ count, int64_t ncell) {
    for (int64_t i = (blockIdx.y * (int64_t)gridDim.x + blockIdx.x) * blockDim.x + threadIdx.x;
         i < ncell; i += 2 * (int64_t)gridDim.x * blockDim.x)
        count[i] = 0;
    const double *x = blockIdx.y ? xq : xs;
    const int64_t n = blockIdx.y ? nq : ns;
    part += (int64_t)blockIdx.y * 5 * gridDim.x;
    __shared__ double lds[5 * 16];
    double v[5] = {INFINITY, -INFINITY, INFINITY, -INFINITY, 0.0};
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        double px = x[i], py = x[n + i];
        v[0] = fmin(v[0], px);
        v[1] = fmax(v[1], px);
        v[2] = fmin(v[2], py);
        v[3] = fmax(v[3], py);
        if (!isfinite(px) || !isfinite(py)) v[4] = 1.0;
    }
    for (int off = 32; off >= 1; off >>= 1) {
        v[0] = fmin(v[0], __shfl_xor(v[0], off, 64));
        v[1] = fmax(v[1], __shfl_xor(v[1], off, 64));
        v[2] = fmin(v[2], __shfl_xor(v[2], off, 64));
        v[3] = fmax(v[3], __shfl_xor(v[3], off, 64));
        v[4] = fmax(v[4], __shfl_xor(v[4], off, 64));
    }
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
    if (lane == 0)
        for (int q = 0; q < 5; ++q) lds[q * 16 + wid] = v[q];
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < nw; ++w) {
            v[0] = fmin(v[0], lds[w]);
            v[1] = fmax(v[1], lds[16 + w]);
            v[2] = fmin(v[2], lds[32 + w]);
            v[3] = fmax(v[3], lds[48 + w]);
            v[4] = fmax(v[4], lds[64 + w]);
        }
        for (int q = 0; q < 5; ++q) part[blockIdx.x * 5 + q] = v[q];
    }
}

constexpr int kBboxBlocks = 256;

// Cells of a grid over ns sources, at most.
__host__ __device__ inline int64_t max_cells(int64_t ns) { return ns / 2 + 8194; }

// Grid from the partial boxes, one block of kBboxBlocks threads.  Two sources
// per cell on average, at most 4096 cells along the longer side.
__global__ void __launch_bounds__(kBboxBlocks) k_grid(const double *__restrict__ part, int64_t ns,
                                                      Grid *__restrict__ g) {
    __shared__ double lds[6][kBboxBlocks];
    const int t = threadIdx.x;
    for (int q = 0; q < 5; ++q) lds[q][t] = part[5 * t + q];
    lds[5][t] = part[5 * (kBboxBlocks + t) + 4];
    for (int w = kBboxBlocks / 2; w > 0; w >>= 1) {
        __syncthreads();
        if (t < w) {
            lds[0][t] = fmin(lds[0][t], lds[0][t + w]);
            lds[1][t] = fmax(lds[1][t], lds[1][t + w]);
            lds[2][t] = fmin(lds[2][t], lds[2][t + w]);
            lds[3][t] = fmax(lds[3][t], lds[3][t + w]);
            lds[4][t] = fmax(lds[4][t], lds[4][t + w]);
            lds[5][t] = fmax(lds[5][t], lds[5][t + w]);
        }
    }
    if (t != 0) return;
    Grid r{};
    // Roots before the product, which could leave the range of doubles.
    const double ex = lds[1][0] - lds[0][0], ey = lds[3][0] - lds[2][0];
    double c = sqrt(fmax(ex, 0.0)) * sqrt(fmax(ey, 0.0)) * sqrt(2.0 / (double)ns);
    c = fmax(c, fmax(ex, ey) / 4096.0);
    if (!(c > 0.0)) c = 1.0;
    r.x0 = lds[0][0];
    r.y0 = lds[2][0];
    // One cell where the extents or the reciprocal are not finite, larger ones
    // should rounding exceed the buffers.
    if (!isfinite(ex) || !isfinite(ey) || !isfinite(1.0 / c)) c = INFINITY;
    for (;; c *= 2.0) {
        const bool one = !(c < INFINITY);
        r.c = c;
        r.inv_c = one ? 0.0 : 1.0 / c;
        r.gx = one ? 1 : (int)(ex * r.inv_c) + 1;
        r.gy = one ? 1 : (int)(ey * r.inv_c) + 1;
        if (one || (int64_t)r.gx * r.gy <= max_cells(ns)) break;
    }
    r.err = (lds[4][0] != 0.0) ? 1 : (lds[5][0] != 0.0) ? 2 : 0;
    *g = r;
}

__global__ void k_cell_count(const double *__restrict__ x, int64_t n, const Grid *__restrict__ gp,
                             int *__restrict__ cell, int *__restrict__ count) {
    const Grid g = *gp;
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n || g.err) return;
    const int cx = cell_coord(x[i], g.x0, g.inv_c, g.gx);
    const int cy = cell_coord(x[n + i], g.y0, g.inv_c, g.gy);
    const int c = cy * g.gx + cx;
    cell[i] = c;
    atomicAdd(&count[c], 1);
}

// Exclusive scan of the cells' counts into start[0..n], n = gx gy, in chunks of
// at least kScanTile cells, at most kScanBlocks of them: chunk sums, then each
// block adds the sums before its own and scans its chunk.  (One workgroup for
// the whole array, as before, took 922 us for 500,000 cells.)
constexpr int kScanT = 256, kScanV = 8, kScanTile = kScanT * kScanV, kScanBlocks = 1024;

__device__ __forceinline__ int64_t scan_chunk(int64_t n) {
    const int64_t per = (n + kScanBlocks - 1) / kScanBlocks;
    return per < kScanTile ? kScanTile : (per + kScanTile - 1) / kScanTile * kScanTile;
}

// Sum of v over the block, in every thread.
__device__ __forceinline__ int block_sum_i32(int v, int *lds) {
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = v;
    __syncthreads();
    int s = 0;
    for (int w = 0; w < kScanT / 64; ++w) s += lds[w];
    return s;
}

__global__ void __launch_bounds__(kScanT) k_scan_sums(const Grid *__restrict__ g,
                                                      const int *__restrict__ count,
                                                      int *__restrict__ sums) {
    __shared__ int lds[kScanT / 64];
    const int64_t n = (int64_t)g->gx * g->gy, chunk = scan_chunk(n);
    const int64_t a = blockIdx.x * chunk, b = min(a + chunk, n);
    int s = 0;
    for (int64_t i = a + threadIdx.x; i < b; i += kScanT) s += count[i];
    s = block_sum_i32(s, lds);
    if (threadIdx.x == 0) sums[blockIdx.x] = s;
}

__global__ void __launch_bounds__(kScanT) k_scan(const Grid *__restrict__ g,
                                                 const int *__restrict__ count,
                                                 const int *__restrict__ sums,
                                                 int *__restrict__ start) {
    __shared__ int lds[kScanT / 64], tot[kScanT];
    const int64_t n = (int64_t)g->gx * g->gy, chunk = scan_chunk(n);
    const int64_t a = blockIdx.x * chunk, b = min(a + chunk, n);
    if (a >= n) return;
    const int t = threadIdx.x;
    int s = 0;
    for (int q = t; q < (int)blockIdx.x; q += kScanT) s += sums[q];
    int carry = block_sum_i32(s, lds);
    for (int64_t base = a; base < b; base += kScanTile) {
        const int64_t i0 = base + (int64_t)t * kScanV;
        int v[kScanV], run = 0;
#pragma unroll
        for (int j = 0; j < kScanV; ++j) {
            v[j] = run;
            run += (i0 + j < b) ? count[i0 + j] : 0;
        }
        __syncthreads();
        tot[t] = run;
        __syncthreads();
        for (int off = 1; off < kScanT; off <<= 1) {
            const int add = (t >= off) ? tot[t - off] : 0;
            __syncthreads();
            tot[t] += add;
            __syncthreads();
        }
        const int before = carry + tot[t] - run;
#pragma unroll
        for (int j = 0; j < kScanV; ++j)
            if (i0 + j < b) start[i0 + j] = before + v[j];
        carry += tot[kScanT - 1];
    }
    if (b == n && t == 0) start[n] = carry;
}

// Sources into their cells; count is used up as each cell's cursor.
__global__ void k_scatter(const double *__restrict__ x, int64_t n, const Grid *__restrict__ g,
                          const int *__restrict__ cell, const int *__restrict__ start,
                          int *__restrict__ count, double2 *__restrict__ sxy,
                          int *__restrict__ sid) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n || g->err) return;
    const int c = cell[i];
    const int pos = start[c] + atomicSub(&count[c], 1) - 1;
    sxy[pos] = double2{x[i], x[n + i]};
    sid[pos] = (int)i;
}

__device__ __forceinline__ double dist2(double2 s, double qx, double qy) {
    const double dx = s.x - qx, dy = s.y - qy;
    return dx * dx + dy * dy;
}

// Calls f(p, |s_p - q|^2) for every source p of the cells x0..x1, y0..y1; the
// next row's range and the next U sources are loaded while these are looked at.
template <int U, class F>
__device__ __forceinline__ void scan_cells(const int *__restrict__ start,
                                           const double2 *__restrict__ sxy, int gx, int x0, int x1,
                                           int y0, int y1, double qx, double qy, F f) {
    int64_t row = (int64_t)y0 * gx;
    int pa = start[row + x0], pb = start[row + x1 + 1];
    for (int y = y0; y <= y1; ++y) {
        if (y < y1) row += gx;
        const int na = start[row + x0], nb = start[row + x1 + 1];
        if (pa < pb) {
            int p = pa;
            double2 s[U], t[U];
            auto load = [&](double2(&v)[U], int at) {
#pragma unroll
                for (int u = 0; u < U; ++u) v[u] = sxy[min(at + u, pb - 1)];
            };
            load(s, p);
            for (; p + U <= pb; p += U) {
                load(t, p + U);
#pragma unroll
                for (int u = 0; u < U; ++u) f(p + u, dist2(s[u], qx, qy));
#pragma unroll
                for (int u = 0; u < U; ++u) s[u] = t[u];
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (p + u < pb) f(p + u, dist2(s[u], qx, qy));
        }
        pa = na;
        pb = nb;
    }
}

// One query per thread, k <= KMAX.  `nearest` keeps the KMAX smallest squared
// distances, sorted, in registers: each candidate goes through one min/max
// chain (two instructions per entry, no indices).  Then the sources
// within the k-th distance are listed (LDS), and each goes to the place that the number
// of smaller distances gives; equal distances are inserted by index.
// The chain's instructions take most of the time on even sets: 10^6 queries,
// k = 28: 452 us; an insertion of (distance, index) pairs by compare and select,
// ring by ring, took 1,928 us (5,700 queries: 82 against 326 us).  On uneven sets, where
// a cell holds thousands of sources, it is the latency of the loads: hence those of
// the next U sources ahead, and a second pass only over a window that holds more
// sources (30,000 sources normal^3, 10,000 queries, whole call: k = 28 4.0 ms,
// k = 64 11.9; two sources ahead and every window again in full 5.4 and 15.4; ring
// by ring 4.2 and 13.4).
constexpr int kQueryT = 64, kListMore = 12;
template <int KMAX>
__global__ void __launch_bounds__(kQueryT) k_query(const double *__restrict__ xq, int64_t nq, int k,
                                                   const Grid *__restrict__ gp,
                                                   const int *__restrict__ start,
                                                   const double2 *__restrict__ sxy,
                                                   const int *__restrict__ sid,
                                                   int *__restrict__ idx) {
    constexpr int CAP = KMAX + kListMore;
    constexpr int kEmpty = 255;
    constexpr int U = KMAX <= 48 ? 4 : 3;  // 10^6 queries, k = 64: 1,955 us, 2,105 with 4
    __shared__ int list[CAP][kQueryT];             // accepted sources, then their indices
    __shared__ unsigned char place[KMAX][kQueryT];  // list entry at each place of the stencil
    static_assert(CAP < kEmpty, "list entries are numbered in bytes");
    const int64_t q = (int64_t)rbf::xcd_block(blockIdx.x, gridDim.x) * kQueryT + threadIdx.x;
    const Grid g = *gp;
    if (q >= nq || g.err) return;
    const int t = threadIdx.x;
    const double qx = xq[q], qy = xq[nq + q];
    int x0, x1, y0, y1;  // cells scanned: the window
    auto count = [&]() {  // sources in them
        int n = 0;
        for (int y = y0; y <= y1; ++y)
            n += start[(int64_t)y * g.gx + x1 + 1] - start[(int64_t)y * g.gx + x0];
        return n;
    };
    double out, r;  // distance to the box of the grid; reach of the window into it
    {
        // Radius of 1.5 k sources at the density of the 5 x 5 cells here.
        const int cx = cell_coord(qx, g.x0, g.inv_c, g.gx), cy = cell_coord(qy, g.y0, g.inv_c, g.gy);
        x0 = max(cx - 2, 0), x1 = min(cx + 2, g.gx - 1);
        y0 = max(cy - 2, 0), y1 = min(cy + 2, g.gy - 1);
        const int n = count();
        const double cells = (double)((x1 - x0 + 1) * (y1 - y0 + 1));
        r = g.c * sqrt(1.5 / M_PI * (double)k * cells / (double)max(n, 1));
        out = fmax(fmax(g.x0 - qx, qx - (g.x0 + g.gx * g.c)), fmax(g.y0 - qy, qy - (g.y0 + g.gy * g.c)));
        out = (out > 0.0) ? out : 0.0;
    }
    double bd[KMAX], T;
    // Cells that hold every source within r (with a margin for rounding;
    // cell_coord is monotonic).
    auto window = [&](double r) {
        const double m = r * (1.0 + 1e-9) + 1e-9 * g.c;
        x0 = cell_coord(qx - m, g.x0, g.inv_c, g.gx), x1 = cell_coord(qx + m, g.x0, g.inv_c, g.gx);
        y0 = cell_coord(qy - m, g.y0, g.inv_c, g.gy), y1 = cell_coord(qy + m, g.y0, g.inv_c, g.gy);
    };
    int n;
    // The smallest squared distances of the window's sources, of those below limit; n
    // sources seen, T the k-th.
    auto nearest = [&](double limit) {
#pragma unroll
        for (int s = 0; s < KMAX; ++s) bd[s] = limit;
        n = 0;
        scan_cells<U>(start, sxy, g.gx, x0, x1, y0, y1, qx, qy, [&](int, double d) {
            ++n;
            if (d < bd[KMAX - 1]) {
#pragma unroll
                for (int s = KMAX - 1; s > 0; --s) bd[s] = fmin(bd[s], fmax(bd[s - 1], d));
                bd[0] = fmin(bd[0], d);
            }
        });
        T = bd[KMAX - 1];
#pragma unroll
        for (int s = 0; s < KMAX - 1; ++s) T = (s == k - 1) ? bd[s] : T;
    };
    auto all = [&]() { return x0 == 0 && y0 == 0 && x1 == g.gx - 1 && y1 == g.gy - 1; };
    // A query outside the box whose window is most of it takes all of it, so that the
    // queries of a wave read the same sources together (30,000 normal sources, queries ten
    // box sides away: 4.0 ms, up to 11 with windows of their own).
    auto widen = [&]() {
        if (out > 0.0 && 2 * (int64_t)(x1 - x0 + 1) * (y1 - y0 + 1) > (int64_t)g.gx * g.gy)
            x0 = y0 = 0, x1 = g.gx - 1, y1 = g.gy - 1;
    };
    // Until k sources are in the window.  (The queries of a wave reach the second part
    // together: windows grown by each in its own pass cost them one another's.)
    double R = out + r;
    window(R);
    for (;;) {
        nearest(INFINITY);
        if (n >= k || all()) break;
        do {
            R = out + (r *= 1.1);
            window(R);
        } while (count() < k && !all());
    }
    // Final when every source outside is farther than T: R^2 must be in the normal
    // range for that.  Else again with the cells that cover T (all where that cannot
    // be told) if they hold more, with only what is nearer than (1 + 1e-15) T of
    // interest.
    if (!all() && !(T <= R * R && T < INFINITY && R * R > 1e-290)) {
        const bool known = T < INFINITY && T > 1e-290;
        window(known ? fmax(sqrt(T) * (1.0 + 1e-15), R) : INFINITY);
        widen();
        if (count() > n) nearest(known ? T * (1.0 + 1e-15) : INFINITY);
    }
    // (Where T is below 1e-290: a difference above its root has a larger square.)
    if (T < INFINITY) window(sqrt(fmax(T, 1e-290)) * (1.0 + 1e-15));
    widen();
    n = 0;
    scan_cells<U>(start, sxy, g.gx, x0, x1, y0, y1, qx, qy, [&](int p, double d) {
        if (d <= T) {
            if (n < CAP) list[n][t] = p;
            ++n;
        }
    });
    // More than the list holds, many at the k-th distance: the nearer ones, fewer than
    // k, are listed again; of those at it the lowest indices follow below.
    const bool over = n > CAP;
    if (over) {
        n = 0;
        scan_cells<U>(start, sxy, g.gx, x0, x1, y0, y1, qx, qy, [&](int p, double d) {
            if (d < T) list[n++][t] = p;
        });
    }
    bool tie = n > k;
#pragma unroll
    for (int s = 0; s + 1 < KMAX; ++s) tie = tie || (s + 1 < k && bd[s] == bd[s + 1]);
#pragma unroll 1
    for (int s = 0; s < k; ++s) place[s][t] = kEmpty;
#pragma unroll 1
    for (int i = 0; i < n; ++i) {
        const int p = list[i][t];
        const double d = dist2(sxy[p], qx, qy);
        int id = sid[p];
        list[i][t] = id;
        int r = 0;
#pragma unroll
        for (int s = 0; s < KMAX; ++s) r += (bd[s] < d) ? 1 : 0;
        if (!tie) {
            place[r][t] = (unsigned char)i;
            continue;
        }
        // The places r .. end - 1 belong to this distance: insert by index.
        int end = r;
#pragma unroll
        for (int s = 0; s < KMAX; ++s) end += (s < k && bd[s] == d) ? 1 : 0;
        int at = i;
        for (; r < end; ++r) {
            const int other = place[r][t];
            if (other == kEmpty) {
                place[r][t] = (unsigned char)at;
                break;
            }
            const int oid = list[other][t];
            if (id < oid) {
                place[r][t] = (unsigned char)at;
                at = other;
                id = oid;
            }
        }
    }
    const int m = min(n, k);
#pragma unroll 1
    for (int s = 0; s < m; ++s) idx[(int64_t)s * nq + q] = list[place[s][t]][t];
    if (!over) return;
    int id[KMAX];  // the lowest indices at distance T, sorted
#pragma unroll
    for (int s = 0; s < KMAX; ++s) id[s] = INT_MAX;
    scan_cells<U>(start, sxy, g.gx, x0, x1, y0, y1, qx, qy, [&](int p, double d) {
        if (d != T) return;
        const int i = sid[p];
        if (i < id[KMAX - 1]) {
#pragma unroll
            for (int s = KMAX - 1; s > 0; --s) id[s] = min(id[s], max(id[s - 1], i));
            id[0] = min(id[0], i);
        }
    });
#pragma unroll
    for (int s = 0; s < KMAX; ++s)
        if (m + s < k) idx[(int64_t)(m + s) * nq + q] = id[s];
}

// Device buffers of one kNN call besides its inputs and output.
struct KnnScratch {
    Grid *grid;
    double *part;  // [2][kBboxBlocks][5] bounding-box partials (sources, queries)
    int *cell, *count, *start, *sums, *sid;
    double2 *sxy;
};

size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

// Lays the buffers out from base; returns their size (base may be null).
size_t carve(char *base, int64_t ns, KnnScratch &s) {
    size_t at = 0;
    auto take = [&](size_t b) {
        char *p = base ? base + at : nullptr;
        at += align256(b);
        return p;
    };
    s.grid = (Grid *)take(sizeof(Grid));
    s.part = (double *)take(2 * kBboxBlocks * 5 * sizeof(double));
    s.sums = (int *)take(kScanBlocks * sizeof(int));
    s.cell = (int *)take(ns * sizeof(int));
    s.sid = (int *)take(ns * sizeof(int));
    s.sxy = (double2 *)take(ns * sizeof(double2));
    s.count = (int *)take(max_cells(ns) * sizeof(int));
    s.start = (int *)take((max_cells(ns) + 1) * sizeof(int));
    return at;
}

rbf_status knn_check_args(const double *xq, int64_t nq, const double *xs, int64_t ns, int32_t k,
                          int32_t *idx) {
    RBF_ARG(k >= 1 && k <= 64, "rbf_knn: k must be in [1, 64] (got %d)", k);
    RBF_ARG(ns >= 1 && k <= ns, "rbf_knn: need 1 <= k <= ns (k=%d, ns=%lld)", k, (long long)ns);
    RBF_ARG(nq >= 0 && nq < INT_MAX && ns < INT_MAX, "rbf_knn: sizes out of range");
    RBF_ARG(xs && (nq == 0 || (xq && idx)), "rbf_knn: NULL pointer");
    return RBF_OK;
}

// Cell grid, counting sort of the sources by cell, then the queries; one
// synchronisation at the end.
rbf_status knn_search(const double *xq, int64_t nq, const double *xs, int64_t ns, int32_t k,
                      int32_t *idx, hipStream_t st, const KnnScratch &s) {
    const int64_t ncell = max_cells(ns);
    const uint32_t sb = (uint32_t)std::min<int64_t>(rbf::blocks_for(ncell, kScanTile), kScanBlocks);
    const dim3 gs(rbf::blocks_for(ns, 256)), b256(256), bs(kScanT);
    hipLaunchKernelGGL(k_bbox_partial, dim3(kBboxBlocks, 2), dim3(256), 0, st, xs, ns, xq, nq, s.part, s.count, ncell);
    hipLaunchKernelGGL(k_grid, dim3(1), dim3(kBboxBlocks), 0, st, s.part, ns, s.grid);
    hipLaunchKernelGGL(k_cell_count, gs, b256, 0, st, xs, ns, s.grid, s.cell, s.count);
    hipLaunchKernelGGL(k_scan_sums, dim3(sb), bs, 0, st, s.grid, s.count, s.sums);
    hipLaunchKernelGGL(k_scan, dim3(sb), bs, 0, st, s.grid, s.count, s.sums, s.start);
    hipLaunchKernelGGL(k_scatter, gs, b256, 0, st, xs, ns, s.grid, s.cell, s.start, s.count, s.sxy, s.sid);
    const dim3 gq(rbf::blocks_for(nq, kQueryT)), bq(kQueryT);
#define RBF_QUERY(KM) \
    hipLaunchKernelGGL(k_query<KM>, gq, bq, 0, st, xq, nq, k, s.grid, s.start, s.sxy, s.sid, idx)
    // The chain's length is fixed at compile time; 28 is the paper's stencil.
    if (k <= 16) RBF_QUERY(16);
    else if (k <= 28) RBF_QUERY(28);
    else if (k <= 32) RBF_QUERY(32);
    else if (k <= 48) RBF_QUERY(48);
    else RBF_QUERY(64);
#undef RBF_QUERY
    Grid g{};
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipMemcpyAsync(&g, s.grid, sizeof(g), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) {
        rbf::set_error("rbf_knn: %s", hipGetErrorString(e));
        return RBF_E_DEVICE;
    }
    RBF_ARG(g.err != 1, "rbf_knn: non-finite source coordinates");
    RBF_ARG(g.err != 2, "rbf_knn: non-finite query coordinates");
    return RBF_OK;
}

}  // namespace

extern "C" rbf_status rbf_knn(const double *xq, int64_t nq, const double *xs, int64_t ns,
                              int32_t k, int32_t *idx, rbf_stream st_) {
    rbf::clear_error();
    rbf_status rc = knn_check_args(xq, nq, xs, ns, k, idx);
    if (rc != RBF_OK || nq == 0) return rc;
    KnnScratch s{};
    char *base = nullptr;
    if (hipMalloc(&base, carve(nullptr, ns, s)) != hipSuccess) {
        rbf::set_error("rbf_knn: device allocation failed");
        return RBF_E_NOMEM;
    }
    carve(base, ns, s);
    rc = knn_search(xq, nq, xs, ns, k, idx, rbf::as_stream(st_), s);
    (void)hipFree(base);
    return rc;
}

// ------------------------------------------------------ no-allocation form --
// A fixed per-device scratch array for callers that cannot allocate device
// memory.  In host code `scratch` names a host-side stand-in, not device
// memory: its device address is taken once per device with
// hipGetSymbolAddress and only that address is used.
namespace {

constexpr size_t kScratchBytes = size_t(64) << 20;
__device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
char *g_scratch_addr[kMaxDevices] = {};

// Device address of `scratch` on the current device (looked up on the first
// call on that device, with that device current).
rbf_status scratch_address(char **out) {
    int dev = -1;
    RBF_HIP(hipGetDevice(&dev));
    RBF_ARG(dev >= 0 && dev < kMaxDevices, "rbf_knn_noalloc: device ordinal %d out of range", dev);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_addr[dev]) {
        void *p = nullptr;
        RBF_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        RBF_ARG(p != nullptr, "rbf_knn_noalloc: no device address for the scratch array");
        g_scratch_addr[dev] = static_cast<char *>(p);
    }
    *out = g_scratch_addr[dev];
    return RBF_OK;
}

}  // namespace

extern "C" rbf_status rbf_knn_noalloc(const double *xq, int64_t nq, const double *xs, int64_t ns,
                                      int32_t k, int32_t *idx, rbf_stream st_) {
    rbf::clear_error();
    rbf_status rc = knn_check_args(xq, nq, xs, ns, k, idx);
    if (rc != RBF_OK || nq == 0) return rc;
    KnnScratch s{};
    // Limit: coordinates, two ints per source and three per cell (the buffers
    // stay below it).
    const size_t part_bytes = align256(2 * kBboxBlocks * 5 * sizeof(double));
    const size_t limit_bytes = part_bytes + 2 * align256(ns * sizeof(int)) +
                               2 * align256(ns * sizeof(double)) +
                               2 * align256(max_cells(ns) * sizeof(int)) +
                               align256((max_cells(ns) + 1) * sizeof(int));
    RBF_ARG(limit_bytes <= kScratchBytes && carve(nullptr, ns, s) <= kScratchBytes,
            "rbf_knn_noalloc: %lld sources exceed the %zu-byte scratch array (at most about "
            "%lld sources)",
            (long long)ns, kScratchBytes,
            (long long)((kScratchBytes - part_bytes - 8194 * 12 - 2048) / 30));
    char *base = nullptr;
    rc = scratch_address(&base);
    if (rc != RBF_OK) return rc;
    carve(base, ns, s);
    return knn_search(xq, nq, xs, ns, k, idx, rbf::as_stream(st_), s);
}
