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
// row are contiguous); when the k-th distance exceeds R, again with R raised
// to it, which is then final.
#include <algorithm>
#include <climits>
#include <cmath>
#include <mutex>

#include "common.h"

namespace {

// Cell grid, made on the device (k_grid).  err: 1 non-finite sources, 2
// non-finite queries (nothing is searched then).  left: queries that k_query
// left to k_query_general.
struct Grid {
    double x0, y0, c, inv_c;
    int gx, gy, err;
    unsigned left;
};

__device__ __forceinline__ bool key_less(double d, int i, double bd, int bi) {
    return d < bd || (d == bd && i < bi);
}

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
// next row's range is loaded while a row is scanned.
template <class F>
__device__ __forceinline__ void scan_cells(const int *__restrict__ start,
                                           const double2 *__restrict__ sxy, int gx, int x0, int x1,
                                           int y0, int y1, double qx, double qy, F f) {
    int64_t row = (int64_t)y0 * gx;
    int pa = start[row + x0], pb = start[row + x1 + 1];
    for (int y = y0; y <= y1; ++y) {
        row += gx;
        const int64_t nrow = (y < y1) ? row : row - gx;
        const int na = start[nrow + x0], nb = start[nrow + x1 + 1];
        int p = pa;
        for (; p + 1 < pb; p += 2) {
            const double2 s0 = sxy[p], s1 = sxy[p + 1];
            f(p, dist2(s0, qx, qy));
            f(p + 1, dist2(s1, qx, qy));
        }
        if (p < pb) f(p, dist2(sxy[p], qx, qy));
        pa = na;
        pb = nb;
    }
}

// One query per thread, k <= KMAX.  Pass A keeps the KMAX smallest squared
// distances, sorted, in registers: each candidate goes through one min/max
// chain (two instructions per entry, no indices).  Pass B lists the sources
// within the k-th distance (LDS), and each goes to the place that the number of
// smaller distances gives; equal distances are inserted by index.
// A query with more sources than the list holds (many at one distance) is left
// to k_query_general: its first entry is set to -1 and counted.
// Bound by the instructions of the chain.  10^6 queries, k = 28: 452 us; an
// insertion of (distance, index) pairs by compare and select, ring by ring,
// took 1,928 us (5,700 queries: 82 against 326 us).
constexpr int kQueryT = 64, kListMore = 12;
template <int KMAX>
__global__ void __launch_bounds__(kQueryT) k_query(const double *__restrict__ xq, int64_t nq, int k,
                                                   Grid *__restrict__ gp,
                                                   const int *__restrict__ start,
                                                   const double2 *__restrict__ sxy,
                                                   const int *__restrict__ sid,
                                                   int *__restrict__ idx) {
    constexpr int CAP = KMAX + kListMore;
    constexpr int kEmpty = 255;
    __shared__ int list[CAP][kQueryT];             // accepted sources, then their indices
    __shared__ unsigned char place[KMAX][kQueryT];  // list entry at each place of the stencil
    static_assert(CAP < kEmpty, "list entries are numbered in bytes");
    const int64_t q = (int64_t)rbf::xcd_block(blockIdx.x, gridDim.x) * kQueryT + threadIdx.x;
    const Grid g = *gp;
    if (q >= nq || g.err) return;
    const int t = threadIdx.x;
    const double qx = xq[q], qy = xq[nq + q];
    int x0, x1, y0, y1;  // cells scanned
    double R;
    {
        // Radius of 1.5 k sources at the density of the 5 x 5 cells here.
        const int cx = cell_coord(qx, g.x0, g.inv_c, g.gx), cy = cell_coord(qy, g.y0, g.inv_c, g.gy);
        x0 = max(cx - 2, 0), x1 = min(cx + 2, g.gx - 1);
        y0 = max(cy - 2, 0), y1 = min(cy + 2, g.gy - 1);
        int n = 0;
        for (int y = y0; y <= y1; ++y)
            n += start[(int64_t)y * g.gx + x1 + 1] - start[(int64_t)y * g.gx + x0];
        const double cells = (double)((x1 - x0 + 1) * (y1 - y0 + 1));
        R = g.c * sqrt(1.5 / M_PI * (double)k * cells / (double)max(n, 1));
    }
    double bd[KMAX], T;
    // Cells that hold every source within r (with a margin for rounding;
    // cell_coord is monotonic).
    auto window = [&](double r) {
        const double m = r * (1.0 + 1e-9) + 1e-9 * g.c;
        x0 = cell_coord(qx - m, g.x0, g.inv_c, g.gx), x1 = cell_coord(qx + m, g.x0, g.inv_c, g.gx);
        y0 = cell_coord(qy - m, g.y0, g.inv_c, g.gy), y1 = cell_coord(qy + m, g.y0, g.inv_c, g.gy);
    };
    for (;;) {
        window(R);
#pragma unroll
        for (int s = 0; s < KMAX; ++s) bd[s] = INFINITY;
        int n = 0;
        scan_cells(start, sxy, g.gx, x0, x1, y0, y1, qx, qy, [&](int, double d) {
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
        // Final when every source outside is farther than T: R^2 must be in the
        // normal range for that, else all cells are scanned.
        const double R2 = R * R;
        const bool all = x0 == 0 && y0 == 0 && x1 == g.gx - 1 && y1 == g.gy - 1;
        if (all || (n >= k && T <= R2 && T < INFINITY && R2 > 1e-290)) break;
        if (n < k) R *= 1.5;
        else R = (T < INFINITY && T > 1e-290) ? fmax(sqrt(T) * (1.0 + 1e-15), R) : INFINITY;
    }
    if (T < INFINITY && T > 1e-290) window(sqrt(T) * (1.0 + 1e-15));
    int n = 0;
    scan_cells(start, sxy, g.gx, x0, x1, y0, y1, qx, qy, [&](int p, double d) {
        if (d <= T) {
            if (n < CAP) list[n][t] = p;
            ++n;
        }
    });
    if (n > CAP) {
        idx[q] = -1;
        atomicAdd(&gp->left, 1u);
        return;
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
#pragma unroll 1
    for (int s = 0; s < k; ++s) idx[(int64_t)s * nq + q] = list[place[s][t]][t];
}

// The same search for the queries that k_query left (idx[q] = -1): square rings
// of cells outward, the best k candidates as a list of (distance, index) sorted
// by insertion.
template <int KMAX>
__global__ void __launch_bounds__(128) k_query_general(const double *__restrict__ xq, int64_t nq,
                                                       int k, const Grid *__restrict__ gp,
                                                       const int *__restrict__ start,
                                                       const double2 *__restrict__ sxy,
                                                       const int *__restrict__ sid,
                                                       int *__restrict__ idx) {
    const int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (q >= nq || idx[q] != -1) return;
    const Grid g = *gp;
    const double qx = xq[q], qy = xq[nq + q];
    const int cx = cell_coord(qx, g.x0, g.inv_c, g.gx);
    const int cy = cell_coord(qy, g.y0, g.inv_c, g.gy);
    double bd[KMAX];
    int bi[KMAX];
#pragma unroll
    for (int s = 0; s < KMAX; ++s) {
        bd[s] = INFINITY;
        bi[s] = INT_MAX;
    }
    double thr_d = INFINITY;
    int thr_i = INT_MAX;
    const int rmax = max(max(cx, g.gx - 1 - cx), max(cy, g.gy - 1 - cy));
    for (int r = 0; r <= rmax; ++r) {
        const int ylo = cy - r, yhi = cy + r;
        for (int iy = max(ylo, 0); iy <= min(yhi, g.gy - 1); ++iy) {
            const bool full_row = (iy == ylo) || (iy == yhi);
            const int step = full_row ? 1 : 2 * r;
            for (int ix = cx - r; ix <= cx + r; ix += (step > 0 ? step : 1)) {
                if (ix < 0 || ix >= g.gx) continue;
                const int c = iy * g.gx + ix;
                const int pe = start[c + 1];
                for (int p = start[c]; p < pe; ++p) {
                    const double d2 = dist2(sxy[p], qx, qy);
                    const int id = sid[p];
                    if (!key_less(d2, id, thr_d, thr_i)) continue;
                    // Sorted insertion; the former last entry drops out.
#pragma unroll
                    for (int s = KMAX - 1; s > 0; --s) {
                        const bool before_prev = key_less(d2, id, bd[s - 1], bi[s - 1]);
                        const bool before_cur = key_less(d2, id, bd[s], bi[s]);
                        if (before_prev) {
                            bd[s] = bd[s - 1];
                            bi[s] = bi[s - 1];
                        } else if (before_cur) {
                            bd[s] = d2;
                            bi[s] = id;
                        }
                    }
                    if (key_less(d2, id, bd[0], bi[0])) {
                        bd[0] = d2;
                        bi[0] = id;
                    }
#pragma unroll
                    for (int s = 0; s < KMAX; ++s)
                        if (s == k - 1) {
                            thr_d = bd[s];
                            thr_i = bi[s];
                        }
                }
                if (step == 0) break;
            }
        }
        if (thr_d == INFINITY) continue;  // fewer than k candidates so far
        // Distance from the query to the nearest cell outside the block.
        double bound = INFINITY;
        if (cx - r > 0) bound = fmin(bound, qx - (g.x0 + (double)(cx - r) * g.c));
        if (cx + r < g.gx - 1) bound = fmin(bound, (g.x0 + (double)(cx + r + 1) * g.c) - qx);
        if (cy - r > 0) bound = fmin(bound, qy - (g.y0 + (double)(cy - r) * g.c));
        if (cy + r < g.gy - 1) bound = fmin(bound, (g.y0 + (double)(cy + r + 1) * g.c) - qy);
        if (bound == INFINITY) break;
        bound -= 1e-9 * g.c;  // margin for the rounding of cell assignment
        if (bound > 0.0 && thr_d < bound * bound) break;
    }
#pragma unroll
    for (int s = 0; s < KMAX; ++s)
        if (s < k) idx[(int64_t)s * nq + q] = bi[s];
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
// synchronisation at the end (two when queries are left to k_query_general).
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
    if (e == hipSuccess && !g.err && g.left > 0) {
        const dim3 gg(rbf::blocks_for(nq, 128)), bg(128);
        if (k <= 32)
            hipLaunchKernelGGL(k_query_general<32>, gg, bg, 0, st, xq, nq, k, s.grid, s.start, s.sxy, s.sid, idx);
        else
            hipLaunchKernelGGL(k_query_general<64>, gg, bg, 0, st, xq, nq, k, s.grid, s.start, s.sxy, s.sid, idx);
        e = hipGetLastError();
        if (e == hipSuccess) e = hipStreamSynchronize(st);
    }
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
