// Pressure solve on general node sets: flexible GMRES (Saad 1993) right-
// preconditioned by a two-level auxiliary-lattice method.  Included by
// solver.hip inside its anonymous namespace (it uses the solver's Krylov
// helpers, the lattice transforms k_pc_fold / k_pc_tri / k_pc_gemm and rbf_solver).
//
// System: the row-scaled bordered Poisson operator of eq. (18),
//   A x = S A0 x + u1 c (1^T x),   S the row scale, u1 = S chi, c = vscale,
// A0: D_Lap^PP on interior rows, n . grad on wall rows (see k_build_poisson).
//
// Preconditioner z = B^-1 y (one application; two smoothing sweeps on each
// side of the lattice correction, the second of each pair weighted by w2):
//   x1 = W y, then x1 += w2 W (y - A_s x1)
//                                 W = omega / (l1 norm of A's rows)
//   r1 = y - A_s x1               A_s: the sparse part of A
//   g  = R (S^-1 r1)              R: normalised bilinear restriction of the
//                                 interior-node residuals to the interior
//                                 points of an auxiliary (Ka+1)^2 lattice
//                                 over the nodes' bounding square
//   e  = (L5)^+ (g - lam)         L5: 5-point Laplacian of the lattice with
//                                 one-sided homogeneous Neumann wall rows,
//                                 inverted by the fast transform (DCT-II along
//                                 x, tridiagonal along y); lam = mean of g,
//                                 e of zero mean
//   x2 = x1 + J e + mu            J: bilinear interpolation to the nodes
//                                 (wall lattice values copied inward);
//                                 mu = (lam / c - sum J e) / m carries the
//                                 border's constant (the exact form for the
//                                 bordered operator A0 + chi c 1^T)
//   z  = x2 + W (y - A_s x2), then z += w2 W (y - A_s z)
// The auxiliary lattice has about one node spacing per cell: the smoother
// removes what the lattice cannot represent, the
// lattice solve removes the smooth error the smoother cannot.  A_s 1 = 0
// (the rows reproduce constants), so mu needs no product.
//
// Precision: T = double (the FP64 solve) or float (mixed precision: each
// restart cycle is one step of iterative refinement whose residual
// b - A x is formed in FP64 from FP64 weights, the cycle itself runs on
// FP32-stored weights, vectors and transforms with FP64 dot products, and
// the correction is added to the FP64 iterate).
//
// FGMRES(mr) with classical Gram-Schmidt, one pass per step: a second one took the same
// number of steps to the same true residual on the h = 1/400 cavity and the cylinder
// (32.3 and 35.2 per time step) for a reduction and a pass over the basis more, and
// convergence is only declared from the true residual recomputed at a restart, so a
// loss of orthogonality can cost steps but not accuracy.  The Hessenberg
// column, the Givens rotations and the residual estimate are updated on the
// device by one workgroup per step; the host follows a word that it
// publishes in pinned memory.  All reductions are fixed-order (block partials reduced by
// one workgroup), so a solve is repeatable bit for bit.
#pragma once

constexpr int kFgMax = 30;        // restart length (basis vectors per cycle)
constexpr int kFgChunk = 6;       // dot products accumulated per pass over the rows
// Smoother damping of the l1-Jacobi sweeps: the l1 norms of RBF-FD rows are
// several times their diagonal, so steps up to about 2.4 still damp (FGMRES
// steps per solve at h = 1/100 and 1/200, rtol 1e-12: 111 and 118 at 1.3,
// 86 and 96 at 2.0, 78 and 84 at 2.4, divergent smoothing from 2.8).
constexpr double kAuxOmega = 2.0;
// Border scale of the FGMRES operator relative to the solver's: any scale
// gives the same p~ (the constant is removed afterwards); the solver's own
// scale happens to slow FGMRES (140 against 111 steps at h = 1/100 for 0.1
// or less of it).
constexpr double kAuxBorder = 0.1;
constexpr double kMixedInner = 1e-4;  // mixed: per-cycle residual reduction
// (Two smoothing sweeps on each side cost two more products per FGMRES step than one and
// cut the steps per solve by about a third: h = 1/100, rtol 1e-10, 71 steps with one
// sweep, 48 with two, 39 with three.)

template <class T>
struct AuxOps {
    const int *idx;
    const T *w;       // [k][m] row-scaled Poisson weights (sparse part of A)
    const T *dinv;    // [m] omega / l1 row norm
    const T *sinv;    // [m] 1 / row scale
    const int *rptr;  // [n*n + 1] restriction rows (interior lattice points)
    const int *rcol;  // node indices
    const T *rval;    // weights, summing to 1 per lattice point
    int64_t m;
    int k;
    // Weight of the second smoothing sweep of each pair relative to the
    // first (chosen at set-up from the spectrum of W A_s, see aux_weight).
    double w2 = 1.0;
};

// FGMRES scalars (device).  Basis vector V_j is stored unnormalised with
// its inverse norm vs[j]; every reader multiplies.
struct FgScal {
    double *vs;      // [mr+1] inverse norms
    double *part;    // [kFgMax + 2][kMaxBlocks] partial sums
    double *h1;      // [mr+1] Gram-Schmidt coefficients
    double *H;       // [(mr+1) * mr] Hessenberg matrix, column-major
    double *cs, *sn; // [mr] Givens rotations
    double *g;       // [mr+1] rotated right-hand side
    double *partZ;   // [kMaxBlocks] sums of J e (interpolated correction)
    double *partO;   // [kMaxBlocks] sums of z (border term of A z)
    double *one;     // [1] = 1.0 (unit scale of an explicit input vector)
    int *flag;
    double *stat;    // the cycle's target, ||b||^2
    // pinned host memory (fg_word): the word of the newest start or step, then
    // ||b||^2 and beta of the cycle
    uint64_t *pub;
};

// What the host follows a cycle by: the cycle's number, the residual estimate
// over its target (the upper half of a float), the steps done and the flag.  One
// 8-byte store, so it is read whole, without a copy or a synchronisation.
__device__ __forceinline__ uint64_t fg_word(uint32_t seq, double ratio, int step, int flag) {
    return (uint64_t)seq << 32 | (uint64_t)(__float_as_uint((float)ratio) & 0xffff0000u) |
           (uint32_t)(step & 0xff) << 8 | (uint32_t)(flag & 0xff);
}

template <class T>
struct FgDev {
    T *V;            // [(mr+1)][m]
    T *Z;            // [mr][m] preconditioned directions
    T *res, *t1;     // [m] preconditioner work
    T *x1, *z1;      // [m] smoothed vectors of the extra sweeps
    T *wd;           // [m] newest basis vector times the smoother diagonal W
    FgScal s;
};

// -------------------------------------------------------------- kernels --
// Row r of A_s applied to the values f(j) at the stencil columns; KT > 0
// fixes the width, its loads issued CH slots at a time (CH divides KT).
// Plain (temporal) loads: the Poisson operator (about 62 MB at h = 1/400)
// and the Krylov vectors of a cycle fit the 256 MB last-level cache
// together and are read several times per FGMRES step (non-temporal loads
// of the operator: 20 us per smoothing product, plain loads: 14.5 us).
template <int KT, int CH, class T, class F>
__device__ __forceinline__ T aux_row(const AuxOps<T> &P, int64_t r, F f) {
    T acc = 0;
    if constexpr (KT > 0) {
        static_assert(KT % CH == 0, "chunk must divide the stencil width");
#pragma unroll
        for (int q0 = 0; q0 < KT; q0 += CH) {
            int jj[CH];
            T ww[CH];
#pragma unroll
            for (int q = 0; q < CH; ++q) jj[q] = *(P.idx + (int64_t)(q0 + q) * P.m + r);
#pragma unroll
            for (int q = 0; q < CH; ++q) ww[q] = *(P.w + (int64_t)(q0 + q) * P.m + r);
#pragma unroll
            for (int q = 0; q < CH; ++q) acc = fma(ww[q], f(jj[q]), acc);
        }
    } else {
        for (int q = 0; q < P.k; ++q)
            acc = fma(P.w[(int64_t)q * P.m + r], f(P.idx[(int64_t)q * P.m + r]), acc);
    }
    return acc;
}

// Two lanes per row for the 28-entry stencils of the smoothing products:
// lanes l and l + 32 of a wave take the two halves of row l's stencil, so a
// launch has twice the waves (and loads in flight) of one lane per row.
constexpr int kRowsPerBlock2 = kThreads / 2;

// This lane's row in the two-lanes-per-row layout (one row pair per thread,
// no grid-stride loop) and the half of the stencil it takes.
__device__ __forceinline__ int64_t row2_of(int &half, uint32_t nb) {
    const int lane = threadIdx.x & 63;
    half = lane >> 5;
    return (int64_t)rbf::xcd_block(blockIdx.x, nb) * kRowsPerBlock2 +
           (threadIdx.x >> 6) * 32 + (lane & 31);
}

// One lane's half of row r of the sparse part: load() issues the entries' loads,
// sum(f) applies them to f and adds the pair's halves (0 + 1) in both lanes.
// Apart, so that whatever else a kernel needs, and the flag that may end it,
// travels with the entries in one memory round trip.
template <int KT, class T>
struct HalfRow {
    static_assert(KT > 0 && KT % 2 == 0, "two halves of a fixed stencil");
    static constexpr int H = KT / 2;
    int jj[H];
    T ww[H];
    __device__ __forceinline__ void load(const AuxOps<T> &P, int64_t r, int half) {
#pragma unroll
        for (int q = 0; q < H; ++q) jj[q] = P.idx[(int64_t)(half * H + q) * P.m + r];
#pragma unroll
        for (int q = 0; q < H; ++q) ww[q] = P.w[(int64_t)(half * H + q) * P.m + r];
    }
    template <class F>
    __device__ __forceinline__ T sum(F f) const {
        T acc = 0;
#pragma unroll
        for (int q = 0; q < H; ++q) acc = fma(ww[q], f(jj[q]), acc);
        return acc + __shfl_xor(acc, 32, 64);
    }
};

// Grid of the smoothing products: one row pair per thread for KT > 0, the
// grid-stride row loop otherwise.
template <int KT>
inline dim3 aux_grid(int64_t m, int nb) {
    return (KT > 0) ? dim3(rbf::blocks_for(m, kRowsPerBlock2)) : dim3(nb);
}

constexpr int kNormRow = kFgMax + 1;  // row of FgScal::part that takes ||w||^2

// Arnoldi step j, one workgroup: Hessenberg column j = h1 with
// H(j+1, j) = ||w||, previous rotations applied, a new rotation, the
// residual estimate |g_{j+1}| and the status (4: the cycle's target met or
// an exact breakdown; 3: the cycle is full; -1: non-finite).
// ||w||^2 is reduced here from the block partials of k_fg_gs (row kNormRow of
// part, nb blocks).  One wave per quarter of the partials, every load in one
// round trip; the column and the rotations are held one entry per lane of wave
// 0, which runs the recurrence on values read by lane.
__device__ __forceinline__ void fg_tail(const FgScal &F, int j, int mr, int nb, uint32_t seq) {
    const int t = threadIdx.x, lane = t & 63;
    const double *pn = F.part + (int64_t)kNormRow * kMaxBlocks;
    double pv[kMaxBlocks / 256];
#pragma unroll
    for (int q = 0; q < kMaxBlocks / 256; ++q) {
        const int b = t + 256 * q;
        pv[q] = (b < nb) ? pn[b] : 0.0;
    }
    const bool first = t < 64;
    const double hl = (first && lane <= j) ? F.h1[lane] : 0.0;
    const double cl = (first && lane < j) ? F.cs[lane] : 0.0;
    const double sl = (first && lane < j) ? F.sn[lane] : 0.0;
    const double gj = F.g[j], target = F.stat[0];
    if (*F.flag != 0) return;
    double v[1] = {(pv[0] + pv[1]) + (pv[2] + pv[3])};
    static_assert(kMaxBlocks == 4 * 256, "four partials per thread");
    __shared__ double lds[4];
    rbf::block_sum<1>(v, lds);
    if (!first) return;
    const double hn = sqrt(v[0]);
    double a = rbf::readlane_double(hl, 0), col = 0.0;
    for (int i = 0; i < j; ++i) {
        const double b = rbf::readlane_double(hl, i + 1), c = rbf::readlane_double(cl, i),
                     s = rbf::readlane_double(sl, i);
        if (lane == i) col = c * a + s * b;
        a = c * b - s * a;
    }
    const double den = hypot(a, hn);
    const double c = (den > 0.0) ? a / den : 1.0, s = (den > 0.0) ? hn / den : 0.0;
    if (lane == j) col = den;
    if (lane <= j + 1) F.H[(int64_t)j * (mr + 1) + lane] = (lane <= j) ? col : 0.0;
    if (lane != 0) return;
    const double res = fabs(s * gj);
    F.cs[j] = c;
    F.sn[j] = s;
    F.g[j] = c * gj;
    F.g[j + 1] = -s * gj;
    F.vs[j + 1] = (hn > 0.0) ? 1.0 / hn : 0.0;
    const int flag = (!isfinite(res) || !isfinite(den))              ? -1
                     : (res <= target || hn == 0.0 || den == 0.0) ? 4
                     : (j + 1 >= mr)                              ? 3
                                                                  : 0;
    if (flag != 0) F.flag[0] = flag;
    rbf::publish(F.pub, fg_word(seq, res / target, j + 1, flag));
}

__global__ void __launch_bounds__(256) k_fg_tail(FgScal F, int j, int mr, int nb, uint32_t seq) {
    fg_tail(F, j, mr, nb, seq);
}

// The tail of an Arnoldi step as work for the next kernel's last block (j < 0: none).
struct FgTail {
    FgScal F;
    int j, mr, nb;
    uint32_t seq;
};

// Pre-smoothing sweep from x = W y: x1 = yd + W (y - A_s yd) with yd = W y (one
// gathered value per neighbour), unscaled: the scale of y may still be in the
// making, by the last block's tail of the step before.  As a launch of its own
// the tail, one workgroup, takes 3.4 us of a step's 57 at h = 1/40.
template <int KT, class T>
__global__ void __launch_bounds__(kThreads) k_aux_pre(AuxOps<T> P, const T *__restrict__ y,
                                                       const T *__restrict__ yd, T *__restrict__ x1,
                                                       const int *flag, FgTail tail) {
    if constexpr (KT > 0) {
        const uint32_t nb = gridDim.x - (tail.j >= 0 ? 1 : 0);
        if (blockIdx.x == nb) {
            fg_tail(tail.F, tail.j, tail.mr, tail.nb, tail.seq);
            return;
        }
        int half;
        const int64_t r = row2_of(half, nb);
        const int64_t rr = (r < P.m) ? r : P.m - 1;
        HalfRow<KT, T> row;
        row.load(P, rr, half);
        const T yr = y[rr], ydr = yd[rr], di = P.dinv[rr];
        if (*flag != 0) return;
        const T ax = row.sum([&](int j) { return yd[j]; });
        if (half == 0 && r < P.m) x1[r] = ydr + (T)P.w2 * di * (yr - ax);
    } else {
        if (*flag != 0) return;
        for (int64_t it = 0;; ++it) {
            const int64_t r = row_of(it);
            if (r - threadIdx.x >= P.m) break;
            if (r < P.m) {
                const T ax = aux_row<KT, 1>(P, r, [&](int j) { return yd[j]; });
                x1[r] = yd[r] + (T)P.w2 * P.dinv[r] * (y[r] - ax);
            }
        }
    }
}

// Preconditioner stage 1: res = S^-1 (sc y - su A_s u) for the smoothed
// vector su u (u gathered once per neighbour; sc = *ys, su = *us).
template <int KT, class T>
__global__ void __launch_bounds__(kThreads) k_aux_res(AuxOps<T> P, const T *__restrict__ y,
                                                       const double *ys, const T *__restrict__ u,
                                                       const double *us, T *__restrict__ res,
                                                       const int *flag) {
    if constexpr (KT > 0) {
        int half;
        const int64_t r = row2_of(half, gridDim.x);
        const int64_t rr = (r < P.m) ? r : P.m - 1;
        HalfRow<KT, T> row;
        row.load(P, rr, half);
        const T sc = (T)*ys, su = (T)*us, yr = y[rr], si = P.sinv[rr];
        if (*flag != 0) return;
        const T ax = row.sum([&](int j) { return u[j]; });
        if (half == 0 && r < P.m) res[r] = si * (sc * yr - su * ax);
    } else {
        if (*flag != 0) return;
        const T sc = (T)*ys, su = (T)*us;
        for (int64_t it = 0;; ++it) {
            const int64_t r = row_of(it);
            if (r - threadIdx.x >= P.m) break;
            if (r < P.m) {
                const T ax = aux_row<KT, 1>(P, r, [&](int j) { return u[j]; });
                res[r] = P.sinv[r] * (sc * y[r] - su * ax);
            }
        }
    }
}

// Power iteration for the largest eigenvalue of W A_s, the smoother's
// operator (set-up only): y = W A_s (s x) and block partial sums of y^2;
// with s = 1 / ||x|| the norm of y estimates the eigenvalue.  ||x||^2 is summed by
// every block from the partials of the step before (null: s = s0), so that the
// steps follow each other without the host (whose sum cost a copy and a
// synchronisation each: solver set-up and first step at h = 1/100 10.0 -> 8.0 ms).  A vanishing or
// non-finite norm ends in NaN and stays.
template <int KT, class T>
__global__ void __launch_bounds__(kThreads) k_aux_power(AuxOps<T> P, const double *__restrict__ x,
                                                         const double *prev, double s0,
                                                         double *__restrict__ y, double *part) {
    double s = s0;
    if (prev) {
        double ss[1];
        load_partials<1>(prev, gridDim.x, ss);
        s = 1.0 / sqrt(ss[0]);
    }
    double acc[1] = {0.0};
    for (int64_t it = 0;; ++it) {
        const int64_t r = row_of(it);
        if (r - threadIdx.x >= P.m) break;
        if (r < P.m) {
            const double ax =
                (double)aux_row<KT, (KT > 0 ? KT : 1)>(P, r, [&](int j) { return (T)x[j]; });
            const double v = s * (double)P.dinv[r] * ax;
            y[r] = v;
            acc[0] += v * v;
        }
    }
    store_partials<1>(acc, part, gridDim.x);
}

// Start vector of the power iteration: a fixed hash pattern in [-1, 1).
__global__ void k_aux_power_start(int64_t m, double *__restrict__ x) {
    const int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (r >= m) return;
    const uint32_t hsh = (uint32_t)r * 2654435761u;
    x[r] = (double)(hsh >> 8) * (1.0 / 8388608.0) - 1.0;
}

// yd = W y for an explicit input vector.
template <class T>
__global__ void k_aux_scale(AuxOps<T> P, const T *__restrict__ y, T *__restrict__ yd) {
    for (int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; r < P.m;
         r += (int64_t)gridDim.x * blockDim.x)
        yd[r] = y[r] * P.dinv[r];
}

// Stage 2: restriction to the interior lattice points, X(q) = sum rval res
// (about five entries per point with one node spacing per cell): 4 lanes per
// point take every 4th entry, then combine in a fixed order.
template <class T>
__global__ void __launch_bounds__(256) k_aux_restrict(AuxOps<T> P, Lat L,
                                                       const T *__restrict__ res, int nq) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    const int q = t >> 2, sub = t & 3, qc = min(q, nq - 1);
    double g = 0.0;
    const int e0 = P.rptr[qc] + sub, e1 = P.rptr[qc + 1];
    if (*L.flag != 0) return;
    // Two entries of a lane at a time (a point has about five entries).
    for (int e = e0; e < e1; e += 8) {
        const int f = min(e + 4, e1 - 1);
        const int c0 = P.rcol[e], c1 = P.rcol[f];
        const double v0 = (double)P.rval[e], v1 = (double)P.rval[f];
        g += v0 * (double)res[c0];
        if (e + 4 < e1) g += v1 * (double)res[c1];
    }
    g += __shfl_xor(g, 1, 64);
    g += __shfl_xor(g, 2, 64);
    if (q < nq && sub == 0) lat_store(L, L.X, q, g);
}

// Lattice value of the transform solve (Z, column-major in X) at lattice
// node (i, j); wall nodes take their inward neighbour's value (homogeneous
// one-sided Neumann rows).
__device__ __forceinline__ double aux_lattice(const Lat &L, int i, int j) {
    const int ci = min(max(i, 1), L.K - 1), cj = min(max(j, 1), L.K - 1);
    return lat_load(L, L.X, (int64_t)(ci - 1) + (int64_t)(cj - 1) * L.n);
}

// Stage 3: t1 = su u + J e for the smoothed vector su u, and block sums of J e.
template <class T>
__global__ void __launch_bounds__(kThreads) k_aux_interp(AuxOps<T> P, Lat L,
                                                          const T *__restrict__ u,
                                                          const double *us, T *__restrict__ t1,
                                                          double *partZ) {
    const int K1 = L.K + 1;
    double acc[1] = {0.0};
    // The first row's data travel with the flag (every block has one).
    int64_t r = row_of(0);
    const int64_t rc = min(r, P.m - 1);
    int c = L.cell[rc];
    double fx = L.fx[rc], fy = L.fy[rc];
    T ur = u[rc];
    const T su = (T)*us;
    if (*L.flag != 0) return;
    for (int64_t it = 0;; ++it) {
        if (it > 0) {
            r = row_of(it);
            if (r - threadIdx.x >= P.m) break;
            if (r < P.m) {
                c = L.cell[r];
                fx = L.fx[r];
                fy = L.fy[r];
                ur = u[r];
            }
        }
        if (r < P.m) {
            const int i0 = c % K1, j0 = c / K1;
            const double z = (1.0 - fy) * ((1.0 - fx) * aux_lattice(L, i0, j0) +
                                           fx * aux_lattice(L, i0 + 1, j0)) +
                             fy * ((1.0 - fx) * aux_lattice(L, i0, j0 + 1) +
                                   fx * aux_lattice(L, i0 + 1, j0 + 1));
            t1[r] = su * ur + (T)z;
            acc[0] += z;
        }
    }
    store_partials<1>(acc, partZ, gridDim.x);
}

// Stage 4: z = t1 + mu + W (y - A_s t1) (MU: the border's constant mu is
// added; later sweeps add none); block sums of z (border term of the
// product that follows).  A_s mu = 0: the rows reproduce constants.
template <int KT, class T, bool MU>
__global__ void __launch_bounds__(kThreads) k_aux_post(AuxOps<T> P, Lat L,
                                                        const T *__restrict__ y, const double *ys,
                                                        const T *__restrict__ t1,
                                                        const double *partZ,
                                                        T *__restrict__ z, double *partO) {
    if (*L.flag != 0) return;
    double mu = 0.0;
    if constexpr (MU) {
        double sz[1];
        load_partials<1>(partZ, gridDim.x, sz);
        mu = (*L.mean / L.c - sz[0]) / (double)P.m;
    }
    const T sc = (T)*ys;
    double acc[1] = {0.0};
    for (int64_t it = 0;; ++it) {
        const int64_t r = row_of(it);
        if (r - threadIdx.x >= P.m) break;
        if (r < P.m) {
            const T at = aux_row<KT, (KT > 0 ? KT : 1)>(P, r, [&](int j) { return t1[j]; });
            const T zr = t1[r] + (T)mu + (MU ? (T)1 : (T)P.w2) * P.dinv[r] * (sc * y[r] - at);
            z[r] = zr;
            acc[0] += (double)zr;
        }
    }
    store_partials<1>(acc, partO, gridDim.x);
}

// The same sweep for 28-entry stencils with two lanes per row: blocks of
// 2 kThreads threads on the same grid and rows per block as k_aux_post, so
// the block sums of z keep their count.
template <class T, bool MU>
__global__ void __launch_bounds__(2 * kThreads) __attribute__((amdgpu_waves_per_eu(4)))
k_aux_post2(AuxOps<T> P, Lat L,
                                                           const T *__restrict__ y,
                                                           const double *ys,
                                                           const T *__restrict__ t1,
                                                           const double *partZ,
                                                           T *__restrict__ z, double *partO) {
    __shared__ double lds[2 * kThreads / 64];
    const int lane = threadIdx.x & 63, half = lane >> 5, wv = threadIdx.x >> 6;
    const int nb = gridDim.x;  // <= kMaxBlocks = 2 blockDim.x: two partials per thread
    // Everything that the first row iteration (every block has one) needs, the
    // partials of mu included, travels with the flag in one round trip; mu is
    // reduced while the gathers are in flight.
    const int64_t bx = rbf::xcd_block(blockIdx.x, nb);
    int64_t r = bx * kThreads + wv * 32 + (lane & 31);
    int64_t rr = (r < P.m) ? r : P.m - 1;
    HalfRow<28, T> row;
    row.load(P, rr, half);
    const double pz0 = (MU && (int)threadIdx.x < nb) ? partZ[threadIdx.x] : 0.0;
    const double pz1 =
        (MU && (int)threadIdx.x + 2 * kThreads < nb) ? partZ[threadIdx.x + 2 * kThreads] : 0.0;
    T tr = t1[rr], yr = y[rr], di = P.dinv[rr];
    const T sc = (T)*ys;
    const double mean = MU ? *L.mean : 0.0;
    if (*L.flag != 0) return;
    T at = row.sum([&](int j) { return t1[j]; });
    double mu = 0.0;
    if constexpr (MU) {
        double sz[1] = {pz0 + pz1};
        rbf::block_sum<1>(sz, lds);
        mu = (mean / L.c - sz[0]) / (double)P.m;
    }
    double acc[1] = {0.0};
#pragma unroll 1
    for (int64_t it = 0;; ++it) {
        if ((bx + it * nb) * kThreads >= P.m) break;
        if (it > 0) {
            r = (bx + it * nb) * kThreads + wv * 32 + (lane & 31);
            rr = (r < P.m) ? r : P.m - 1;
            row.load(P, rr, half);
            tr = t1[rr], yr = y[rr], di = P.dinv[rr];
            at = row.sum([&](int j) { return t1[j]; });
        }
        if (half == 0 && r < P.m) {
            const T zr = tr + (T)mu + (MU ? (T)1 : (T)P.w2) * di * (sc * yr - at);
            z[r] = zr;
            acc[0] += (double)zr;
        }
    }
    rbf::block_sum<1>(acc, lds);
    if (threadIdx.x == 0) partO[blockIdx.x] = acc[0];
}

// Cycle start: r = b - A x in FP64 (FP64 weights and border), V_0 = r and
// W V_0; block sums of ||r||^2 and ||b||^2 (rows 0 and 1 of part).
template <int KT, class T>
__global__ void __launch_bounds__(kThreads) k_fg_init(EllM A, const double *__restrict__ b,
                                                       const double *__restrict__ x,
                                                       const double *partX, T *__restrict__ V0,
                                                       const T *__restrict__ dinv,
                                                       T *__restrict__ wd, double *part) {
    const int nb = gridDim.x;
    double sx[1] = {0.0};
    if (A.u1) load_partials<1>(partX, nb, sx);
    double acc[2] = {0.0, 0.0};
    for (int64_t it = 0;; ++it) {
        const int64_t r = row_of(it);
        if (r - threadIdx.x >= A.n) break;
        if (r < A.n) {
            double ax[1][1] = {};
            const double *ws[1] = {A.w};
            rbf::ell_row<KT, 1>(A.idx, ws, A.n, r, A.k, GatherN<1>{x, A.n}, ax);
            const double u1 = A.u1 ? A.u1[r] * A.vscale : 0.0;
            const double rr = b[r] - (ax[0][0] + u1 * sx[0]);
            V0[r] = (T)rr;
            wd[r] = (T)rr * dinv[r];
            acc[0] += rr * rr;
            acc[1] += b[r] * b[r];
        }
    }
    double v0[1] = {acc[0]}, v1[1] = {acc[1]};
    store_partials<1>(v0, part, nb);
    store_partials<1>(v1, part + kMaxBlocks, nb);
}

// Reduce rows of nb block partials (row q at q * kMaxBlocks) into out[q]: one
// workgroup per row, a fixed order; exits when the flag is set.
__global__ void __launch_bounds__(256) k_fg_reduce(const double *part, int nb, double *out,
                                                   const int *flag) {
    if (*flag != 0) return;
    const int q = blockIdx.x;
    double v[1] = {0.0};
    for (int b = threadIdx.x; b < nb; b += 256) v[0] += part[(int64_t)q * kMaxBlocks + b];
    __shared__ double lds[4];
    rbf::block_sum<1>(v, lds);
    if (threadIdx.x == 0) out[q] = v[0];
}

// Cycle start, one workgroup: beta = ||r||, the cycle's target (FP64:
// tol ||b||; mixed: also kMixedInner beta), convergence of the true
// residual (flag 1), g = beta e_1.  ||r||^2 and ||b||^2 from the nb block partials
// of k_fg_init; ||b|| is taken from the first cycle.
__global__ void __launch_bounds__(256) k_fg_start(FgScal F, int nb, double tol, int mixed,
                                                   int first, uint32_t seq) {
    double v[2] = {0.0, 0.0};
#pragma unroll
    for (int q = 0; q < kMaxBlocks / 256; ++q) {
        const int at = threadIdx.x + 256 * q;
        v[0] += (at < nb) ? F.part[at] : 0.0;
        v[1] += (at < nb) ? F.part[kMaxBlocks + at] : 0.0;
    }
    const double bb0 = F.stat[1];
    __shared__ double lds[2 * 4];
    rbf::block_sum<2>(v, lds);
    if (threadIdx.x != 0) return;
    const double rr = v[0], bbv = first ? v[1] : bb0;
    const double beta = sqrt(rr);
    const double goal = tol * sqrt(fmax(bbv, 1e-300));
    F.stat[1] = bbv;
    int flag = 0;
    double target = 1.0;
    if (!isfinite(beta)) {
        flag = -1;
    } else if (beta <= goal || beta == 0.0) {
        flag = 1;
    } else {
        target = mixed ? fmax(goal, kMixedInner * beta) : goal;
        F.stat[0] = target;
        F.vs[0] = 1.0 / beta;
        F.g[0] = beta;
    }
    F.flag[0] = flag;
    rbf::publish(F.pub + 1, bbv);
    rbf::publish(F.pub + 2, beta);
    __hip_atomic_store(F.pub, fg_word(seq, beta / target, 0, flag), __ATOMIC_RELEASE,
                       __HIP_MEMORY_SCOPE_SYSTEM);
}

// Block partial dots (V_i vs_i, w) for i <= j, kFgChunk at a time; w is
// this thread's rows of the new vector (re-read per chunk).
template <class T>
__device__ __forceinline__ void fg_dots(const T *V, const double *vs, const T *w, int64_t m, int j,
                                        double *part) {
#pragma unroll 1
    for (int i0 = 0; i0 <= j; i0 += kFgChunk) {
        double acc[kFgChunk];
#pragma unroll
        for (int c = 0; c < kFgChunk; ++c) acc[c] = 0.0;
#pragma unroll 1
        for (int64_t it = 0;; ++it) {
            const int64_t r = row_of(it);
            if (r - threadIdx.x >= m) break;
            if (r < m) {
                const double wr = (double)w[r];
#pragma unroll
                for (int c = 0; c < kFgChunk; ++c)
                    if (i0 + c <= j) acc[c] += (double)V[(int64_t)(i0 + c) * m + r] * wr;
            }
        }
#pragma unroll
        for (int c = 0; c < kFgChunk; ++c) acc[c] *= (i0 + c <= j) ? vs[i0 + c] : 0.0;
        __shared__ double lds[kFgChunk * (kThreads / 64)];
        rbf::block_sum<kFgChunk>(acc, lds);
        if (threadIdx.x == 0)
            for (int c = 0; c < kFgChunk && i0 + c <= j; ++c)
                part[(int64_t)(i0 + c) * kMaxBlocks + blockIdx.x] = acc[c];
    }
}

// Arnoldi step j, product: w = A z_j (sparse part in T plus the border with
// sum z_j from partO; u1 must not be null), stored in V[j+1]; block partial
// dots (V_i vs_i, w).
template <int KT, class T>
__global__ void __launch_bounds__(kThreads) k_fg_av(AuxOps<T> P, const double *__restrict__ u1,
                                                     double vscale, FgDev<T> F, int j) {
    if (*F.s.flag != 0) return;
    double sz[1];
    load_partials<1>(F.s.partO, gridDim.x, sz);
    const double bterm = vscale * sz[0];  // border: u1 c (1^T z)
    const T *z = F.Z + (int64_t)j * P.m;
    T *w = F.V + (int64_t)(j + 1) * P.m;
#pragma unroll 1
    for (int64_t it = 0;; ++it) {
        const int64_t r = row_of(it);
        if (r - threadIdx.x >= P.m) break;
        if (r < P.m) {
            const T az = aux_row<KT, (KT > 0 ? KT : 1)>(P, r, [&](int c) { return z[c]; });
            w[r] = (T)((double)az + u1[r] * bterm);
        }
    }
    fg_dots(F.V, F.s.vs, w, P.m, j, F.s.part);
}

// The same step for 28-entry stencils with two lanes per row: blocks of
// 2 kThreads threads on the same grid (and the same kThreads rows per block
// and grid-stride iteration), so the partial sums keep their count; lanes l
// and l + 32 of a wave take the two halves of row l's stencil.  The dots are
// taken in the same pass over the rows: lane l + 32 h multiplies w by the
// basis vectors i = 2c + h (slot c), so that each vector is read once, and
// the slots are summed per half-wave by DPP, then over the waves in a fixed
// order.
constexpr int kAvThreads = 2 * kThreads;
constexpr int kFgSlots = (kFgMax + 1) / 2;  // basis vectors per half-wave

// Slot sums in LDS: column wv of lds (2 kFgSlots rows of NW) holds wave
// wv's running sums of the basis vectors i = 2c (half 0) and 2c + 1
// (half 1), owned by the wave's lane 0.  fg_slot_add adds one pass's
// products (half-wave sums by DPP; every lane must be active);
// fg_slot_partials sums the waves in a fixed order and writes the block
// partials of rows i <= j of part, scaled by vs_i (vsq: thread i's).
template <int NW>
__device__ __forceinline__ void fg_slot_zero(int ns, double *lds) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0)
        for (int i = 0; i < 2 * ns; ++i) lds[i * NW + wv] = 0.0;
}

template <int NW>
__device__ __forceinline__ void fg_slot_add(const double (&prod)[kFgSlots], int ns, double *lds) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int c = 0; c < kFgSlots; ++c) {
        if (c < ns) {
            double se, so;
            rbf::half_wave_sums(prod[c], se, so);
            if (lane == 0) {
                lds[(2 * c) * NW + wv] += se;
                lds[(2 * c + 1) * NW + wv] += so;
            }
        }
    }
}

template <int NW>
__device__ __forceinline__ void fg_slot_partials(int j, double vsq, double *part,
                                                 const double *lds) {
    __syncthreads();
    if ((int)threadIdx.x <= j) {
        const int q = threadIdx.x;
        double t = 0.0;
#pragma unroll
        for (int v = 0; v < NW; ++v) t += lds[q * NW + v];
        part[(int64_t)q * kMaxBlocks + blockIdx.x] = t * vsq;
    }
}

// EARLY: the basis values are loaded with the row's entries, before the product
// (for grids of at most one block per CU, where registers are not scarce).
template <class T, bool EARLY>
__device__ __forceinline__ void fg_av2_rows(const AuxOps<T> &P, const double *__restrict__ u1,
                                            double vscale, const FgDev<T> &F, int j) {
    constexpr int NW = kAvThreads / 64;
    __shared__ double lds[2 * kFgSlots * NW];
    const int lane = threadIdx.x & 63, half = lane >> 5, wv = threadIdx.x >> 6;
    const int nb = gridDim.x;  // <= kMaxBlocks = 2 blockDim.x: two partials per thread
    const T *z = F.Z + (int64_t)j * P.m;
    T *w = F.V + (int64_t)(j + 1) * P.m;
    const int ns = (j + 2) >> 1;
    // What the first row iteration (every block has one) needs, the partials of
    // 1^T z included, travels with the flag in one round trip; the border sum is
    // reduced while the gathers are in flight.
    const int64_t bx = rbf::xcd_block(blockIdx.x, nb);
    int64_t r = bx * kThreads + wv * 32 + (lane & 31);
    int64_t rr = (r < P.m) ? r : P.m - 1;
    HalfRow<28, T> row;
    row.load(P, rr, half);
    const double po0 = ((int)threadIdx.x < nb) ? F.s.partO[threadIdx.x] : 0.0;
    const double po1 =
        ((int)threadIdx.x + kAvThreads < nb) ? F.s.partO[threadIdx.x + kAvThreads] : 0.0;
    double ur = u1[rr];
    const double vsq = ((int)threadIdx.x <= j) ? F.s.vs[threadIdx.x] : 0.0;
    // Slot c of half 1 reads V[j+1] (this row of w, not yet stored) when
    // 2c + 1 > j; that value is not used.
    double vv[kFgSlots];
    auto basis = [&]() {
        const T *Vh = F.V + (int64_t)half * P.m + rr;
#pragma unroll
        for (int c = 0; c < kFgSlots; ++c)
            vv[c] = (c < ns) ? (double)Vh[(int64_t)(2 * c) * P.m] : 0.0;
    };
    if constexpr (EARLY) basis();
    if (*F.s.flag != 0) return;
    T az = row.sum([&](int c) { return z[c]; });
    double sz[1] = {po0 + po1};
    rbf::block_sum<1>(sz, lds);
    const double bterm = vscale * sz[0];  // border: u1 c (1^T z)
    fg_slot_zero<NW>(ns, lds);
#pragma unroll 1
    for (int64_t it = 0;; ++it) {
        if ((bx + it * nb) * kThreads >= P.m) break;
        if (it > 0) {
            r = (bx + it * nb) * kThreads + wv * 32 + (lane & 31);
            rr = (r < P.m) ? r : P.m - 1;
            row.load(P, rr, half);
            ur = u1[rr];
            az = row.sum([&](int c) { return z[c]; });
        }
        const T wt = (T)((double)az + ur * bterm);
        // Not EARLY: the basis is read after the product, so that the two sets
        // of loads in flight do not share the registers.
        if (!EARLY || it > 0) {
            __builtin_amdgcn_sched_barrier(0);
            basis();
        }
        const double wr = (r < P.m) ? (double)wt : 0.0;
        double prod[kFgSlots];
#pragma unroll
        for (int c = 0; c < kFgSlots; ++c) prod[c] = (c < ns && 2 * c + half <= j) ? vv[c] * wr : 0.0;
        if (half == 0 && r < P.m) w[r] = wt;
        fg_slot_add<NW>(prod, ns, lds);
    }
    fg_slot_partials<NW>(j, vsq, F.s.part, lds);
}

template <class T>
__global__ void __launch_bounds__(kAvThreads) __attribute__((amdgpu_waves_per_eu(4)))
k_fg_av2(AuxOps<T> P, const double *__restrict__ u1, double vscale, FgDev<T> F, int j) {
    fg_av2_rows<T, false>(P, u1, vscale, F, j);
}

template <class T>
__global__ void __launch_bounds__(kAvThreads) __attribute__((amdgpu_waves_per_eu(2)))
k_fg_av2_few(AuxOps<T> P, const double *__restrict__ u1, double vscale, FgDev<T> F, int j) {
    fg_av2_rows<T, true>(P, u1, vscale, F, j);
}

// Gram-Schmidt update w -= sum_i h_i vs_i V_i (i <= j), then block partial
// ||w||^2, and W w for the next preconditioner application.
// Blocks of 2 kThreads threads on the kThreads-rows grid: lanes l and l + 32
// of a wave share row l, each reading the basis vectors of one parity
// (slot c: i = 2c + h).
constexpr int kSumBlocks = 64;         // SUM: largest grid
template <class T, bool SUM>
__global__ void __launch_bounds__(2 * kThreads) __attribute__((amdgpu_waves_per_eu(4))) k_fg_gs(FgDev<T> F, const double *h,
                                                         const T *__restrict__ dinv, int64_t m,
                                                         int j) {
    constexpr int NW = 2 * kThreads / 64;
    __shared__ double c[kFgMax + 1];
    __shared__ double lds[NW];
    const int lane = threadIdx.x & 63, half = lane >> 5, wv = threadIdx.x >> 6;
    const int nb = gridDim.x;
    const int ns = (j + 2) >> 1;
    const int64_t bx = rbf::xcd_block(blockIdx.x, nb);
    T *w = F.V + (int64_t)(j + 1) * m;
    double nrm[1] = {0.0};
    int64_t r, rr;
    double vv[kFgSlots], wr;
    T di;
    auto rows = [&](int64_t it) {
        r = (bx + it * nb) * kThreads + wv * 32 + (lane & 31);
        rr = (r < m) ? r : m - 1;
        // Slot q of half 1 reads V[j+1] = w when 2q + 1 > j (not used).
        const T *Vh = F.V + (int64_t)half * m + rr;
#pragma unroll
        for (int q = 0; q < kFgSlots; ++q) vv[q] = (q < ns) ? (double)Vh[(int64_t)(2 * q) * m] : 0.0;
        wr = (double)w[rr];
        di = dinv[rr];
    };
    // The first row iteration's loads, the coefficients and the flag in one
    // round trip.  SUM: the coefficients are summed here from the block partials
    // of the dots, 16 lanes each (grids of at most kSumBlocks blocks: one launch
    // less per step); block 0 stores them for k_fg_tail.
    rows(0);
    const int q16 = threadIdx.x >> 4, l16 = threadIdx.x & 15;
    double hs = 0.0, vsq = 0.0;
    if constexpr (SUM) {
        double pt[kSumBlocks / 16];
#pragma unroll
        for (int b = 0; b < kSumBlocks / 16; ++b) {
            const int at = l16 + 16 * b;
            pt[b] = (q16 <= j && at < nb) ? F.s.part[(int64_t)q16 * kMaxBlocks + at] : 0.0;
        }
#pragma unroll
        for (int b = 0; b < kSumBlocks / 16; ++b) hs += pt[b];
        vsq = (q16 <= j) ? F.s.vs[q16] : 0.0;
    } else if ((int)threadIdx.x <= j) {
        hs = h[threadIdx.x];
        vsq = F.s.vs[threadIdx.x];
    }
    if (*F.s.flag != 0) return;
    if constexpr (SUM) {
        hs += rbf::dpp_move<0x128>(hs);
        hs += rbf::dpp_move<0x124>(hs);
        hs += rbf::dpp_move<0x4E>(hs);
        hs += rbf::dpp_move<0xB1>(hs);
        if (l16 == 0 && q16 <= j) {
            c[q16] = hs * vsq;
            if (blockIdx.x == 0) F.s.h1[q16] = hs;
        }
    } else if ((int)threadIdx.x <= j) {
        c[threadIdx.x] = hs * vsq;
    }
    __syncthreads();
#pragma unroll 1
    for (int64_t it = 0;; ++it) {
        if ((bx + it * nb) * kThreads >= m) break;
        if (it > 0) rows(it);
        double s = 0.0;
#pragma unroll
        for (int q = 0; q < kFgSlots; ++q)
            if (q < ns && 2 * q + half <= j) s += c[2 * q + half] * vv[q];
        s += __shfl_xor(s, 32, 64);
        const T wt = (T)(wr - s);
        if (half == 0 && r < m) {
            w[r] = wt;
            F.wd[r] = wt * di;
            nrm[0] += (double)wt * (double)wt;
        }
    }
    // Row kNormRow: the partials of the dots (row 0 on) may still be read.
    rbf::block_sum<1>(nrm, lds);
    if (threadIdx.x == 0) F.s.part[(int64_t)kNormRow * kMaxBlocks + blockIdx.x] = nrm[0];
}

// End of a cycle of nstep steps: back substitution H y = g and x += sum_i y_i Z_i
// (FP64 iterate), with block sums of the new x (weighted by sumw unless null) for
// the next cycle's border term.  The substitution is done by the first wave of
// every block, one unknown per lane, while the rows' Z are on their way: as a
// launch of its own, one thread's chain of 30 divisions, it took 9.7 us, the
// update 6.2 and the sum 2.5; 7.2 us for the three at h = 1/40.
template <class T>
__global__ void __launch_bounds__(kThreads) k_fg_x(FgScal F, const T *__restrict__ Z, int nstep,
                                                    int mr, int64_t m, double *__restrict__ x,
                                                    const double *__restrict__ sumw, double *partX) {
    __shared__ double ys[kFgMax];
    double zv[kFgMax], xv, wv = 1.0;
    auto load = [&](int64_t r) {
#pragma unroll
        for (int i = 0; i < kFgMax; ++i) zv[i] = (i < nstep) ? (double)Z[(int64_t)i * m + r] : 0.0;
        xv = x[r];
        if (sumw) wv = sumw[r];
    };
    load(min(row_of(0), m - 1));
    if (threadIdx.x < 64) {
        const int lane = threadIdx.x;
        double h[kFgMax];
#pragma unroll
        for (int l = 0; l < kFgMax; ++l)
            h[l] = (l < nstep && lane <= l) ? F.H[(int64_t)l * (mr + 1) + lane] : 0.0;
        double g = (lane < nstep) ? F.g[lane] : 0.0, y = 0.0;
        const double d = (lane < nstep) ? F.H[(int64_t)lane * (mr + 1) + lane] : 1.0;
        const double inv = (d != 0.0) ? 1.0 / d : 0.0;
#pragma unroll
        for (int l = kFgMax - 1; l >= 0; --l) {
            if (l >= nstep) continue;
            const double gl = rbf::readlane_double(g, l), il = rbf::readlane_double(inv, l),
                         dl = rbf::readlane_double(d, l);
            const double y0 = gl * il, yl = fma(fma(-y0, dl, gl), il, y0);  // g / d, corrected
            if (lane == l) y = yl;
            g = fma(-h[l], yl, g);
        }
        if (lane < kFgMax) ys[lane] = y;
    }
    __syncthreads();
    double acc[1] = {0.0};
    for (int64_t it = 0;; ++it) {
        const int64_t r = row_of(it);
        if (r - threadIdx.x >= m) break;
        if (it > 0) load(min(r, m - 1));
        if (r < m) {
            double s = xv;
#pragma unroll
            for (int i = 0; i < kFgMax; ++i)
                if (i < nstep) s += ys[i] * zv[i];
            x[r] = s;
            acc[0] += wv * s;
        }
    }
    store_partials<1>(acc, partX, gridDim.x);
}

// l1 row norms of the stored Poisson rows: dinv = omega / sum |w|, and
// 1 / row scale.
__global__ void k_aux_rows(int64_t m, int k, const double *__restrict__ w,
                           const double *__restrict__ rs, double *dinv, double *sinv) {
    const int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (r >= m) return;
    double s = 0.0;
    for (int q = 0; q < k; ++q) s += fabs(w[(int64_t)q * m + r]);
    dinv[r] = (s > 0.0) ? kAuxOmega / s : 0.0;
    sinv[r] = 1.0 / rs[r];
}

// FP32 copies for the mixed-precision cycles.
__global__ void k_aux_to_f32(int64_t n, const double *__restrict__ a, float *__restrict__ b) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        b[i] = (float)a[i];
}
