// Reverse-mode derivative of one step of Sec. 3 (eqs. (14)-(21)), kernels.
// Included by solver.hip inside its anonymous namespace.
//
// The adjoint of the step transposes its stages in reverse order (u_bar:
// adjoint of u, and so on; chi: interior indicator; G = D^VP, D = D^PV):
//   u**_bar = u_{j+1}_bar,  p~_bar -= dt (Gx^T u_bar + Gy^T v_bar)      (20)
//   rhs_bar = S w, (A_s + u1 c 1^T)^T w = p~_bar - mean(p~_bar)         (18)
//   F_bar = chi_P rhs_bar / dt,  u**_bar += Dx^T F_bar, v likewise      (17)
//   r_bar = H^-T u**_bar (both components)                              (16)
//   nu_bar += dt/2 sum chi r_bar o L (u* + u**)   (H and (I + aL) in nu)
//   u*_bar = chi r_bar + a L^T (chi r_bar);  u_bc_bar += (1 - chi) r_bar;
//   p~_j_bar = dt (Gx^T ((1 - chi) r_u_bar) + Gy^T ((1 - chi) r_v_bar)) (21)
//   C_j_bar = 3/2 dt u*_bar + (C_j as the next step's C_{j-1})_bar,
//   C_{j-1}_bar = -1/2 dt u*_bar (folded into C_j_bar at j = 0)         (14)
//   u_j_bar = u*_bar - Dx u o Cu_bar - Dx^T(u o Cu_bar) - Dy^T(v o Cu_bar)
//             - Dx v o Cv_bar, v_j_bar likewise                         (15)
// Here S is the row scale of the stored Poisson rows A_s = S A0 and
// u1 = S chi: the transpose of the zero-mean bordered solve of the forward
// step is a solve with (A_s + u1 c 1^T)^T followed by the row scale.
#pragma once

// out = alpha a + beta b (elementwise; b may alias out).
__global__ void k_adj_axpby(int64_t n, double alpha, const double *__restrict__ a, double beta,
                            const double *b, double *out) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        out[i] = alpha * a[i] + beta * b[i];
}

// Split r by the V-node tags: ri = chi r (interior), rw = (1 - chi) r.
__global__ void k_adj_split(int64_t n, const int8_t *__restrict__ tag, const double *__restrict__ r,
                            double *ri, double *rw) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const bool wall = tag[i] != 0;
        ri[i] = wall ? 0.0 : r[i];
        rw[i] = wall ? r[i] : 0.0;
    }
}

// out = a o b (elementwise product).
__global__ void k_adj_mul(int64_t n, const double *__restrict__ a, const double *__restrict__ b,
                          double *out) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        out[i] = a[i] * b[i];
}

// F_bar = chi_P s o w / dt (row scale s, interior P rows only).
__global__ void k_adj_fbar(int64_t m, const int8_t *__restrict__ ptag, const double *__restrict__ s,
                           const double *__restrict__ w, double inv_dt, double *fb) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < m;
         i += (int64_t)gridDim.x * blockDim.x)
        fb[i] = (ptag[i] == 0) ? s[i] * w[i] * inv_dt : 0.0;
}

// Advection adjoint, pointwise part: with cu_b, cv_b the adjoints of C_j,
//   ub -= (Dx u) cu_b + (Dx v) cv_b,  vb -= (Dy u) cu_b + (Dy v) cv_b,
// and the gather inputs of the transposed products
//   qx = u cu_b, qy = v cu_b (for u_bar), px = u cv_b, py = v cv_b (for v_bar).
__global__ void k_adj_adv(int64_t n, const double *__restrict__ u, const double *__restrict__ v,
                          const double *__restrict__ dxu, const double *__restrict__ dyu,
                          const double *__restrict__ dxv, const double *__restrict__ dyv,
                          const double *__restrict__ cub, const double *__restrict__ cvb,
                          double *ub, double *vb, double *qx, double *qy, double *px, double *py) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const double a = cub[i], b = cvb[i];
        ub[i] -= dxu[i] * a + dxv[i] * b;
        vb[i] -= dyu[i] * a + dyv[i] * b;
        qx[i] = u[i] * a;
        qy[i] = v[i] * a;
        px[i] = u[i] * b;
        py[i] = v[i] * b;
    }
}

// Up to four dot products (x_q, y_q), or sums when y_q is null.
struct AdjDots {
    const double *x[4];
    const double *y[4];
};

// Block partial sums of NQ dot products of d (row q at q * kMaxBlocks).
template <int NQ>
__global__ void __launch_bounds__(kThreads) k_adj_dots(int64_t n, AdjDots d, double *part) {
    double acc[NQ] = {};
    for (int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kThreads) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) acc[q] += d.x[q][i] * (d.y[q] ? d.y[q][i] : 1.0);
    }
    __shared__ double lds[NQ * (kThreads / 64)];
    rbf::block_sum<NQ>(acc, lds);
    if (threadIdx.x == 0)
        for (int q = 0; q < NQ; ++q) part[(int64_t)q * kMaxBlocks + blockIdx.x] = acc[q];
}

// z += c (elementwise constant).
__global__ void k_adj_addc(int64_t n, double c, double *z) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        z[i] += c;
}

// tag[r] = 1 for the wall rows in list (the array is zero beforehand).
__global__ void k_adj_wallmask(int64_t nwall, const int *__restrict__ list, int8_t *tag) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < nwall) tag[list[i]] = 1;
}

// ------------------------------------ transposed pressure preconditioner --
// B^-T of the auxiliary-lattice preconditioner (pressure_aux.h), the right
// preconditioner of flexible GMRES on A^T = A_s^T + c 1 u1^T.  With the smoother
// pair S = W + w2 W (I - A_s W), the transposed application is, last stage first,
//   v1 = v - w2 A_s^T W v
//   v2 = v1 - A_s^T W v1
//   h  = J^T (v2 - mean v2),  e = (L5)^+ h,
//   q  = S_r^-1 R^T (e + sum v2 / (m c n^2))   (S_r the row scale; the constant
//                                              is the transpose of mu)
//   u  = v2 - A_s^T q
//   z  = w2 W v + W v1 + q + W u + w2 W (u - A_s^T W u):
// four products, as the forward application takes, and the same transforms.
// A_s^T is stored as rows padded to a common length (a multiple of kAtChunk)
// with zero weights on the row itself, so that a row's loads are independent.
constexpr int kAtChunk = 8;
constexpr int kAtMax = 256;  // longest padded row (longer columns: BiCGSTAB)

struct AdjPre {
    AuxOps<double> P;            // padded A_s^T with W, S_r^-1 and w2
    const int *jptr, *jcol;      // J^T: rows of the interior lattice points (X order)
    const double *jval;
    const int *tq;               // R^T: [4][m] lattice entries (Z order), weight 0 if unused
    const double *tv;            // [4][m]
    const double *u1;            // [m] border column
    double *v1, *g1, *v2, *q, *u, *gu;  // [m] work
    double *partS, *sum;         // sums of v2: block partials, total
};

// CSR columns of a transposed ELL operator as rows padded to kt entries.
__global__ void k_at_pad(int64_t n, int kt, const int64_t *__restrict__ colptr,
                         const int *__restrict__ src, const double *__restrict__ wt,
                         int *__restrict__ idx, double *__restrict__ w) {
    const int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (c >= n) return;
    const int64_t b = colptr[c], len = colptr[c + 1] - b;
    for (int s = 0; s < kt; ++s) {
        idx[(int64_t)s * n + c] = (s < len) ? src[b + s] : (int)c;
        w[(int64_t)s * n + c] = (s < len) ? wt[b + s] : 0.0;
    }
}

// Row r of the padded operator applied to x.
__device__ __forceinline__ double at_row(const AuxOps<double> &P, int64_t r, const double *x) {
    double acc = 0.0;
    for (int q0 = 0; q0 < P.k; q0 += kAtChunk) {
        int jj[kAtChunk];
        double ww[kAtChunk];
#pragma unroll
        for (int q = 0; q < kAtChunk; ++q) jj[q] = P.idx[(int64_t)(q0 + q) * P.m + r];
#pragma unroll
        for (int q = 0; q < kAtChunk; ++q) ww[q] = P.w[(int64_t)(q0 + q) * P.m + r];
#pragma unroll
        for (int q = 0; q < kAtChunk; ++q) acc = fma(ww[q], x[jj[q]], acc);
    }
    return acc;
}

// The four products (STAGE 1..4 as v1, v2, u, z above); STAGE 2 sums v2,
// STAGE 4 u1 z (border term of the product that follows), per block.
template <int STAGE>
__global__ void __launch_bounds__(kThreads) k_at_row(AdjPre D, const double *__restrict__ y,
                                                      const double *__restrict__ yd,
                                                      const double *ys, double *__restrict__ z,
                                                      double *part, const int *flag) {
    if (*flag != 0) return;
    const AuxOps<double> &P = D.P;
    const double sc = (STAGE == 1 || STAGE == 4) ? *ys : 0.0;
    double acc[1] = {0.0};
    for (int64_t it = 0;; ++it) {
        const int64_t r = row_of(it);
        if (r - threadIdx.x >= P.m) break;
        if (r >= P.m) continue;
        if constexpr (STAGE == 1) {
            const double v = sc * (y[r] - P.w2 * at_row(P, r, yd));
            D.v1[r] = v;
            D.g1[r] = P.dinv[r] * v;
        } else if constexpr (STAGE == 2) {
            const double v = D.v1[r] - at_row(P, r, D.g1);
            D.v2[r] = v;
            acc[0] += v;
        } else if constexpr (STAGE == 3) {
            const double v = D.v2[r] - at_row(P, r, D.q);
            D.u[r] = v;
            D.gu[r] = P.dinv[r] * v;
        } else {
            const double u = D.u[r];
            const double v = D.q[r] + P.dinv[r] * (P.w2 * sc * y[r] + D.v1[r] + u +
                                                   P.w2 * (u - at_row(P, r, D.gu)));
            z[r] = v;
            acc[0] += D.u1[r] * v;
        }
    }
    if constexpr (STAGE == 2 || STAGE == 4) store_partials<1>(acc, part, gridDim.x);
}

// h = J^T (v2 - mean v2), four lanes per lattice point.
__global__ void __launch_bounds__(kThreads) k_at_restrict(AdjPre D, Lat L, int nbS) {
    if (*L.flag != 0) return;
    double s[1];
    load_partials<1>(D.partS, nbS, s);
    const double mean = s[0] / (double)D.P.m;
    if (blockIdx.x == 0 && threadIdx.x == 0) *D.sum = s[0];
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    const int q = t >> 2, sub = t & 3, nq = L.n * L.n;
    double g = 0.0;
    if (q < nq) {
        const int e1 = D.jptr[q + 1];
        for (int e = D.jptr[q] + sub; e < e1; e += 4) g += D.jval[e] * (D.v2[D.jcol[e]] - mean);
    }
    g += __shfl_xor(g, 1, 64);
    g += __shfl_xor(g, 2, 64);
    if (q < nq && sub == 0) lat_store(L, L.X, q, g);
}

// q = S_r^-1 R^T (e + sum v2 / (m c n^2)).
__global__ void __launch_bounds__(kThreads) k_at_prolong(AdjPre D, Lat L) {
    if (*L.flag != 0) return;
    const int64_t m = D.P.m;
    const double add = *D.sum / ((double)m * L.c * (double)L.n * (double)L.n);
    for (int64_t r = blockIdx.x * (int64_t)kThreads + threadIdx.x; r < m;
         r += (int64_t)gridDim.x * kThreads) {
        double v = 0.0;
#pragma unroll
        for (int c = 0; c < 4; ++c)
            v += D.tv[c * m + r] * (lat_load(L, L.X, D.tq[c * m + r]) + add);
        D.q[r] = D.P.sinv[r] * v;
    }
}

// Block sums of w x (weighted form of k_sum).
__global__ void __launch_bounds__(kThreads) k_wsum(int64_t n, const double *__restrict__ w,
                                                    const double *__restrict__ x, double *part) {
    double acc[1] = {0.0};
    for (int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kThreads)
        acc[0] += w[i] * x[i];
    store_partials<1>(acc, part, gridDim.x);
}

// a[i] = c (elementwise constant).
__global__ void k_adj_fill(int64_t n, double c, double *a) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        a[i] = c;
}
