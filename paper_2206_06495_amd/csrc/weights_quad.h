// Weights of the paper's stencil (n = 28 nodes, r^7, cubic polynomials): four
// systems per wavefront, 16 lanes each, by the null-space method.  Included
// by weights.hip inside its anonymous namespace.
//
// System of eq. (9): [A P; P^T 0] [w; c] = [f; g].  r^7 is conditionally
// positive definite of order 4, so A is positive definite on the null space
// of P^T (cubics and below), and no pivoting is needed there:
//   1. ten nodes B on which P is well conditioned are chosen by elimination of
//      P with row pivoting (in FP32: it only orders the nodes) and the nodes
//      renumbered, B first;
//   2. P_B = L U, M = P_N P_B^-1 (18 x 10), null-space basis Z = [-M^T; I];
//   3. K = Z^T A Z = A_NN - M A_BN - (A_NB - M A_BB) M^T (18 x 18), K = L D L^T;
//   4. w = w0 + Z y: P_B^T w0 = g, K y = Z^T (f - A w0); P_B c = (f - A w)_B;
//   5. one refinement step: the residual of the whole saddle-point system in
//      exact sums (below), then step 4 for the correction.
// Against block elimination with A first (k_weights_pair) this halves the
// arithmetic, and every product that another lane's value enters is one
// v_fmac_f64 whose first operand is broadcast inside the 16-lane row by DPP
// (row_newbcast), without LDS or readlane.
//
// Lanes and rows: after the renumbering, slot 0 of lanes 0..9 holds the rows
// of B, slot 0 of lanes 10 and 11 the first two rows of N, slot 1 of lane l
// row 12 + l.  Rows 10 and 11 are eliminated first, so that the rest of the
// factorisation runs in slot 1 with all 16 lanes.  K stays symmetric during
// the elimination: column s of the lanes below is also row s, and lane s keeps
// the entries of its own row beyond the diagonal for the back substitution.
//
// A is computed once per pair of nodes into LDS (packed, 3 KB per system) and
// read back by rows, for the residual too.
//
// Residual: w and c are cut to 30 bits and every factor a is split into two
// parts of 18 bits and the rest, each on one grid for the whole row, so that 28
// products of a part with w sum within 53 bits: the FMAs of the first two sums
// are exact, and the third is 2^-36 of the result.  That is as good as a
// double-FP64 sum at 3 FMAs per product instead of 10 operations: the rms error
// of the weights against the same system in extended precision is that of
// k_weights_pair to four digits (1.5e-16 of a row's largest weight for D_x of the
// V-nodes at h = 1/400).  A two-part split with 24 bits each left up to 1.9 times
// that error.
//
// Measured (10^6 V-nodes, D_x, D_y, Lap): 5.1 ms against 18.3 ms of
// k_weights_pair.  Bound by the FP64 instructions at two waves a SIMD (256
// VGPRs): 7,212 vector instructions per wavefront of four systems (4,068 per
// system before), which keep the vector unit busy 62 % of the time; the rest is
// the latency of the factorisation's chain.
//
// A system that is not clearly definite on these pivots (coincident nodes,
// nodes on a cubic curve, non-finite coordinates, an index out of range) is
// left to the pivoted kernels: its first weight is set to NaN, and *todo to 1.

constexpr int kQuadTri = kPairN * (kPairN - 1) / 2;  // 378 pairs of nodes

struct QuadLds {
    double a[kQuadTri + 6];  // A, strictly lower triangle, row by row (+ 6: the last round's idle lanes)
    double2 c[kPairN];       // scaled coordinates in the new order
    double t[18 * kPairKP];  // pivot rows; M; P of one slot
    int node[kPairN];        // stencil slot of a position
};

// Pair e of the strictly lower triangle: i << 8 | j, i > j.
struct QuadPairs {
    uint16_t v[kQuadTri + 6];
    constexpr QuadPairs() : v() {
        int e = 0;
        for (int i = 1; i < kPairN; ++i)
            for (int j = 0; j < i; ++j) v[e++] = (uint16_t)(i << 8 | j);
        for (; e < kQuadTri + 6; ++e) v[e] = (uint16_t)(1 << 8);
    }
};
__constant__ QuadPairs kPairs = QuadPairs();

template <class F, int... I>
__device__ __forceinline__ void static_for_impl(F &&f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
// f(0), ..., f(N - 1) with compile-time indices.
template <int N, class F>
__device__ __forceinline__ void static_for(F &&f) {
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}
#define QUAD_FN(...) [&](__VA_ARGS__) __attribute__((always_inline))

// Value of lane L of each 16-lane row.
template <int L>
__device__ __forceinline__ double row_bcast(double v) {
    return __longlong_as_double(
        __builtin_amdgcn_update_dpp(0ll, __double_as_longlong(v), 0x150 + L, 0xF, 0xF, true));
}

// Fused multiply-adds with a row broadcast as first factor, in groups behind
// one s_nop (a DPP operand may not have been written by the two instructions
// before it; the compiler does not look into the groups).  Every lane must be
// active.
#define QUAD_FMAC(d, s, m, l) \
    "v_fmac_f64_dpp %" #d ", %" #s ", %" #m " row_newbcast:%" #l " row_mask:0xf bank_mask:0xf\n\t"

// d[i] += bcast(s, L0 + i) * m for i < N.
template <int L0, int N>
__device__ __forceinline__ void fmac_lanes(double *d, double s, double m) {
    if constexpr (N >= 8) {
        asm("s_nop 1\n\t" QUAD_FMAC(0, 8, 9, 10) QUAD_FMAC(1, 8, 9, 11) QUAD_FMAC(2, 8, 9, 12)
                QUAD_FMAC(3, 8, 9, 13) QUAD_FMAC(4, 8, 9, 14) QUAD_FMAC(5, 8, 9, 15)
                    QUAD_FMAC(6, 8, 9, 16) QUAD_FMAC(7, 8, 9, 17)
            : "+&v"(d[0]), "+&v"(d[1]), "+&v"(d[2]), "+&v"(d[3]), "+&v"(d[4]), "+&v"(d[5]),
              "+&v"(d[6]), "+&v"(d[7])
            : "v"(s), "v"(m), "n"(L0), "n"(L0 + 1), "n"(L0 + 2), "n"(L0 + 3), "n"(L0 + 4),
              "n"(L0 + 5), "n"(L0 + 6), "n"(L0 + 7));
        fmac_lanes<L0 + 8, N - 8>(d + 8, s, m);
    } else if constexpr (N >= 4) {
        asm("s_nop 1\n\t" QUAD_FMAC(0, 4, 5, 6) QUAD_FMAC(1, 4, 5, 7) QUAD_FMAC(2, 4, 5, 8)
                QUAD_FMAC(3, 4, 5, 9)
            : "+&v"(d[0]), "+&v"(d[1]), "+&v"(d[2]), "+&v"(d[3])
            : "v"(s), "v"(m), "n"(L0), "n"(L0 + 1), "n"(L0 + 2), "n"(L0 + 3));
        fmac_lanes<L0 + 4, N - 4>(d + 4, s, m);
    } else if constexpr (N >= 2) {
        asm("s_nop 1\n\t" QUAD_FMAC(0, 2, 3, 4) QUAD_FMAC(1, 2, 3, 5)
            : "+&v"(d[0]), "+&v"(d[1])
            : "v"(s), "v"(m), "n"(L0), "n"(L0 + 1));
        fmac_lanes<L0 + 2, N - 2>(d + 2, s, m);
    } else if constexpr (N == 1) {
        asm("s_nop 1\n\t" QUAD_FMAC(0, 1, 2, 3) : "+&v"(d[0]) : "v"(s), "v"(m), "n"(L0));
    }
}

// d[i] += bcast(s[i], L) * m for i < N; d and s distinct.
template <int L, int N>
__device__ __forceinline__ void fmac_lane(double *d, const double *s, double m) {
    if constexpr (N >= 5) {
        asm("s_nop 1\n\t" QUAD_FMAC(0, 5, 10, 11) QUAD_FMAC(1, 6, 10, 11) QUAD_FMAC(2, 7, 10, 11)
                QUAD_FMAC(3, 8, 10, 11) QUAD_FMAC(4, 9, 10, 11)
            : "+&v"(d[0]), "+&v"(d[1]), "+&v"(d[2]), "+&v"(d[3]), "+&v"(d[4])
            : "v"(s[0]), "v"(s[1]), "v"(s[2]), "v"(s[3]), "v"(s[4]), "v"(m), "n"(L));
        fmac_lane<L, N - 5>(d + 5, s + 5, m);
    } else if constexpr (N >= 3) {
        asm("s_nop 1\n\t" QUAD_FMAC(0, 3, 6, 7) QUAD_FMAC(1, 4, 6, 7) QUAD_FMAC(2, 5, 6, 7)
            : "+&v"(d[0]), "+&v"(d[1]), "+&v"(d[2])
            : "v"(s[0]), "v"(s[1]), "v"(s[2]), "v"(m), "n"(L));
        fmac_lane<L, N - 3>(d + 3, s + 3, m);
    } else if constexpr (N == 2) {
        asm("s_nop 1\n\t" QUAD_FMAC(0, 2, 4, 5) QUAD_FMAC(1, 3, 4, 5)
            : "+&v"(d[0]), "+&v"(d[1])
            : "v"(s[0]), "v"(s[1]), "v"(m), "n"(L));
    } else if constexpr (N == 1) {
        asm("s_nop 1\n\t" QUAD_FMAC(0, 1, 2, 3) : "+&v"(d[0]) : "v"(s[0]), "v"(m), "n"(L));
    }
}

// d[i] += bcast(d[i], L) * m for i < N (m = 0 in lane L).
template <int L, int N>
__device__ __forceinline__ void fmac_self(double *d, double m) {
    if constexpr (N >= 5) {
        asm("s_nop 1\n\t" QUAD_FMAC(0, 0, 5, 6) QUAD_FMAC(1, 1, 5, 6) QUAD_FMAC(2, 2, 5, 6)
                QUAD_FMAC(3, 3, 5, 6) QUAD_FMAC(4, 4, 5, 6)
            : "+&v"(d[0]), "+&v"(d[1]), "+&v"(d[2]), "+&v"(d[3]), "+&v"(d[4])
            : "v"(m), "n"(L));
        fmac_self<L, N - 5>(d + 5, m);
    } else if constexpr (N >= 3) {
        asm("s_nop 1\n\t" QUAD_FMAC(0, 0, 3, 4) QUAD_FMAC(1, 1, 3, 4) QUAD_FMAC(2, 2, 3, 4)
            : "+&v"(d[0]), "+&v"(d[1]), "+&v"(d[2])
            : "v"(m), "n"(L));
        fmac_self<L, N - 3>(d + 3, m);
    } else if constexpr (N == 2) {
        asm("s_nop 1\n\t" QUAD_FMAC(0, 0, 2, 3) QUAD_FMAC(1, 1, 2, 3)
            : "+&v"(d[0]), "+&v"(d[1])
            : "v"(m), "n"(L));
    } else if constexpr (N == 1) {
        asm("s_nop 1\n\t" QUAD_FMAC(0, 0, 1, 2) : "+&v"(d[0]) : "v"(m), "n"(L));
    }
}
// s_q[i] += bcast(x[i], L) * a_q for the three parts q of a split factor, i < N.
template <int L, int N>
__device__ __forceinline__ void fmac_split(double *s1, double *s2, double *s3, const double *x,
                                           double a1, double a2, double a3) {
    if constexpr (N == 3)
        asm("s_nop 1\n\t" QUAD_FMAC(0, 9, 12, 15) QUAD_FMAC(1, 10, 12, 15) QUAD_FMAC(2, 11, 12, 15)
                QUAD_FMAC(3, 9, 13, 15) QUAD_FMAC(4, 10, 13, 15) QUAD_FMAC(5, 11, 13, 15)
                    QUAD_FMAC(6, 9, 14, 15) QUAD_FMAC(7, 10, 14, 15) QUAD_FMAC(8, 11, 14, 15)
            : "+&v"(s1[0]), "+&v"(s1[1]), "+&v"(s1[2]), "+&v"(s2[0]), "+&v"(s2[1]), "+&v"(s2[2]),
              "+&v"(s3[0]), "+&v"(s3[1]), "+&v"(s3[2])
            : "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(a1), "v"(a2), "v"(a3), "n"(L));
    else if constexpr (N == 2)
        asm("s_nop 1\n\t" QUAD_FMAC(0, 6, 8, 11) QUAD_FMAC(1, 7, 8, 11) QUAD_FMAC(2, 6, 9, 11)
                QUAD_FMAC(3, 7, 9, 11) QUAD_FMAC(4, 6, 10, 11) QUAD_FMAC(5, 7, 10, 11)
            : "+&v"(s1[0]), "+&v"(s1[1]), "+&v"(s2[0]), "+&v"(s2[1]), "+&v"(s3[0]), "+&v"(s3[1])
            : "v"(x[0]), "v"(x[1]), "v"(a1), "v"(a2), "v"(a3), "n"(L));
    else
        asm("s_nop 1\n\t" QUAD_FMAC(0, 3, 4, 7) QUAD_FMAC(1, 3, 5, 7) QUAD_FMAC(2, 3, 6, 7)
            : "+&v"(s1[0]), "+&v"(s2[0]), "+&v"(s3[0])
            : "v"(x[0]), "v"(a1), "v"(a2), "v"(a3), "n"(L));
}
#undef QUAD_FMAC

// Sum, or largest value, over each 16-lane row, in every lane of it.
__device__ __forceinline__ double row_sum(double v) {
    v += dpp_d<kDppRor8>(v);
    v += dpp_d<kDppRor4>(v);
    v += dpp_d<kDppSwap2>(v);
    return v + dpp_d<kDppSwap1>(v);
}
__device__ __forceinline__ double row_max(double v) {
    v = fmax(v, dpp_d<kDppRor8>(v));
    v = fmax(v, dpp_d<kDppRor4>(v));
    v = fmax(v, dpp_d<kDppSwap2>(v));
    return fmax(v, dpp_d<kDppSwap1>(v));
}
__device__ __forceinline__ unsigned row_max(unsigned k) {
    k = max(k, (unsigned)__builtin_amdgcn_update_dpp(0, (int)k, kDppRor8, 0xF, 0xF, false));
    k = max(k, (unsigned)__builtin_amdgcn_update_dpp(0, (int)k, kDppRor4, 0xF, 0xF, false));
    k = max(k, (unsigned)__builtin_amdgcn_update_dpp(0, (int)k, kDppSwap2, 0xF, 0xF, false));
    return max(k, (unsigned)__builtin_amdgcn_update_dpp(0, (int)k, kDppSwap1, 0xF, 0xF, false));
}

// Square root of a normal d (NaN for 0), as by P. Markstein, "Software division
// and square root using Goldschmidt's algorithms" (2004): from the reciprocal
// square root one Goldschmidt step on g -> sqrt(d) and h -> 1 / (2 sqrt(d)), then
// two corrections by the fused residual d - g^2.  No scaling for subnormal d: a
// pair of nodes that close makes the system singular, and it goes to
// k_weights_pair.
__device__ __forceinline__ double sqrt_normal(double d) {
    const double y = __builtin_amdgcn_rsq(d);
    double g = d * y, h = 0.5 * y;
    const double r = fma(-h, g, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    g = fma(fma(-g, g, d), h, g);
    return fma(fma(-g, g, d), h, g);
}

// The ten monomials of degree <= 3 in graded order, as pow_chain products.
template <class T>
__device__ __forceinline__ void quad_mono(T x, T y, T (&p)[kPairKP]) {
    const T xx = x * x, yy = y * y;
    p[0] = T(1);
    p[1] = x;
    p[2] = y;
    p[3] = xx;
    p[4] = x * y;
    p[5] = yy;
    p[6] = xx * x;
    p[7] = xx * y;
    p[8] = x * yy;
    p[9] = yy * y;
}

// v rounded to a multiple of the power of two that `magic` = 1.5 * 2^52 * unit
// stands for (|v| well below magic).
__device__ __forceinline__ double round_to(double v, double magic) { return (v + magic) - magic; }

// magic that cuts values up to vmax to 30 bits.
__device__ __forceinline__ double cut_magic(double vmax) {
    int E = 0;
    frexp(vmax, &E);
    return ldexp(1.5, E - 30 + 52);
}

template <int NO>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2)))
k_weights_quad(const double *__restrict__ xq, int64_t nq, const double *__restrict__ xs, int64_t ns,
               const int *__restrict__ idx, OpSet ops, double *__restrict__ w,
               unsigned long long *__restrict__ todo) {
    constexpr int N = kPairN, KP = kPairKP, M = 7;
    __shared__ QuadLds lds[4];
    const int lane = threadIdx.x, l = lane & 15;
    QuadLds &S = lds[lane >> 4];
    const int64_t row_ = (int64_t)rbf::xcd_block(blockIdx.x, gridDim.x) * 4 + (lane >> 4);
    const bool valid = row_ < nq;
    const int64_t row = valid ? row_ : nq - 1;
    bool suspect = false;
    auto leave = [&]() {
        w[row] = NAN;  // slot 0 of the first operator marks the row
        // (Looked at first: 160,000 rows that all add to it take 1.5 ms.)
        if (__hip_atomic_load(todo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) == 0)
            __hip_atomic_store(todo, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    auto all_left = [&]() {
        unsigned long long sm = __ballot(suspect);
        sm |= sm >> 8, sm |= sm >> 4, sm |= sm >> 2, sm |= sm >> 1;
        return (sm & 0x0001000100010001ull) == 0x0001000100010001ull;
    };

    // Stencil nodes l and 16 + l, shifted and scaled by a power of two.
    const bool has1 = l < N - 16;
    double x0, y0, x1, y1;
    {
        int j0 = idx[(int64_t)l * nq + row], j1 = has1 ? idx[(int64_t)(16 + l) * nq + row] : 0;
        if (j0 < 0 || (int64_t)j0 >= ns) suspect = true, j0 = 0;
        if (j1 < 0 || (int64_t)j1 >= ns) suspect = true, j1 = 0;
        const double qx = xq[row], qy = xq[nq + row];
        x0 = xs[j0] - qx, y0 = xs[ns + j0] - qy;
        x1 = has1 ? xs[j1] - qx : 0.0, y1 = has1 ? xs[ns + j1] - qy : 0.0;
    }
    const double d2max = row_max(fmax(x0 * x0 + y0 * y0, x1 * x1 + y1 * y1));
    int E = 0;
    frexp(d2max, &E);
    const int e = (E >= 0) ? (E + 1) / 2 : -((-E) / 2);
    if (!(d2max > 0.0) || !isfinite(d2max)) suspect = true;
    x0 = ldexp(x0, -e), y0 = ldexp(y0, -e), x1 = ldexp(x1, -e), y1 = ldexp(y1, -e);

    // 1. The nodes of B: elimination of P in FP32 with row pivoting.  The key
    // of a candidate holds its stencil slot in its low five bits.
    {
        float q0[KP], q1[KP];
        quad_mono((float)x0, (float)y0, q0);
        quad_mono((float)x1, (float)y1, q1);
        unsigned used = 0;
        int pos0 = -1, pos1 = -1;
        float *buf = reinterpret_cast<float *>(S.t);
#pragma unroll
        for (int k = 0; k < KP; ++k) {
            const unsigned k0 = (used >> l & 1) ? 0u : ((__float_as_uint(fabsf(q0[k])) & ~31u) | (31 - l));
            const unsigned k1 = (!has1 || (used >> (16 + l) & 1))
                                    ? 0u
                                    : ((__float_as_uint(fabsf(q1[k])) & ~31u) | (15 - l));
            const int id = 31 - (int)(row_max(max(k0, k1)) & 31u);
            used |= 1u << id;
            float *pr = buf + (k & 1) * 12;
            if ((id & 15) == l) {
                (id >> 4 ? pos1 : pos0) = k;
#pragma unroll
                for (int j = k; j < KP; ++j) pr[j] = id >> 4 ? q1[j] : q0[j];
            }
            __syncthreads();
            const float inv = __builtin_amdgcn_rcpf(pr[k]);
            const float f0 = -q0[k] * inv, f1 = -q1[k] * inv;
#pragma unroll
            for (int j = k + 1; j < KP; ++j) {
                q0[j] = fmaf(f0, pr[j], q0[j]);
                q1[j] = fmaf(f1, pr[j], q1[j]);
            }
        }
        if (__popc(used) != KP) suspect = true;  // NaN keys can name a slot twice
        // The other nodes follow in stencil order.
        const unsigned rest = ~used & ((1u << N) - 1);
        if (pos0 < 0) pos0 = KP + __popc(rest & ((1u << l) - 1));
        if (pos1 < 0) pos1 = KP + __popc(rest & ((1u << (16 + l)) - 1));
        pos0 = min(pos0, N - 1), pos1 = min(pos1, N - 1);
        S.c[pos0] = double2{x0, y0};
        S.node[pos0] = l;
        if (has1) {
            S.c[pos1] = double2{x1, y1};
            S.node[pos1] = 16 + l;
        }
    }
    __syncthreads();
    int r0 = min(l, 11), r1 = 12 + l;  // rows of this lane's slots
    x0 = S.c[r0].x, y0 = S.c[r0].y, x1 = S.c[r1].x, y1 = S.c[r1].y;

    // Between the steps: what can be read from LDS or computed from the
    // coordinates again is, instead of being kept in registers.
#define QUAD_STEP() \
    asm volatile("" : "+v"(x0), "+v"(y0), "+v"(x1), "+v"(y1), "+v"(r0), "+v"(r1) : : "memory")
    // 2. P_B = L U in slot 0 (rows 10 and 11 are eliminated along).
    double p0[KP], m[KP], myui = 0.0;
    quad_mono(x0, y0, p0);
    quad_mono(x1, y1, m);
    double ui[KP];
    static_for<KP>(QUAD_FN(auto kc) {
        constexpr int k = kc;
        const double d = row_bcast<k>(p0[k]);
        if (!(fabs(d) > 0x1p-20)) suspect = true;
        ui[k] = recip_nr(d);
        const double lk = p0[k] * ui[k];
        const double nl = (l > k) ? -lk : 0.0;
        if (l == k) myui = ui[k];
        p0[k] = (l > k) ? lk : p0[k];
        fmac_self<k, KP - 1 - k>(p0 + k + 1, nl);
    });
    // A wavefront whose four systems are all left ends here: where all rows are (nodes
    // squeezed to 1:100), a call with 160,000 takes 3.07 ms, 3.85 if they run to the end,
    // and 2.98 without this kernel.
    if (all_left()) {
        if (valid && l == 0) leave();
        return;
    }
    // A, one evaluation per pair (24 rounds of 16 pairs).
#pragma unroll 4
    for (int e0 = 0; e0 < kQuadTri; e0 += 16) {
        const unsigned ij = kPairs.v[e0 + l];
        const double2 ci = S.c[ij >> 8], cj = S.c[ij & 255];
        const double dx = ci.x - cj.x, dy = ci.y - cj.y;
        const double dd = dx * dx + dy * dy;
        S.a[e0 + l] = ((dd * dd) * dd) * sqrt_normal(dd);
    }

    QUAD_STEP();
    // Columns of P_B^-1: lane k < 10 holds column k.
    double v[KP];
#pragma unroll
    for (int t = 0; t < KP; ++t) v[t] = (t == l) ? 1.0 : 0.0;
    static_for<KP - 1>(QUAD_FN(auto kc) {
        constexpr int k = kc;
        fmac_lanes<k + 1, KP - 1 - k>(v + k + 1, p0[k], -v[k]);
    });
    static_for<KP>(QUAD_FN(auto kc) {
        constexpr int k = KP - 1 - kc;
        v[k] *= ui[k];
        fmac_lanes<0, k>(v, p0[k], -v[k]);
    });
    // M: rows 12..27 in m, rows 10 and 11 in p0 of lanes 10 and 11.
    static_for<KP>(QUAD_FN(auto kc) {
        constexpr int k = kc;
        m[k] *= ui[k];
        fmac_lane<k, KP - 1 - k>(m + k + 1, p0 + k + 1, -m[k]);
    });
    static_for<KP - 1>(QUAD_FN(auto kc) {
        constexpr int k = KP - 1 - kc;
        fmac_lane<k, k>(m, p0, -m[k]);
        fmac_self<k, k>(p0, (l >= KP) ? -p0[k] : 0.0);
    });
    __syncthreads();  // S.t: pivot rows read, M written
#pragma unroll
    for (int k = 0; k < KP; ++k) {
        S.t[(2 + l) * KP + k] = m[k];
        if (l == 10 || l == 11) S.t[(l - 10) * KP + k] = p0[k];
    }

    // 3. K.  Entries of A from LDS: row r, column j.
    auto entry0 = QUAD_FN(auto jc) {
        constexpr int j = jc;
        if constexpr (j >= 12) {
            return S.a[j * (j - 1) / 2 + r0];
        } else {
            const double a = S.a[(j < r0) ? r0 * (r0 - 1) / 2 + j : j * (j - 1) / 2 + r0];
            return (j == r0) ? 0.0 : a;
        }
    };
    auto entry1 = QUAD_FN(auto jc) {
        constexpr int j = jc;
        if constexpr (j < 12) {
            return S.a[r1 * (r1 - 1) / 2 + j];
        } else {
            const double a = S.a[(j < r1) ? r1 * (r1 - 1) / 2 + j : j * (j - 1) / 2 + r1];
            return (j == r1) ? 0.0 : a;
        }
    };
    double a1[N], ka, kb;  // slot 1: columns 10..27 of K; lanes 10, 11: columns 10, 11 of their rows
    double nw[NO], ws0[NO], ws1[NO], f0[NO], f1[NO], bb0[NO], bb1[NO];
    // w0 = P_B^-T g, in lanes 0..9.
#pragma unroll
    for (int o = 0; o < NO; ++o) {
        const int code = ops.code[o];
        ws0[o] = (code == RBF_OP_ID) ? v[0]
                 : (code == RBF_OP_DX) ? v[1]
                 : (code == RBF_OP_DY) ? v[2]
                                       : 2.0 * v[3] + 2.0 * v[5];
        f0[o] = rhs_phs(x0, y0, M, code);
        f1[o] = rhs_phs(x1, y1, M, code);
        bb0[o] = f0[o];
        bb1[o] = f1[o];
    }
    {
        double a0[12], ap[KP];
        static_for<12>(QUAD_FN(auto jc) { a0[jc] = entry0(jc); });
        static_for<N>(QUAD_FN(auto jc) { a1[jc] = entry1(jc); });
        // bb = f - A w0.
        static_for<KP>(QUAD_FN(auto kc) {
            constexpr int k = kc;
            fmac_lane<k, NO>(bb0, ws0, -a0[k]);
            fmac_lane<k, NO>(bb1, ws0, -a1[k]);
        });
#pragma unroll
        for (int k = 0; k < KP; ++k) ap[k] = a0[k];
        static_for<KP>(QUAD_FN(auto kc) {
            constexpr int k = kc;
            fmac_lane<k, KP>(ap, a0, -p0[k]);
        });
        ka = a0[10], kb = a0[11];
        static_for<KP>(QUAD_FN(auto kc) {
            constexpr int k = kc;
            fmac_lanes<10, 1>(&ka, a0[k], -p0[k]);
            fmac_lanes<11, 1>(&kb, a0[k], -p0[k]);
            fmac_lanes<10, 1>(&ka, p0[k], -ap[k]);
            fmac_lanes<11, 1>(&kb, p0[k], -ap[k]);
        });
#pragma unroll
        for (int k = 0; k < KP; ++k) ap[k] = a1[k];
        static_for<KP>(QUAD_FN(auto kc) {
            constexpr int k = kc;
            fmac_lane<k, KP>(ap, a0, -m[k]);
        });
        static_for<KP>(QUAD_FN(auto kc) {
            constexpr int k = kc;
            fmac_lanes<10, 2>(a1 + 10, a0[k], -m[k]);
            fmac_lanes<10, 2>(a1 + 10, p0[k], -ap[k]);
            fmac_lanes<0, 16>(a1 + 12, a1[k], -m[k]);
            fmac_lanes<0, 16>(a1 + 12, m[k], -ap[k]);
        });
    }
    QUAD_STEP();
    double mt[18];  // lanes 0..9: column of M
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 18; ++i) mt[i] = S.t[i * KP + min(l, KP - 1)];

    // K = L D L^T: rows 10 and 11, then the 16 lanes of slot 1.
    const double k1110 = row_bcast<11>(ka);
    const double d10 = row_bcast<10>(ka), di10 = recip_nr(d10), l1110 = k1110 * di10;
    const double d11 = fma(-l1110, k1110, row_bcast<11>(kb)), di11 = recip_nr(d11);
    double kmax = fmax(d10, d11), dmin = fmin(d10, d11);
    {
        const double nl = -a1[10] * di10;
        fmac_lanes<0, 16>(a1 + 12, a1[10], nl);
        a1[11] = fma(nl, k1110, a1[11]);
        a1[10] = nl;
        const double nl2 = -a1[11] * di11;
        fmac_lanes<0, 16>(a1 + 12, a1[11], nl2);
        a1[11] = nl2;
    }
    double mydi = 0.0;
    static_for<16>(QUAD_FN(auto sc) {
        constexpr int s = sc;
        const double c = a1[12 + s];
        const double d = row_bcast<s>(c), di = recip_nr(d);
        kmax = fmax(kmax, d);
        dmin = (d < dmin || !(d == d)) ? d : dmin;
        const double nl = (l > s) ? -c * di : 0.0;
        fmac_lanes<s + 1, 15 - s>(a1 + 13 + s, c, nl);
        a1[12 + s] = (l > s) ? nl : c;
        if (l == s) mydi = di;
    });
    if (!(dmin > 0x1p-40 * kmax) || !isfinite(kmax)) suspect = true;
    // Lanes below the diagonal hold -L, lanes above it -U / D.
    static_for<16>(QUAD_FN(auto sc) {
        constexpr int s = sc;
        a1[12 + s] = (l < s) ? -a1[12 + s] * mydi : a1[12 + s];
    });

    // K y = Z^T b (b in bb0, bb1; overwritten), then w = w0 + Z y for w0 in
    // ws0 of lanes 0..9: results in ws0, ws1.
    auto reduced_solve = QUAD_FN() {
        double c0[NO];
#pragma unroll
        for (int o = 0; o < NO; ++o) c0[o] = bb0[o];
        static_for<KP>(QUAD_FN(auto kc) {
            constexpr int k = kc;
            fmac_lane<k, NO>(bb1, c0, -m[k]);
            fmac_lane<k, NO>(bb0, c0, -p0[k]);  // lanes 10, 11
        });
        double z10[NO], z11[NO];
#pragma unroll
        for (int o = 0; o < NO; ++o) {
            z10[o] = row_bcast<10>(bb0[o]);
            z11[o] = fma(-l1110, z10[o], row_bcast<11>(bb0[o]));
            bb1[o] = fma(a1[11], z11[o], fma(a1[10], z10[o], bb1[o]));
        }
        static_for<15>(QUAD_FN(auto sc) {
            constexpr int s = sc;
            fmac_self<s, NO>(bb1, (l > s) ? a1[12 + s] : 0.0);
        });
#pragma unroll
        for (int o = 0; o < NO; ++o) bb1[o] *= mydi;
        static_for<15>(QUAD_FN(auto sc) {
            constexpr int s = 15 - sc;
            fmac_self<s, NO>(bb1, (l < s) ? a1[12 + s] : 0.0);
        });
#pragma unroll
        for (int o = 0; o < NO; ++o) {
            ws1[o] = bb1[o];
            z11[o] = fma(z11[o], di11, row_sum(a1[11] * ws1[o]));
            z10[o] = fma(-l1110, z11[o], fma(z10[o], di10, row_sum(a1[10] * ws1[o])));
            ws0[o] = fma(-mt[1], z11[o], fma(-mt[0], z10[o], ws0[o]));
        }
        static_for<16>(QUAD_FN(auto ic) {
            constexpr int i = ic;
            fmac_lane<i, NO>(ws0, ws1, -mt[2 + i]);
        });
#pragma unroll
        for (int o = 0; o < NO; ++o) ws0[o] = (l < KP) ? ws0[o] : (l == 10) ? z10[o] : z11[o];
    };

    // 4. First solution, then c from the rows of B.
    reduced_solve();
    QUAD_STEP();
    double c[NO];
    {
#pragma unroll
        for (int o = 0; o < NO; ++o) c[o] = f0[o];
        static_for<N>(QUAD_FN(auto jc) {
            constexpr int j = jc;
            const double na = -entry0(jc);
            if constexpr (j < 12) fmac_lane<j, NO>(c, ws0, na);
            else fmac_lane<j - 12, NO>(c, ws1, na);
        });
        static_for<KP - 1>(QUAD_FN(auto kc) {
            constexpr int k = kc;
            fmac_self<k, NO>(c, (l > k) ? -p0[k] : 0.0);
        });
        static_for<KP>(QUAD_FN(auto kc) {
            constexpr int k = KP - 1 - kc;
            double t[NO];
#pragma unroll
            for (int o = 0; o < NO; ++o) t[o] = c[o] * myui;
            if constexpr (k > 0) fmac_lane<k, NO>(c, t, (l < k) ? -p0[k] : 0.0);
        });
#pragma unroll
        for (int o = 0; o < NO; ++o) c[o] = (l < KP) ? c[o] * myui : 0.0;
    }

    QUAD_STEP();
    // 5. The iterate is cut to 30 bits (the correction makes up for that) and
    // its residuals formed: rows of A and P in bb0, bb1, constraints in rc
    // (lanes 0..9).
    double rc[NO], wf0[NO], wf1[NO];
    {
#pragma unroll
        for (int o = 0; o < NO; ++o) {
            const double gw = cut_magic(row_max(fmax((l < 12) ? fabs(ws0[o]) : 0.0, fabs(ws1[o]))));
            wf0[o] = round_to(ws0[o], gw);
            wf1[o] = round_to(ws1[o], gw);
            c[o] = round_to(c[o], cut_magic(row_max(fabs(c[o]))));
        }
        // 18-bit parts: A < 2^7 in units 2^-11 and 2^-29, P <= 1 in 2^-18 and 2^-36.
        constexpr double kA1 = 1.5 * 0x1p41, kA2 = 1.5 * 0x1p23, kP1 = 1.5 * 0x1p34, kP2 = 1.5 * 0x1p16;
        double sa[3][NO], sp[3][NO];
        auto product = QUAD_FN(auto lc, double a, double m1, double m2, const double *x,
                               double (&s)[3][NO]) {
            const double h = round_to(a, m1), rest = a - h, mid = round_to(rest, m2);
            fmac_split<lc, NO>(s[0], s[1], s[2], x, h, mid, rest - mid);
        };
        // r = f - sum of the parts, the large ones with their rounding errors.
        auto finish = QUAD_FN(const double *f, double *r) {
#pragma unroll
            for (int o = 0; o < NO; ++o) {
                double t = f[o], err = 0.0;
                auto take = QUAD_FN(double b) {
                    const double u = t - b, bv = u - t;
                    err += (t - (u - bv)) + (-b - bv);
                    t = u;
                };
                take(sa[0][o]);
                take(sp[0][o]);
                take(sa[1][o]);
                take(sp[1][o]);
                r[o] = t + (err - (sa[2][o] + sp[2][o]));
            }
        };
        auto clear = QUAD_FN() {
#pragma unroll
            for (int o = 0; o < NO; ++o)
                for (int q = 0; q < 3; ++q) sa[q][o] = sp[q][o] = 0.0;
        };
        auto rows = QUAD_FN(auto slot) {
            QUAD_STEP();
            static_for<N>(QUAD_FN(auto jc) {
                constexpr int j = jc;
                double a;
                if constexpr (slot == 0) a = entry0(jc);
                else a = entry1(jc);
                if constexpr (j < 12) product(jc, a, kA1, kA2, wf0, sa);
                else product(std::integral_constant<int, j - 12>{}, a, kA1, kA2, wf1, sa);
            });
            double q[KP];
            if constexpr (slot == 0) quad_mono(x0, y0, q);
            else quad_mono(x1, y1, q);
            static_for<KP>(QUAD_FN(auto tc) { product(tc, q[tc], kP1, kP2, c, sp); });
        };
        clear();
        rows(std::integral_constant<int, 0>{});
        finish(f0, bb0);
        clear();
        rows(std::integral_constant<int, 1>{});
        finish(f1, bb1);
        // Constraints: P by columns through LDS, slot 1's nodes, then slot 0's.
        clear();
        const int lt = min(l, KP - 1);
        double q[KP];
        QUAD_STEP();
        quad_mono(x1, y1, q);
        __syncthreads();
#pragma unroll
        for (int t = 0; t < KP; ++t) S.t[l * KP + t] = q[t];
        __syncthreads();
        static_for<16>(QUAD_FN(auto ic) {
            product(ic, S.t[ic * KP + lt], kP1, kP2, wf1, sa);
        });
        quad_mono(x0, y0, q);
        __syncthreads();
#pragma unroll
        for (int t = 0; t < KP; ++t) S.t[l * KP + t] = q[t];
        __syncthreads();
        static_for<12>(QUAD_FN(auto ic) {
            product(ic, S.t[ic * KP + lt], kP1, kP2, wf0, sa);
        });
        int ta, tb;
        mono_exp(lt, ta, tb);
        double g[NO];
#pragma unroll
        for (int o = 0; o < NO; ++o) g[o] = rhs_poly(ta, tb, ops.code[o]);
        finish(g, rc);
    }
    QUAD_STEP();
    // Correction: the same solve with w0 = P_B^-T rc.
#pragma unroll
    for (int o = 0; o < NO; ++o) nw[o] = 0.0;
    static_for<KP>(QUAD_FN(auto tc) { fmac_lane<tc, NO>(nw, rc, v[tc]); });
#pragma unroll
    for (int o = 0; o < NO; ++o) ws0[o] = nw[o];
    static_for<KP>(QUAD_FN(auto kc) {
        constexpr int k = kc;
        fmac_lane<k, NO>(bb0, nw, -entry0(kc));
        fmac_lane<k, NO>(bb1, nw, -entry1(kc));
    });
    reduced_solve();

    // 6. Weights in physical units.
    bool finite = true;
#pragma unroll
    for (int o = 0; o < NO; ++o) {
        wf0[o] = ldexp(wf0[o] + ws0[o], -e * ops.order[o]);
        wf1[o] = ldexp(wf1[o] + ws1[o], -e * ops.order[o]);
        finite = finite && isfinite(wf0[o]) && isfinite(wf1[o]);
    }
    suspect = suspect || !finite;
    const bool redo = (__ballot(suspect) >> (lane & 48) & 0xffffull) != 0;
    if (!valid) return;
    const int n0 = S.node[r0], n1 = S.node[r1];
    if (redo) {
        if (l == 0) leave();
        return;
    }
#pragma unroll
    for (int o = 0; o < NO; ++o) {
        if (l < 12) w[((int64_t)o * N + n0) * nq + row] = wf0[o];
        w[((int64_t)o * N + n1) * nq + row] = wf1[o];
    }
}
#undef QUAD_FN
#undef QUAD_STEP
