// Cell passes of the upwind form through the block structure of A_K.
//
// Condensation (Step 1) and recovery (Step 3) both apply A_K^-1.  Stored as
// dense maps (A^-1 Mtilde, A^-1 B, C A^-1 Mtilde) that is nc (nc + 2 nt) numbers a
// cell, 13 KB at p = 3, and the passes do nothing but read them.  With
//   A = [[A_pp, k G], [-k G^T, A_uu]],  A_uu = M + dt f J (J the rotation),
// elimination of u leaves Sigma = A_pp + k^2 G A_uu^-1 G^T on the n depth
// unknowns, and every other factor is a reference-element table times the cell's
// affine map.  With X_f = M^-1 T_f, D_r = M^-1 G_r, K_r = M^-1 G_r^T (reference,
// r the reference direction) and Z = A_uu^-1 M (a complex n x n matrix on u1 + i u2):
//   v   = Z (r_u - (k/|J|) sum_f n_f L_f X_f lam_f)
//   w   = hs r_h + (k t/|J|) sum_f L_f X_f lam_f - k D.v
//   phi = (Sigma^-1 M) w
//   u   = v + Z k K phi
// Uniform f: Z = 1 / (1 + i dt f) is a number, and a cell stores Sigma^-1 M (n^2) and 14
// geometry factors, 0.9 KB at p = 3.  Where f varies inside the cells (rotating
// sphere) a cell stores Z (2 n^2) and, instead of Sigma^-1 M and the product D.v, the depth
// rows of A^-1 M (3 n^2), so that each is read once: phi = rows (w, y), u = Z (y + t), 4.1 KB;
// the condensation, which needs C A^-1 M alone (2.9 KB), keeps that dense map there.
// Measured (dense maps before): 256x256 torus, p = 3, one right-hand side: recovery 217 -> 42 us
// (168 MB of cell data and vectors, 4.0 TB/s), condensation with its gather 83 -> 35 us; 16:
// 721 -> 300 and 341 -> 267 us.  Level-6 sphere, p = 3: recovery at 1 / 3 / 8 / 16 / 32
// right-hand sides 147 / 1244 / 601 / 470 / 645 -> 82 / 108 / 205 / 348 / 440 us.
// One thread per (cell, right-hand side), right-hand side fastest; the tables are
// wave-uniform (scalar loads), the cell factors are 16-byte loads, consecutive
// cells in consecutive lanes.  All products are written as fma in one order, so
// a column's result does not depend on the batch it is in.
#include "hdg_device.h"
#include "hdg_kernels.h"

namespace hdg {

namespace {

template <int P>
struct CellTab {   // offsets of the tables (cell_tables)
    static constexpr int n = (P + 1) * (P + 2) / 2, m = P + 1;
    static constexpr int D = 0, K = 2 * n * n, X = 4 * n * n, F = X + 3 * n * m, MI = F + m * m, W = MI + n * n;
};

// lattice node (i, j) at counter-clockwise position k of local facet f
template <int P>
__device__ __forceinline__ constexpr int facet_node(int f, int k) {
    const int i = f == 0 ? P - k : (f == 1 ? 0 : k), j = f == 0 ? k : (f == 1 ? P - k : 0);
    return j * (P + 1) - j * (j - 1) / 2 + i;
}

__device__ __forceinline__ double fm(double a, double b, double c) { return __builtin_fma(a, b, c); }

// The tables are read by scalar loads (constant address space).  Hoisted together they need more
// scalar registers than there are, and the spills (2000 lane reads in the recovery at
// p = 3) cost more than the arithmetic: tie() makes the table's address depend on a
// value just computed, so that the next rows are not loaded before it.  (256x256 torus, p = 3, 16
// right-hand sides: recovery 506 -> 295 us; the condensation, which has no X tables and
// few spills, is faster without: 268 us, tied 430 us.)
typedef const __attribute__((address_space(4))) double *ctab;
__device__ __forceinline__ ctab as_tab(const double *p) { return (ctab)p; }
template <bool ON = true>
__device__ __forceinline__ void tie(ctab &tab, double &v) {
    if constexpr (ON) asm volatile("" : "+s"(tab), "+v"(v));
}

// A cell's factors, 16-byte pairs a fixed stride apart: in memory, or the block's copy in LDS
typedef __attribute__((address_space(3))) const dbl2_t lds_pair;
struct FromMem {
    const dbl2_t *p;
    size_t stride;
    __device__ __forceinline__ dbl2_t operator[](int q) const { return p[q * stride]; }
};
struct FromLds {
    lds_pair *p;
    int stride;
    __device__ __forceinline__ dbl2_t operator[](int q) const { return p[q * stride]; }
};

struct Geo {
    double j00, j01, j10, j11;   // k d(xi_r)/d(x_d)
    double ax[3], ay[3], b[3];   // k L n_x / |J|, k L n_y / |J|, k t L / |J| per facet
    double g;                    // |J| / k
};
template <typename F>
__device__ __forceinline__ Geo load_geo(const F &geo) {
    dbl2_t v[7];
#pragma unroll
    for (int q = 0; q < 7; ++q) v[q] = geo[q];
    return Geo{v[0].x, v[0].y, v[1].x, v[1].y, {v[2].x, v[3].x, v[4].x}, {v[2].y, v[3].y, v[4].y},
               {v[5].x, v[5].y, v[6].x}, v[6].y};
}

// t_d = k (M^-1 G_d^T phi), a node of phi at a time: g_r += K_r[.][j] phi_j, then the affine map
template <int P>
__device__ __forceinline__ void grad_t_add(ctab tab, int j, double pj,
                                           double (&g0)[CellTab<P>::n], double (&g1)[CellTab<P>::n]) {
    using T = CellTab<P>;
    constexpr int n = T::n;
#pragma unroll
    for (int i = 0; i < n; ++i) {
        g0[i] = fm(tab[T::K + j * n + i], pj, g0[i]);
        g1[i] = fm(tab[T::K + n * n + j * n + i], pj, g1[i]);
    }
}
template <int P>
__device__ __forceinline__ void grad_t_map(const Geo &g, double (&g0)[CellTab<P>::n], double (&g1)[CellTab<P>::n]) {
#pragma unroll
    for (int i = 0; i < CellTab<P>::n; ++i) {
        const double a = g0[i], b = g1[i];
        g0[i] = fm(g.j00, a, g.j10 * b);
        g1[i] = fm(g.j01, a, g.j11 * b);
    }
}
template <int P, bool TIE>
__device__ __forceinline__ void grad_t(ctab tab, const Geo &g,
                                       const double (&phi)[CellTab<P>::n], double (&t1)[CellTab<P>::n],
                                       double (&t2)[CellTab<P>::n]) {
    constexpr int n = CellTab<P>::n;
#pragma unroll
    for (int i = 0; i < n; ++i) t1[i] = t2[i] = 0.0;
#pragma unroll
    for (int j = 0; j < n; ++j) {
        grad_t_add<P>(tab, j, phi[j], t1, t2);
        tie<TIE>(tab, t2[n - 1]);
    }
    grad_t_map<P>(g, t1, t2);
}

// w -= k (D_1 v1 + D_2 v2)
template <int P, bool TIE>
__device__ __forceinline__ void sub_div(ctab tab, const Geo &g,
                                        const double (&v1)[CellTab<P>::n], const double (&v2)[CellTab<P>::n],
                                        double (&w)[CellTab<P>::n]) {
    using T = CellTab<P>;
    constexpr int n = T::n;
#pragma unroll
    for (int j = 0; j < n; ++j) {
        const double p = -fm(g.j00, v1[j], g.j01 * v2[j]), s = -fm(g.j10, v1[j], g.j11 * v2[j]);
#pragma unroll
        for (int i = 0; i < n; ++i) w[i] = fm(tab[T::D + j * n + i], p, fm(tab[T::D + n * n + j * n + i], s, w[i]));
        tie<TIE>(tab, w[n - 1]);
    }
}

// f uniform.  On entry w, y1, y2: the cell's right-hand side (hs r_h, r_u) less the trace
// terms; on exit phi in w and u in y1, y2: v = Z y, w -= k D.v, phi = (Sigma^-1 M) w, u = v + Z t
template <int P, bool TIE, typename F>
__device__ __forceinline__ void cell_inverse(const CellFactors &c, ctab tab, const Geo &g, const F &fs,
                                             double (&w)[CellTab<P>::n], double (&y1)[CellTab<P>::n],
                                             double (&y2)[CellTab<P>::n]) {
    constexpr int n = CellTab<P>::n;
    double phi[n], t1[n], t2[n];
#pragma unroll
    for (int i = 0; i < n; ++i) {
        const double a = y1[i];
        phi[i] = 0.0;
        y1[i] = fm(-c.zb, y2[i], c.za * a);
        y2[i] = fm(c.za, y2[i], c.zb * a);
    }
    sub_div<P, TIE>(tab, g, y1, y2, w);
#pragma unroll
    for (int q = 0; q < (n * n + 1) / 2; ++q) {
        const dbl2_t a = fs[q];
        phi[(2 * q) / n] = fm(a.x, w[(2 * q) % n], phi[(2 * q) / n]);
        if (2 * q + 1 < n * n) phi[(2 * q + 1) / n] = fm(a.y, w[(2 * q + 1) % n], phi[(2 * q + 1) / n]);
    }
    grad_t<P, TIE>(tab, g, phi, t1, t2);
#pragma unroll
    for (int i = 0; i < n; ++i) {
        w[i] = phi[i];
        y1[i] = fm(-c.zb, t2[i], fm(c.za, t1[i], y1[i]));
        y2[i] = fm(c.za, t2[i], fm(c.zb, t1[i], y2[i]));
    }
}

// f varying: q = (hs^-1 phi, u) written to dst (stride nb), a row at a time: phi_i = rows_i
// (w, y), t += K phi_i; then u_i = Z_i (y + t).  The next row's loads are in flight while a
// row is used; the row loops are not unrolled beyond that pair, or all their loads
// would be hoisted to the front (500 registers).
template <int P, typename F>
__device__ __forceinline__ void cell_inverse_vf(const CellFactors &c, ctab tab, const Geo &g, const F &fs, const F &z,
                                                const double (&w)[CellTab<P>::n], double (&y1)[CellTab<P>::n],
                                                double (&y2)[CellTab<P>::n], int nb, double *dst) {
    constexpr int n = CellTab<P>::n, RW = (3 * n + 1) / 2;   // rows of 3 n padded to pairs
    const double ih = 1.0 / c.hs;
    double t1[n], t2[n];
#pragma unroll
    for (int i = 0; i < n; ++i) t1[i] = t2[i] = 0.0;
    auto in = [&](int j) { return j < n ? w[j] : (j < 2 * n ? y1[j - n] : y2[j - 2 * n]); };
    auto row = [&](int i, dbl2_t (&a)[RW]) {
        const int q0 = min(i, n - 1) * RW;
#pragma unroll
        for (int q = 0; q < RW; ++q) a[q] = fs[q0 + q];
    };
    auto use = [&](int i, const dbl2_t (&a)[RW]) {
        double p = 0.0;
#pragma unroll
        for (int q = 0; q < RW; ++q) {
            p = fm(a[q].x, in(2 * q), p);
            if (2 * q + 1 < 3 * n) p = fm(a[q].y, in(2 * q + 1), p);
        }
        dst[i * nb] = ih * p;
        grad_t_add<P>(tab, i, p, t1, t2);
    };
    {
        dbl2_t a[RW], b[RW];
        row(0, a);
#pragma unroll 1
        for (int i = 0; i < n; i += 2) {
            row(i + 1, b);
            use(i, a);
            row(i + 2, a);
            if (i + 1 < n) use(i + 1, b);
        }
    }
    grad_t_map<P>(g, t1, t2);
#pragma unroll
    for (int i = 0; i < n; ++i) {
        y1[i] += t1[i];
        y2[i] += t2[i];
    }
    auto zrow = [&](int i, dbl2_t (&a)[n]) {
        const int q0 = min(i, n - 1) * n;
#pragma unroll
        for (int j = 0; j < n; ++j) a[j] = z[q0 + j];
    };
    auto zuse = [&](int i, const dbl2_t (&a)[n]) {
        double a1 = 0.0, a2 = 0.0;
#pragma unroll
        for (int j = 0; j < n; ++j) {
            a1 = fm(-a[j].y, y2[j], fm(a[j].x, y1[j], a1));
            a2 = fm(a[j].x, y2[j], fm(a[j].y, y1[j], a2));
        }
        dst[(n + i) * nb] = a1;
        dst[(2 * n + i) * nb] = a2;
    };
    dbl2_t a[n], b[n];
    zrow(0, a);
#pragma unroll 1
    for (int i = 0; i < n; i += 2) {
        zrow(i + 1, b);
        zuse(i, a);
        zrow(i + 2, a);
        if (i + 1 < n) zuse(i + 1, b);
    }
}

constexpr int CELL_THREADS = 256;
template <int P, bool VF>
constexpr int FACTOR_PAIRS = 7 + (VF ? CellTab<P>::n * ((3 * CellTab<P>::n + 1) / 2) + CellTab<P>::n * CellTab<P>::n
                                     : (CellTab<P>::n * CellTab<P>::n + 1) / 2);
// What a block passes through LDS:
//   CP_VECTORS  the cells' vectors: the inputs up to CELL_SMALL_RHS right-hand sides (a thread's
//               values lie nc nb doubles from its neighbour cell's), the results always;
//   CP_DIRECT   nothing: vectors are read and written in place, whole segments of right-hand
//               sides at a time;
//   CP_FACTORS  the cells' factors, vectors in place.  With many right-hand sides a wavefront's lanes
//               read one or two cells' factors, and a 16-byte load returns 1 KB to them through L1 for
//               the 16 or 32 it needs (f varying, p = 3: 257 loads, as long as the whole pass); from
//               LDS half of that, and each factor comes from memory once per block.
// REC: recovery, else condensation.
constexpr int CP_VECTORS = 0, CP_DIRECT = 1, CP_FACTORS = 2;
template <int P, bool VF, int MODE, bool REC>
__global__ __launch_bounds__(CELL_THREADS) void k_cell_pass(int nk, int nb, CellFactors c,
                                                            const int *__restrict__ cell_facet,
                                                            const int8_t *__restrict__ cell_rev,
                                                            const double *__restrict__ rc,
                                                            const double *__restrict__ lam, double *__restrict__ out) {
    using T = CellTab<P>;
    constexpr int n = T::n, m = T::m, nc = 3 * n;
    constexpr bool ST = MODE == CP_VECTORS, FL = MODE == CP_FACTORS;
    constexpr int NF = (FACTOR_PAIRS<P, VF>) - 7 - (VF ? n * n : 0);   // pairs of fs
    extern __shared__ double sm[];
    const size_t NK = (size_t)nk;
    ctab tab = as_tab(c.tab);
    const int cpb = MODE != CP_DIRECT ? CELL_THREADS / nb : 0, per = nc * nb;
    const int64_t t = (int64_t)xcd_block() * CELL_THREADS + threadIdx.x;
    const int K0 = xcd_block() * cpb, cnt = MODE != CP_DIRECT ? min(cpb, nk - K0) : 0;
    int cl, r, K;
    bool live;
    if constexpr (MODE != CP_DIRECT) {
        if (cnt <= 0) return;   // the whole block
        cl = threadIdx.x / nb;
        r = threadIdx.x - cl * nb;
        K = K0 + cl;
        live = cl < cnt;
        if (ST && nb <= CELL_SMALL_RHS) {
            stage_cells(rc + (size_t)K0 * per, sm, cnt * per);
            __syncthreads();
        }
        if constexpr (FL) {
            dbl2_t *dst = reinterpret_cast<dbl2_t *>(sm);
            for (int i = threadIdx.x; i < (FACTOR_PAIRS<P, VF>) * cpb; i += CELL_THREADS) {
                const int q = i / cpb, k = min(K0 + i - q * cpb, nk - 1);
                const double *src = q < 7 ? c.geo : (q < 7 + NF ? c.fs : c.zt);
                const int o = q < 7 ? q : (q < 7 + NF ? q - 7 : q - 7 - NF);
                dst[i] = reinterpret_cast<const dbl2_t *>(src)[o * NK + k];
            }
            __syncthreads();
        }
    } else {
        K = (int)(t / nb);
        r = (int)(t - (int64_t)K * nb);
        cl = 0;
        live = K < nk;
        if (!live) return;
    }
    if (live) {
        auto factor = [&](const double *src, int q) {
            if constexpr (FL) return FromLds{(lds_pair *)sm + q * cpb + cl, cpb};
            else return FromMem{reinterpret_cast<const dbl2_t *>(src) + K, NK};
        };
        const Geo g = load_geo(factor(c.geo, 0));
        double w[n], y1[n], y2[n];
        const double *src = ST && nb <= CELL_SMALL_RHS ? sm + cl * per + r : rc + (size_t)K * per + r;
#pragma unroll
        for (int i = 0; i < n; ++i) {
            w[i] = c.hs * src[i * nb];
            y1[i] = src[(n + i) * nb];
            y2[i] = src[(2 * n + i) * nb];
        }
        if constexpr (REC) {
#pragma unroll
            for (int f = 0; f < 3; ++f) {
                const int e = cell_facet[f * NK + K], rev = cell_rev[f * NK + K];
                double l[m], lr[m];
#pragma unroll
                for (int k = 0; k < m; ++k) l[k] = lam[((size_t)e * m + k) * nb + r];
#pragma unroll
                for (int k = 0; k < m; ++k) lr[k] = rev ? l[P - k] : l[k];
#pragma unroll
                for (int i = 0; i < n; ++i) {
                    double x = 0.0;
#pragma unroll
                    for (int k = 0; k < m; ++k) x = fm(tab[T::X + (f * n + i) * m + k], lr[k], x);
                    w[i] = fm(g.b[f], x, w[i]);
                    y1[i] = fm(-g.ax[f], x, y1[i]);
                    y2[i] = fm(-g.ay[f], x, y2[i]);
                    if (i == n / 2 || i == n - 1) tie(tab, y2[i]);
                }
            }
        }
        double *dst = ST ? sm + cl * per + r : out + (size_t)K * per + r;
        if constexpr (VF) cell_inverse_vf<P>(c, tab, g, factor(c.fs, 7), factor(c.zt, 7 + NF), w, y1, y2, nb, dst);
        else cell_inverse<P, REC>(c, tab, g, factor(c.fs, 7), w, y1, y2);
        if constexpr (VF) {
        } else if constexpr (REC) {
            const double ih = 1.0 / c.hs;
#pragma unroll
            for (int i = 0; i < n; ++i) {
                dst[i * nb] = ih * w[i];
                dst[(n + i) * nb] = y1[i];
                dst[(2 * n + i) * nb] = y2[i];
            }
        } else {
            // C q: the traces t phi + n.u of the facet's nodes against the trace mass
#pragma unroll
            for (int f = 0; f < 3; ++f) {
                double e[m];
#pragma unroll
                for (int k = 0; k < m; ++k) {
                    const int i = facet_node<P>(f, k);
                    e[k] = g.g * fm(g.b[f], w[i], fm(g.ax[f], y1[i], g.ay[f] * y2[i]));
                }
#pragma unroll
                for (int k = 0; k < m; ++k) {
                    double s = 0.0;
#pragma unroll
                    for (int l = 0; l < m; ++l) s = fm(tab[T::F + k * m + l], e[l], s);
                    out[((size_t)(f * m + k) * NK + K) * nb + r] = s;
                }
            }
        }
    }
    if constexpr (ST && REC) {
        __syncthreads();
        stage_cells(sm, out + (size_t)K0 * per, cnt * per);
    }
}

// out = scale (q - r), r the right-hand side for which the stage equations hold with q and
// the trace lam = half[0] + half[1]: M r = A q + B lam, evaluated term by term
// (E_f phi = T_f times the facet's nodal values; the rotation's quadrature where f varies)
template <int P, bool VF>
__global__ __launch_bounds__(CELL_THREADS) void k_cell_tendency(int nk, int nb, CellFactors c, double scale, double dt,
                                                                double f0, double omega,
                                                                const double *__restrict__ corners,
                                                                const double *__restrict__ qx,
                                                                const int *__restrict__ cell_facet,
                                                                const int8_t *__restrict__ cell_rev,
                                                                const double *__restrict__ q,
                                                                const double *__restrict__ half,
                                                                double *__restrict__ out) {
    using T = CellTab<P>;
    constexpr int n = T::n, m = T::m, nc = 3 * n, nq = (P + 3) * (P + 3);
    const int64_t t = (int64_t)xcd_block() * CELL_THREADS + threadIdx.x;
    const int K = (int)(t / nb), r = (int)(t - (int64_t)K * nb);
    if (K >= nk) return;
    const size_t NK = (size_t)nk;
    ctab tab = as_tab(c.tab);
    const Geo g = load_geo(FromMem{reinterpret_cast<const dbl2_t *>(c.geo) + K, NK});
    double phi[n], u1[n], u2[n], d0[n], d1[n], d2[n];   // d = r - q
    const double *src = q + (size_t)K * nc * nb + r;
#pragma unroll
    for (int i = 0; i < n; ++i) {
        phi[i] = c.hs * src[i * nb];
        u1[i] = src[(n + i) * nb];
        u2[i] = src[(2 * n + i) * nb];
        d0[i] = 0.0;
    }
    sub_div<P, true>(tab, g, u1, u2, d0);
    grad_t<P, true>(tab, g, phi, d1, d2);
#pragma unroll
    for (int i = 0; i < n; ++i) {
        d0[i] = -d0[i];
        d1[i] = -d1[i];
        d2[i] = -d2[i];
    }
#pragma unroll
    for (int f = 0; f < 3; ++f) {
        const int e = cell_facet[f * NK + K], rev = cell_rev[f * NK + K];
        double l[m], lr[m];
#pragma unroll
        for (int k = 0; k < m; ++k)
            l[k] = half[(((size_t)e * 2 + 0) * m + k) * nb + r] + half[(((size_t)e * 2 + 1) * m + k) * nb + r];
#pragma unroll
        for (int k = 0; k < m; ++k) lr[k] = rev ? l[P - k] : l[k];
#pragma unroll
        for (int i = 0; i < n; ++i) {
            double x = 0.0, xp = 0.0;
#pragma unroll
            for (int k = 0; k < m; ++k) {
                const double a = tab[T::X + (f * n + i) * m + k];
                x = fm(a, lr[k], x);
                xp = fm(a, phi[facet_node<P>(f, k)] - lr[k], xp);
            }
            d0[i] = fm(g.b[f], xp, d0[i]);
            d1[i] = fm(g.ax[f], x, d1[i]);
            d2[i] = fm(g.ay[f], x, d2[i]);
            if (i == n / 2 || i == n - 1) tie(tab, d2[i]);
        }
    }
    if constexpr (!VF) {
#pragma unroll
        for (int i = 0; i < n; ++i) {
            d1[i] = fm(-dt * f0, u2[i], d1[i]);
            d2[i] = fm(dt * f0, u1[i], d2[i]);
        }
    } else {
        // M^-1 (f phi_j, phi_i) u by the setup's quadrature rule (weights and basis values in the tables)
        const double *X = corners + 9 * (size_t)K;
        double s1[n], s2[n];
#pragma unroll
        for (int i = 0; i < n; ++i) s1[i] = s2[i] = 0.0;
        for (int k = 0; k < nq; ++k) {
            double x[3];
#pragma unroll
            for (int d = 0; d < 3; ++d) x[d] = X[d] + qx[2 * k] * (X[3 + d] - X[d]) + qx[2 * k + 1] * (X[6 + d] - X[d]);
            const double f = f0 + 2.0 * omega * x[2] / sqrt(x[0] * x[0] + x[1] * x[1] + x[2] * x[2]);
            const ctab ph = tab + T::W + nq + k * n;
            double a1 = 0.0, a2 = 0.0;
#pragma unroll
            for (int j = 0; j < n; ++j) {
                a1 = fm(ph[j], u1[j], a1);
                a2 = fm(ph[j], u2[j], a2);
            }
            const double wf = dt * f * tab[T::W + k];
            a1 *= wf;
            a2 *= wf;
#pragma unroll
            for (int i = 0; i < n; ++i) {
                s1[i] = fm(ph[i], a1, s1[i]);
                s2[i] = fm(ph[i], a2, s2[i]);
            }
        }
#pragma unroll
        for (int i = 0; i < n; ++i)
#pragma unroll
            for (int j = 0; j < n; ++j) {
                const double a = tab[T::MI + i * n + j];
                d1[i] = fm(-a, s2[j], d1[i]);
                d2[i] = fm(a, s1[j], d2[i]);
            }
    }
    double *dst = out + (size_t)K * nc * nb + r;
    const double ih = 1.0 / c.hs;
#pragma unroll
    for (int i = 0; i < n; ++i) {
        dst[i * nb] = -scale * ih * d0[i];
        dst[(n + i) * nb] = -scale * d1[i];
        dst[(2 * n + i) * nb] = -scale * d2[i];
    }
}

// ------------------------------------------------------------------ setup of Z (f varying inside the cells)
//
// Z = (M + i dt M_f)^-1 M as the real 2n x 2n system [[M, -dt M_f], [dt M_f, M]] (both
// over |J|) with right-hand side [M; 0]: a lane per row, two cells per wavefront, the
// row in registers, eliminated in order (its symmetric part is M + M: no pivoting).
template <int P>
__global__ __launch_bounds__(64) void k_cell_rot(int nk, const double *__restrict__ corners,
                                                 const double *__restrict__ rM, const double *__restrict__ qx,
                                                 const double *__restrict__ tab, double dt, double f0, double omega,
                                                 double *__restrict__ zt) {
    using T = CellTab<P>;
    constexpr int n = T::n, N = 2 * n, LD = 3 * n, nq = (P + 3) * (P + 3);
    static_assert(N <= 32, "a 32-lane half holds the rows of a cell");
    __shared__ double sphi[nq * n], tM[n * n], fq[2][nq], Mf[2][n * n], prow[2][LD];
    const int lane = threadIdx.x, h = lane >> 5, r = lane & 31;
    const int pair = xcd_block();
    if (2 * pair >= nk) return;
    const bool live = 2 * pair + h < nk;
    const int K = live ? 2 * pair + h : nk - 1;
    const double *X = corners + 9 * (size_t)K;
    for (int i = lane; i < nq * n; i += 64) sphi[i] = tab[T::W + nq + i];
    for (int i = lane; i < n * n; i += 64) tM[i] = rM[i];
    for (int k = r; k < nq; k += 32) {
        double x[3];
        for (int d = 0; d < 3; ++d) x[d] = X[d] + qx[2 * k] * (X[3 + d] - X[d]) + qx[2 * k + 1] * (X[6 + d] - X[d]);
        fq[h][k] = tab[T::W + k] * (f0 + 2.0 * omega * x[2] / sqrt(x[0] * x[0] + x[1] * x[1] + x[2] * x[2]));
    }
    __syncthreads();
    for (int e = r; e < n * n; e += 32) {
        double s = 0.0;
        for (int k = 0; k < nq; ++k) s += fq[h][k] * sphi[k * n + e / n] * sphi[k * n + e % n];
        Mf[h][e] = dt * s;
    }
    __syncthreads();
    const bool row_ok = r < N;
    const int hi = row_ok ? r / n : 0, i = row_ok ? r % n : 0;
    double a[LD];
#pragma unroll
    for (int c = 0; c < LD; ++c) {
        const int j = c % n;
        double v = 0.0;
        if (c >= N) v = hi == 0 ? tM[i * n + j] : 0.0;
        else if ((c < n) == (hi == 0)) v = tM[i * n + j];
        else v = hi == 0 ? -Mf[h][i * n + j] : Mf[h][i * n + j];
        a[c] = row_ok ? v : 0.0;
    }
#pragma unroll
    for (int k = 0; k < N; ++k) {
        if (r == k) {
            const double ip = 1.0 / a[k];
#pragma unroll
            for (int c = k + 1; c < LD; ++c) {
                a[c] *= ip;
                prow[h][c] = a[c];
            }
        }
        __syncthreads();
        if (r != k) {
            const double g = a[k];
#pragma unroll
            for (int c = k + 1; c < LD; ++c) a[c] -= g * prow[h][c];
        }
        __syncthreads();
    }
    if (live && row_ok) {
#pragma unroll
        for (int j = 0; j < n; ++j) zt[((size_t)(i * n + j) * nk + K) * 2 + hi] = a[N + j];
    }
}

template <int P, bool VF, bool REC>
void launch_pass(int nk, int nb, const CellFactors &c, const int *cell_facet, const int8_t *cell_rev, const double *rc,
                 const double *lam, double *out, hipStream_t s) {
    constexpr int nc = 3 * CellTab<P>::n;
    auto grid8 = [](int64_t blocks) { return dim3((unsigned)((blocks + N_XCD - 1) / N_XCD * N_XCD)); };
    const int cpb = CELL_THREADS / nb;
    const size_t vectors = sizeof(double) * cpb * nc * nb, factors = (size_t)16 * (FACTOR_PAIRS<P, VF>) * cpb;
#define GO(MODE, BYTES)                                                                                            \
    hipLaunchKernelGGL((k_cell_pass<P, VF, MODE, REC>),                                                            \
                       grid8(MODE == CP_DIRECT ? ((int64_t)nk * nb + CELL_THREADS - 1) / CELL_THREADS              \
                                               : (nk + cpb - 1) / cpb),                                            \
                       dim3(CELL_THREADS), BYTES, s, nk, nb, c, cell_facet, cell_rev, rc, lam, out)
    if constexpr (VF) {
        // Factors through LDS as soon as they fit (p = 3: from 17 right-hand sides on); else results
        // through LDS, as the row loops write them one by one (a store to memory there holds up the next
        // row's loads, which the same counter waits for).  Recovery on the level-6 sphere, results / factors
        // (dense maps): p = 1 at 16, 32, 64 right-hand sides 65 / 49 (56), 138 / 103 (108), 252 / 186 (192) us;
        // p = 2 168 / 125 (195), 315 / 207 (298), 596 / 363 (461); p = 3 at 20, 32, 64
        // 432 / 339 (555), 644 / 440 (619), 1225 / 718 (953).
        if (nb > CELL_SMALL_RHS && factors <= 65536) GO(CP_FACTORS, factors);
        else GO(CP_VECTORS, vectors);
    } else if (nb <= CELL_SMALL_RHS) {
        GO(CP_VECTORS, vectors);
    } else {
        // Condensation at p = 3, where a wavefront has at most two cells: 200x200 torus, direct / factors
        // (dense map): 32 right-hand sides 301 / 273 (302), 64 553 / 499 (524) us; 96x96 61.5 / 63.1 (62), 48
        // 106 / 96 (97), 64 140 / 129 (129); at 9 to 28 the direct form is up to 1.14 times faster there.
        // The recovery has fewer wavefronts with it (200x200, 16: 184 / 205).
        if constexpr (!REC && P == 3) {
            if (nb > 32) {
                GO(CP_FACTORS, factors);
                return;
            }
        }
        GO(CP_DIRECT, 0);
    }
#undef GO
}

}  // namespace

void launch_cell_pass(int p, bool rec, int nk, int nb, const CellFactors &c, const int *cell_facet,
                      const int8_t *cell_rev, const double *rc, const double *lam, double *out, hipStream_t s) {
#define CP(P, VF, REC)                                                                                        \
    launch_pass<P, VF, REC>(nk, nb, c, cell_facet, cell_rev, rc, lam, out, s)
    if (c.zt) { switch (p) { case 1: CP(1, true, true); break; case 2: CP(2, true, true); break; default: CP(3, true, true); break; } }
    else if (rec) { switch (p) { case 1: CP(1, false, true); break; case 2: CP(2, false, true); break; default: CP(3, false, true); break; } }
    else { switch (p) { case 1: CP(1, false, false); break; case 2: CP(2, false, false); break; default: CP(3, false, false); break; } }
#undef CP
}

void launch_cell_tendency(int p, int nk, int nb, const CellFactors &c, double scale, double dt, double f0, double omega,
                          const double *corners, const double *qx, const int *cell_facet, const int8_t *cell_rev,
                          const double *q, const double *half, double *out, hipStream_t s) {
    const int64_t blocks = ((int64_t)nk * nb + CELL_THREADS - 1) / CELL_THREADS;
    const dim3 grid((unsigned)((blocks + N_XCD - 1) / N_XCD * N_XCD));
#define CT(P, VF) hipLaunchKernelGGL((k_cell_tendency<P, VF>), grid, dim3(CELL_THREADS), 0, s, nk, nb, c, scale, dt, f0, \
                                     omega, corners, qx, cell_facet, cell_rev, q, half, out)
    if (c.zt) { switch (p) { case 1: CT(1, true); break; case 2: CT(2, true); break; default: CT(3, true); break; } }
    else { switch (p) { case 1: CT(1, false); break; case 2: CT(2, false); break; default: CT(3, false); break; } }
#undef CT
}

void launch_cell_rot(int p, int nk, const double *corners, const double *ref_M, const double *qx, const double *tab,
                     double dt, double f0, double omega, double *zt, hipStream_t s) {
    const dim3 grid((unsigned)(((nk + 1) / 2 + N_XCD - 1) / N_XCD * N_XCD));
#define CR(P) hipLaunchKernelGGL(k_cell_rot<P>, grid, dim3(64), 0, s, nk, corners, ref_M, qx, tab, dt, f0, omega, zt)
    switch (p) { case 1: CR(1); break; case 2: CR(2); break; default: CR(3); break; }
#undef CR
}

}  // namespace hdg
