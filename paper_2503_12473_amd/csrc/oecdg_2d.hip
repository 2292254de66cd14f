// oecdg_2d.hip -- 2D RK-OECDG on periodic Cartesian primal and dual meshes,
// tensor-product Q^k Legendre modes or the total-degree P^k (k = 1, 2, 3),
// linear advection or Euler.
//
// Per RK stage (eq:RKCDG):
//   k_stage2d   one workgroup per tile of TX x TY primal cells and the dual
//               cells with the same indices, one thread per cell.  Its threads
//               load the cells that the tile's operator reads, apply the OE
//               step of the previous stage to them in registers (OEstep2D solved
//               exactly, from the damping numerators of k_delta2d and sigma) and
//               put them in LDS; each thread then evaluates the operator of
//               eq:2D_H on its cell, takes the RK combination (the c/d table of
//               eq:RKCDG: SSP-RK3 by default, forward Euler, SSP-RK2 or
//               classical RK4) and writes the undamped stage output and, per
//               wave, its partial statistics;
//   k_delta2d   the damping numerators of that output (the edge integrals of
//               Sec. 2.2), one component and mesh of a tile of cells per
//               workgroup; its first workgroups reduce the partial statistics to
//               the global scalars (per mesh and component the domain average and
//               sigma of Sec. 2.2, the largest x and y wave speeds, and at a step
//               start tau and tau_max, tau_max = C_CFL / (beta_x/h_x +
//               beta_y/h_y), Sec. 2.1).
// k_stats2d and k_reduce2d give the statistics of a run's initial data;
// k_damp2d damps a state without a stage (the end of a run or of a single stage).
//
// Layout (global): u[(((q*(k+1) + a)*(k+1) + b)*ny + iy)*nx + ix]; dual cell
// (ix, iy) is centred on the lower-left vertex of primal cell (ix, iy), so
// primal (i, j) overlaps dual (i..i+1, j..j+1) and dual (i, j) overlaps
// primal (i-1..i, j-1..j).
#include "oecdg_device.h"
#include "oecdg_internal.h"
#include "oecdg_tables.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>

namespace oecdg {

// ---------------------------------------------------------------- fluxes ---

// 1/x from the hardware estimate and two Newton steps (within an ulp or so of
// the correctly rounded quotient; the flux divisions do not need the full
// IEEE division sequence).
__device__ inline double rcp_nr(double x) {
    double r = __builtin_amdgcn_rcp(x);
    double e = fma(-x, r, 1.0);
    r = fma(r, e, r);
    e = fma(-x, r, 1.0);
    return fma(r, e, r);
}

struct FPar2 {
    double a, b, gamma;      // advection velocity (a, b); ideal-gas gamma
};

template <int FLUX> struct Flux2D;

template <> struct Flux2D<OECDG_FLUX_ADVECTION> {
    static constexpr int NC = 1;
    __device__ static inline void both(const double *w, double *f1, double *f2, const FPar2 &p) {
        f1[0] = p.a * w[0];
        f2[0] = p.b * w[0];
    }
    // flux along direction dir (0 = x, 1 = y)
    __device__ static inline void one(int dir, const double *w, double *o, const FPar2 &p) {
        o[0] = (dir ? p.b : p.a) * w[0];
    }
    __device__ static inline void speeds(const double *, double &x, double &y, const FPar2 &p) {
        x = fabs(p.a);
        y = fabs(p.b);
    }
    __device__ static inline bool physical(const double *, const FPar2 &) { return true; }
};

template <> struct Flux2D<OECDG_FLUX_EULER> {
    static constexpr int NC = 4;    // rho, rho u, rho v, E
    __device__ static inline void both(const double *w, double *f1, double *f2, const FPar2 &p) {
        const double ir = rcp_nr(w[0]);
        const double u = w[1] * ir, v = w[2] * ir;
        const double pr = (p.gamma - 1.0) * (w[3] - 0.5 * (w[1] * u + w[2] * v));
        const double H = w[3] + pr;
        f1[0] = w[1];
        f1[1] = w[1] * u + pr;
        f1[2] = w[2] * u;
        f1[3] = H * u;
        f2[0] = w[2];
        f2[1] = w[1] * v;
        f2[2] = w[2] * v + pr;
        f2[3] = H * v;
    }
    __device__ static inline void one(int dir, const double *w, double *o, const FPar2 &p) {
        const double ir = rcp_nr(w[0]);
        const double pr = (p.gamma - 1.0) * (w[3] - 0.5 * (w[1] * w[1] + w[2] * w[2]) * ir);
        const double un = (dir ? w[2] : w[1]) * ir;
        o[0] = dir ? w[2] : w[1];
        o[1] = w[1] * un + (dir ? 0.0 : pr);
        o[2] = w[2] * un + (dir ? pr : 0.0);
        o[3] = (w[3] + pr) * un;
    }
    // spectral radii of f_1' and f_2'
    __device__ static inline void speeds(const double *w, double &x, double &y, const FPar2 &p) {
        const double ir = 1.0 / w[0];
        const double u = w[1] * ir, v = w[2] * ir;
        const double pr = (p.gamma - 1.0) * (w[3] - 0.5 * (w[1] * u + w[2] * v));
        const double c = sqrt(p.gamma * pr * ir);
        x = fabs(u) + c;
        y = fabs(v) + c;
    }
    __device__ static inline bool physical(const double *w, const FPar2 &p) {
        if (!(w[0] > 0.0)) return false;
        const double pr = (p.gamma - 1.0) * (w[3] - 0.5 * (w[1] * w[1] + w[2] * w[2]) / w[0]);
        return pr > 0.0;
    }
};

// ---------------------------------------------------------------- tables ---

template <int K>
struct Tab2 {
    static constexpr int K1 = K + 1, Q = K + 1, NSP = 2 * K + 4;
    double w[Q];                  // Gauss-Legendre weights on [-1, 1]
    double own[K1][2][Q][K1];     // [d][half][g][n]: P_n^(d) at node g of the half, own coordinate
    double nb[K1][2][Q][K1];      // the same point in the overlapping cell's coordinate (+1 / -1)
    double e1[K1][K1];            // [d][n]: P_n^(d)(1)
    double e0[K1][K1];            // [d][n]: P_n^(d)(0)
    double sp[NSP][K1];           // P_n at the sigma sample points (-1, half nodes, +1)
    double cdel[K1];              // (2m+1) / ((2K-1) m!)
    double sh[2][K1][K1];         // [half][n][m]: P_n(x + 1) (half 0) or P_n(x - 1) (half 1) = sum_m sh P_m(x)
};

template <int K>
constexpr Tab2<K> make_tab2() {
    Tab2<K> t{};
    constexpr int K1 = K + 1, Q = K + 1;
    constexpr auto g = ct::gauss<Q>();
    // weights whose sum is 2 exactly (a constant state stays one, and the averages'
    // sum changes by rounding errors of both signs only)
    for (int i = 0; i < Q; ++i) t.w[i] = Q == 2 ? 1.0 : (Q == 3 ? (i == 1 ? 8.0 / 9.0 : 5.0 / 9.0) : g.w[1]);
    if (Q == 4) t.w[0] = t.w[3] = 1.0 - g.w[1];
    for (int d = 0; d < K1; ++d)
        for (int hf = 0; hf < 2; ++hf)
            for (int i = 0; i < Q; ++i) {
                const double xi = hf == 0 ? 0.5 * (g.s[i] - 1.0) : 0.5 * (g.s[i] + 1.0);
                const double xn = hf == 0 ? xi + 1.0 : xi - 1.0;
                for (int n = 0; n < K1; ++n) {
                    t.own[d][hf][i][n] = ct::legd(n, d, xi);
                    t.nb[d][hf][i][n] = ct::legd(n, d, xn);
                }
            }
    for (int d = 0; d < K1; ++d)
        for (int n = 0; n < K1; ++n) {
            t.e1[d][n] = ct::legd(n, d, 1.0);
            t.e0[d][n] = ct::legd(n, d, 0.0);
        }
    double pts[2 * K + 4] = {};
    pts[0] = -1.0;
    for (int i = 0; i < Q; ++i) pts[1 + i] = 0.5 * (g.s[i] - 1.0);
    for (int i = 0; i < Q; ++i) pts[1 + Q + i] = 0.5 * (g.s[i] + 1.0);
    pts[2 * K + 3] = 1.0;
    for (int j = 0; j < 2 * K + 4; ++j)
        for (int n = 0; n < K1; ++n) t.sp[j][n] = ct::leg(n, pts[j]);
    double fact = 1.0;
    for (int m = 0; m < K1; ++m) {
        if (m > 1) fact *= m;
        t.cdel[m] = K > 0 ? (2.0 * m + 1.0) / ((2.0 * K - 1.0) * fact) : 0.0;
    }
    for (int n = 0; n < K1; ++n) {
        ct::Poly p = ct::shifted(ct::legpoly(n));                      // P_n(x - 1) in monomials
        for (int m = n; m >= 0; --m) {                                 // highest power first: c_m / lead(P_m)
            const ct::Poly l = ct::legpoly(m);
            const ct::Rat c = ct::rmul(p.c[m], ct::rat(l.c[m].q, l.c[m].p));
            for (int j = 0; j <= m; ++j) p.c[j] = ct::radd(p.c[j], ct::rmul(ct::rat(-c.p, c.q), l.c[j]));
            t.sh[1][n][m] = (double)c.p / (double)c.q;
            t.sh[0][n][m] = ((n + m) & 1) ? -t.sh[1][n][m] : t.sh[1][n][m];   // P_n(x+1) = (-1)^n P_n(-x-1)
        }
    }
    return t;
}

// ------------------------------------------------------- device structs ---

// Global scalars of the current stage (written by k_reduce2d).
struct Stats2 {
    double isig[2][4];            // recip_sigma of sigma, per mesh and component
    int small;                    // whether one of them is of a subnormal sigma
    double bx, by;                // largest x / y wave speeds at cell averages (both meshes)
    double t;                     // start time of the current step
    double tau, tau_max;          // the current step
    double fx, fy, ratio;         // its 2 tau_max / h_x, 2 tau_max / h_y and tau / tau_max
    double tau_damp;              // tau of the OE step applied to the next tile kernel's input
    long long nexec;              // completed steps
    int pending, last, bad;       // bad: no admissible time step
    int done[2];                  // the run has ended, by the parity of the stage index: the reduction for the
                                  // next stage writes its entry while k_delta2d of this one reads the other
};

enum { R2_STEP = 0, R2_STAGE = 1, R2_FINAL = 2, R2_SINGLE = 3, R2_STATS = 4 };

struct Stage2Args {
    int nx, ny, ntx, nty;
    long long plane;              // nx * ny
    double hx, hy;
    FPar2 fp;
    const double *inC, *inD;      // tile input (pre-damping, or damped when damp == 0)
    double *outC, *outD;          // stage output (undamped) or damped state (final mode)
    const double *unC, *unD;      // u^n as the step's first stage read it (stages l > 0)
    double *facC, *facD;          // its damping factors [K][ny][nx]: written at stage 0, read later (null: undamped)
    double *part;                 // partial statistics, a record (Rec2) per wave of primal and of dual cells
    double *numC, *numD;          // damping numerators [m*NC + q][ny][nx]: written by k_delta2d, read by k_stage2d
    double *AC, *AD;              // classical RK4: weighted sum of the damped inputs of stages 1 and 2
    const Stats2 *st;
    int *err;                     // [0] non-finite, [1] non-physical, [2] no admissible step
    int l, gpar, damp;            // stage, parity of the stage index (st->done), OE on the input
    int nred;                     // k_delta2d: leading workgroups that reduce the statistics (reduce2d)
    RKStage rs;                   // c/d coefficients of stage l of the RK method (eq:RKCDG)
};

// Reduction of the partial records into the global scalars.
struct Red2Args {
    const double *part;
    int nrec, per, nb, mode;      // records, records per workgroup, workgroups
    int gpar;                     // parity of the stage index that the result is for
    long long ncell;
    double t_end, dt_fixed, cfl, hx, hy;
    double tau_o, taumax_o;       // single-stage call
    double *fold;                 // [nb][Rec2::N]
    unsigned *count;              // workgroups that have written their record (0 between launches)
    Stats2 *st;
    int *err;
};

// A partial record: per mesh (sum of averages, max, min of the samples) of each
// component, then the largest x and y wave speeds.
template <int NC> struct Rec2 {
    static constexpr int NM = 3 * NC + 2, N = 2 * NM;
    static constexpr int G = NC == 4 ? 32 : 16;   // threads of a record (the first N of them hold a value)
    static_assert(N <= G, "a thread per value");
    __device__ static inline int kind(int j) { return j % NM < 3 * NC ? j % NM % 3 : 1; }
};

// ------------------------------------------------------------ helpers ---

// Tile of a workgroup; a band of consecutive tiles per XCD (xcd_tile).
__device__ inline int tile_of_block(int nt) { return xcd_tile(blockIdx.x, nt); }

// sqrt(x) for finite x > 0 from the hardware estimate r of 1/sqrt (relative error
// below 2^-22, of subnormal x too) and one third-order step: with t = x r and
// e = 1 - t r, sqrt(x) = t (1 - e)^(-1/2) = t + t e (1/2 + 3/8 e + O(e^2)), within an ulp
// of the correctly rounded root.  The IEEE sequence (range scaling, three steps,
// class checks) was 40 % of k_delta2d.  0 and infinity give NaN: a sum under the root
// begins with SQRT_TINY, the smallest double, whose root is 2^-537 exactly, and
// edge_norms takes the roots of sums that were 0, and the NaN of infinite ones, out of
// its results.
constexpr double SQRT_TINY = 0x1p-1074;
__device__ inline double sqrt_nr(double x) {
    const double r = __builtin_amdgcn_rsq(x);
    const double t = x * r;
    const double e = fma(-t, r, 1.0);
    return fma(t * e, fma(e, 0.375, 0.5), t);
}

// c x + y and c x for a constant c: no multiplication by 1 (the compiler may not
// drop an addition of 0 or a product that it has to round).
__device__ inline double mad_c(double c, double x, double y) { return c == 1.0 ? x + y : fma(c, x, y); }
__device__ inline double mul_c(double c, double x) { return c == 1.0 ? x : c * x; }

// x with its sign bit flipped by mask (0 or 0x80000000).
__device__ inline double flip_sign(double x, unsigned mask) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
    return __builtin_bit_cast(double, b ^ ((unsigned long long)mask << 32));
}

__device__ inline int wrap_idx(int i, int n, bool small) {
    if (small) return ((i % n) + n) % n;
    return i < 0 ? i + n : (i >= n ? i - n : i);
}

// PK: the total-degree space P^K.  Modes with a + b > K are zero in every
// state, so the unrolled loops skip them at compile time.
template <int K, bool PK>
__host__ __device__ constexpr bool kept(int a, int b) { return !PK || a + b <= K; }
// Modes per component that are kept, and the place of mode (a, b) among them.
template <int K, bool PK>
__host__ __device__ constexpr int kept_modes() { return PK ? (K + 1) * (K + 2) / 2 : (K + 1) * (K + 1); }
template <int K, bool PK>
__host__ __device__ constexpr int kept_index(int a, int b) {
    int n = 0;
    for (int i = 0; i < a; ++i)
        for (int j = 0; j <= K; ++j) n += kept<K, PK>(i, j);
    for (int j = 0; j < b; ++j) n += kept<K, PK>(a, j);
    return n;
}

// The damping numerators N^m_q of global cell g of a mesh.
template <int K, int NC>
__device__ inline void load_numerators(const double *__restrict__ N, long long plane, long long g,
                                       double (&nv)[(K + 1) * NC]) {
    const double *p = N + g;
#pragma unroll
    for (int e = 0; e < (K + 1) * NC; ++e, p += plane) nv[e] = *p;
}

// Damping factors exp(-tau sum_{m<=j} delta^m), j = 1..K, of a cell of a mesh,
// delta^m = max_q N^m_q / sigma_q.
template <int K, int NC>
__device__ inline void damp_factors(const double (&nv)[(K + 1) * NC], const Stats2 *__restrict__ st, int mesh,
                                    double (&f)[K]) {
    double isig[NC], tau = st->tau_damp;
#pragma unroll
    for (int q = 0; q < NC; ++q) isig[q] = st->isig[mesh][q];
    if (st->small) scale_small(isig, tau);
    double S = 0.0;
#pragma unroll
    for (int m = 0; m <= K; ++m) {
        double dm = 0.0;                         // (drops a NaN: the wave speed of a cell of negative pressure)
#pragma unroll
        for (int q = 0; q < NC; ++q) dm = max_d(dm, nv[m * NC + q] * fabs(isig[q]));
        S += dm;
        if (m >= 1) f[m - 1] = exp(-tau * S);
    }
}

// ----------------------------------------------------------- stage kernel ---

// Largest and smallest value of one component over S x S, S = {+-1, +-nodes}:
// in each direction the even and the odd part at +x give the values at +x and
// -x, whose larger and smaller are even +- |odd|.
template <int K, bool PK>
__device__ inline void sample_extrema(const double (&u)[K + 1][K + 1], double &mx, double &mn) {
    constexpr int K1 = K + 1, NSP = 2 * K + 4;
    constexpr Tab2<K> tb = make_tab2<K>();
    mx = -INFINITY;
    mn = INFINITY;
#pragma unroll
    for (int i = K + 2; i < NSP; ++i) {          // the sample points x > 0
        double rp[K1], rm[K1];
#pragma unroll
        for (int j = 0; j < K1; ++j) {
            double ev = 0.0, od = 0.0;
#pragma unroll
            for (int c = 0; c < K1; ++c) {
                if (!kept<K, PK>(c, j)) continue;
                if (c & 1) od = fma(u[c][j], tb.sp[i][c], od);
                else ev = c == 0 ? u[c][j] : fma(u[c][j], tb.sp[i][c], ev);
            }
            rp[j] = ev + od;
            rm[j] = ev - od;
        }
#pragma unroll
        for (int y = K + 2; y < NSP; ++y)
#pragma unroll
            for (int sg = 0; sg < 2; ++sg) {
                const double *b = sg ? rm : rp;
                double ev = b[0], hi, lo;
#pragma unroll
                for (int j = 2; j < K1; j += 2) ev = mad_c(tb.sp[y][j], b[j], ev);
                if constexpr (K1 < 4) {          // one odd mode: |od| = y |b_1|
                    hi = fma(tb.sp[y][1], fabs(b[1]), ev);
                    lo = fma(-tb.sp[y][1], fabs(b[1]), ev);
                } else {
                    const double od = fma(b[3], tb.sp[y][3], b[1] * tb.sp[y][1]);
                    hi = ev + fabs(od);
                    lo = ev - fabs(od);
                }
                mx = max_d(mx, hi);
                mn = min_d(mn, lo);
            }
        __builtin_amdgcn_sched_barrier(0);       // one line of samples at a time: bounds the live registers
    }
}

// Partial record of a wave's cells of mesh `mesh` (valid: this lane holds one)
// from its first lane's view: u(q) gives the modes of component q, ub the cell
// averages.  Lane 63 writes the mesh's half of the record.  Every lane takes part.
template <int K, int FLUX, bool PK, class U>
__device__ inline void wave_record(const Stage2Args &a, int mesh, bool valid, U &&u, double *rec) {
    using F = Flux2D<FLUX>;
    constexpr int NC = F::NC, K1 = K + 1, NM = Rec2<NC>::NM;
    double v[NM], ub[NC];
#pragma unroll
    for (int q = 0; q < NC; ++q) {
        double m[K1][K1], mx, mn;
        u(q, m);
        sample_extrema<K, PK>(m, mx, mn);
        ub[q] = valid ? m[0][0] : 1.0;
        v[3 * q] = wave_reduce(0, valid ? m[0][0] : 0.0);
        v[3 * q + 1] = wave_reduce(1, valid ? mx : -INFINITY);
        v[3 * q + 2] = wave_reduce(2, valid ? mn : INFINITY);
    }
    double bx, by;
    F::speeds(ub, bx, by, a.fp);
    v[3 * NC] = wave_reduce(1, valid ? bx : -INFINITY);
    v[3 * NC + 1] = wave_reduce(1, valid ? by : -INFINITY);
    if (valid && !F::physical(ub, a.fp)) a.err[1] = 1;
    if (threadIdx.x % WAVE == WAVE - 1) {
#pragma unroll
        for (int j = 0; j < NM; ++j) rec[mesh * NM + j] = v[j];
    }
}

// Cells of a tile that its operator reads, per mesh: (TX+1) x (TY+1), primal
// i0-1 .. i0+TX-1, dual i0 .. i0+TX (rows likewise).  In these indices an owned
// cell of either mesh at (s, r) overlaps the other mesh's cells s..s+1, r..r+1.
template <int TX, int TY>
struct Halo2 {
    static constexpr int W = TX + 1, H = TY + 1, N = W * H;
};

// Doubles of a cell in LDS: its entries one after another (an entry is then at a
// constant offset from the cell's address), to an odd stride, which spreads the
// cells of a wave over the banks.
__host__ __device__ constexpr int lds_stride(int ne) { return ne | 1; }
// Threads of a stage workgroup: whole waves of primal and of dual cells.
__host__ __device__ constexpr int mesh_threads(int tx, int ty) { return (tx * ty + 63) / 64 * 64; }

// Table entries of Gauss node p of the upper half, for a loop over the nodes.
template <int K>
struct NodeTab {
    double w, nb[K + 1], p[K + 1], dp[K + 1];    // weight; P_n of the overlapping cell; P_n and P_n' of the own cell
};
template <int K>
struct NodeTabs {
    NodeTab<K> t[K + 1];
};
template <int K>
constexpr NodeTabs<K> make_node_tabs() {
    constexpr Tab2<K> tb = make_tab2<K>();
    NodeTabs<K> r{};
    for (int p = 0; p <= K; ++p) {
        r.t[p].w = tb.w[p];
        for (int n = 0; n <= K; ++n) {
            r.t[p].nb[n] = tb.nb[0][1][p][n];
            r.t[p].p[n] = tb.own[0][1][p][n];
            r.t[p].dp[n] = tb.own[1][1][p][n];
        }
    }
    return r;
}
template <int K>
__constant__ constexpr NodeTabs<K> node_tabs = make_node_tabs<K>();
template <int K>
__device__ inline NodeTab<K> node_tab(int p) { return node_tabs<K>.t[p]; }

// Coupling and volume terms of eq:2D_H for one owned cell: R[q][a][b] = their
// integral against P_a P_b (own-cell part of the coupling left to the caller), times
// 16 tau_max / (h_x h_y): the coupling then has no factor but the weights.  (With
// 1 / tau_max, the area and the inverse mass as factors their roundings, which are the
// same in every cell and stage, added up: the sum of the averages drifted by up to 2e-14
// in 120 stages, where it now keeps to 5e-16.)  From the damped cells of the other mesh in LDS
// (oth, lds_stride apart).
//
// A quadrant (sx, sy) is evaluated in its mirror image on the upper right one.
// With P_n(-x) = (-1)^n P_n(x) and the symmetric Gauss rule, mirroring x turns a
// mode a into (-1)^a times itself and the x momentum into its negative, and the
// mirrored state obeys the same equations; so all quadrants use the same
// compile-time tables, and only signs of the loaded modes (flip_sign) and, where
// the quadrant loop crosses an axis, of the sums R change.
template <int K, int FLUX, int TX, int TY, bool PK>
__device__ inline void volume2d(const Stage2Args &a, const double *oth, int s, int r, double sxx, double syy,
                                double (&R)[Flux2D<FLUX>::NC][K + 1][K + 1]) {
    using F = Flux2D<FLUX>;
    constexpr int NC = F::NC, K1 = K + 1, Q = K + 1, NM = kept_modes<K, PK>();
    constexpr int W = Halo2<TX, TY>::W, LS = lds_stride(NC * NM);
    constexpr Tab2<K> tb = make_tab2<K>();
#pragma unroll
    for (int q = 0; q < NC; ++q)
#pragma unroll
        for (int i = 0; i < K1; ++i)
#pragma unroll
            for (int j = 0; j < K1; ++j) R[q][i][j] = 0.0;

    // component q of a mirrored state changes sign along x (y) if it is the x (y) momentum
    constexpr auto vecx = [](int q) { return NC == 4 && q == 1; };
    constexpr auto vecy = [](int q) { return NC == 4 && q == 2; };
    // quadrants (0,0), (1,0), (1,1), (0,1): one axis is crossed each time
#pragma unroll 1
    for (int qd = 0; qd < 4; ++qd) {
        const int sy = qd >> 1, sx = (qd ^ sy) & 1;
        const unsigned mx = sx ? 0u : 0x80000000u, my = sy ? 0u : 0x80000000u;
        const unsigned cx = (qd & 1) ? 0x80000000u : 0u, cy = qd == 2 ? 0x80000000u : 0u;
#pragma unroll
        for (int q = 0; q < NC; ++q)
#pragma unroll
            for (int i = 0; i < K1; ++i)
#pragma unroll
                for (int j = 0; j < K1; ++j) {
                    if (!kept<K, PK>(i, j)) continue;
                    const bool ox = (i & 1) != (int)vecx(q), oy = (j & 1) != (int)vecy(q);
                    if (ox || oy) R[q][i][j] = flip_sign(R[q][i][j], (ox ? cx : 0u) ^ (oy ? cy : 0u));
                }
        const double *o = oth + ((r + sy) * W + s + sx) * LS;
        FPar2 fp = a.fp;
        if constexpr (NC == 1) {                 // advection: the mirrored velocity
            fp.a = flip_sign(fp.a, mx);
            fp.b = flip_sign(fp.b, my);
        }
        double d[NC][K1][K1];                    // the overlapping cell's modes, mirrored
#pragma unroll
        for (int q = 0; q < NC; ++q)
#pragma unroll
            for (int c = 0; c < K1; ++c)
#pragma unroll
                for (int e = 0; e < K1; ++e) {
                    d[q][c][e] = 0.0;
                    if (!kept<K, PK>(c, e)) continue;
                    const double x = o[q * NM + kept_index<K, PK>(c, e)];
                    const bool ox = (c & 1) != (int)vecx(q), oy = (e & 1) != (int)vecy(q);
                    d[q][c][e] = (ox || oy) ? flip_sign(x, (ox ? mx : 0u) ^ (oy ? my : 0u)) : x;
                }
        // One node in x at a time, a loop at run time (its table entries are
        // uniform loads): unrolled, the live values pass 256 registers.
#pragma unroll 1
        for (int p = 0; p < Q; ++p) {
            const NodeTab<K> nt = node_tab<K>(p);
            double cxv[NC][K1];                  // the line x = node p, modes in y
#pragma unroll
            for (int q = 0; q < NC; ++q)
#pragma unroll
                for (int e = 0; e < K1; ++e) {
                    double t = d[q][0][e];
#pragma unroll
                    for (int c = 1; c < K1; ++c)
                        if (kept<K, PK>(c, e)) t = fma(d[q][c][e], nt.nb[c], t);
                    cxv[q][e] = t;
                }
            // A_j: coupling and y flux against P_j(y), P_j'(y); B_j: x flux against P_j(y)
            double A[NC][K1], B[NC][K1];
#pragma unroll
            for (int q = 0; q < NC; ++q)
#pragma unroll
                for (int j = 0; j < K1; ++j) A[q][j] = B[q][j] = 0.0;
#pragma unroll
            for (int g = 0; g < Q; ++g) {
                double w[NC], f1[NC], f2[NC];
#pragma unroll
                for (int q = 0; q < NC; ++q) {
                    double t = cxv[q][0];
#pragma unroll
                    for (int e = 1; e < K1; ++e) t = fma(cxv[q][e], tb.nb[0][1][g][e], t);
                    w[q] = t;
                }
                F::both(w, f1, f2, fp);
                const double wd = tb.w[g] * syy;
#pragma unroll
                for (int q = 0; q < NC; ++q)
#pragma unroll
                    for (int j = 0; j < K1; ++j) {
                        A[q][j] = fma(tb.w[g] * tb.own[0][1][g][j], w[q], A[q][j]);
                        if (j > 0) A[q][j] = fma(wd * tb.own[1][1][g][j], f2[q], A[q][j]);
                        B[q][j] = fma(tb.w[g] * tb.own[0][1][g][j], f1[q], B[q][j]);
                    }
            }
            const double wpx = nt.w * sxx;
#pragma unroll
            for (int q = 0; q < NC; ++q)
#pragma unroll
                for (int i = 0; i < K1; ++i)
#pragma unroll
                    for (int j = 0; j < K1; ++j) {
                        if (!kept<K, PK>(i, j)) continue;
                        R[q][i][j] = fma(nt.w * nt.p[i], A[q][j], R[q][i][j]);
                        if (i > 0) R[q][i][j] = fma(wpx * nt.dp[i], B[q][j], R[q][i][j]);
                    }
        }
    }
    // the loop ends in the frame of quadrant (0, 1): back across x
#pragma unroll
    for (int q = 0; q < NC; ++q)
#pragma unroll
        for (int i = 0; i < K1; ++i)
#pragma unroll
            for (int j = 0; j < K1; ++j)
                if (kept<K, PK>(i, j) && (i & 1) != (int)vecx(q)) R[q][i][j] = -R[q][i][j];

}

// Edge terms of eq:2D_H added to R, scaled like it: f_dir of the other mesh on its centre line
// along each half-edge of direction dir; the W (S) edge is mirrored onto the E (N)
// edge as above, the halves have tables of their own.
template <int K, int FLUX, int TX, int TY, bool PK>
__device__ inline void edges2d(const Stage2Args &a, const double *oth, int s, int r, double sxx, double syy,
                               double (&R)[Flux2D<FLUX>::NC][K + 1][K + 1]) {
    using F = Flux2D<FLUX>;
    constexpr int NC = F::NC, K1 = K + 1, Q = K + 1, NM = kept_modes<K, PK>();
    constexpr int W = Halo2<TX, TY>::W, LS = lds_stride(NC * NM);
    constexpr Tab2<K> tb = make_tab2<K>();
#pragma unroll
    for (int dir = 0; dir < 2; ++dir) {
        constexpr auto vecn = [](int dr, int q) { return NC == 4 && q == 1 + dr; };   // momentum normal to the edge
        const double ht = -2.0 * (dir ? syy : sxx);
#pragma unroll 1
        for (int side = 0; side < 2; ++side) {
            const unsigned fn = side ? 0u : 0x80000000u;
            FPar2 fp = a.fp;
            if constexpr (NC == 1) {
                fp.a = flip_sign(fp.a, fn);
                fp.b = flip_sign(fp.b, fn);
            }
            double Y[NC][K1];
#pragma unroll
            for (int q = 0; q < NC; ++q)
#pragma unroll
                for (int t = 0; t < K1; ++t) Y[q][t] = 0.0;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const double *o = oth + (dir ? (r + side) * W + s + h : (r + h) * W + s + side) * LS;
                double l[NC][K1];
#pragma unroll
                for (int q = 0; q < NC; ++q)
#pragma unroll
                    for (int t = 0; t < K1; ++t) {
                        double sum = 0.0;
#pragma unroll
                        for (int n = 0; n < K1; n += 2) {             // P_n(0) = 0 for odd n
                            if (!kept<K, PK>(t, n)) continue;
                            const double x = o[q * NM + (dir ? kept_index<K, PK>(t, n) : kept_index<K, PK>(n, t))];
                            sum = n == 0 ? x : fma(x, tb.e0[0][n], sum);
                        }
                        l[q][t] = vecn(dir, q) ? flip_sign(sum, fn) : sum;
                    }
#pragma unroll
                for (int g = 0; g < Q; ++g) {
                    double w[NC], f[NC];
#pragma unroll
                    for (int q = 0; q < NC; ++q) {
                        double t = l[q][0];
#pragma unroll
                        for (int e = 1; e < K1; ++e) t = fma(l[q][e], tb.nb[0][h][g][e], t);
                        w[q] = t;
                    }
                    F::one(dir, w, f, fp);
#pragma unroll
                    for (int q = 0; q < NC; ++q)
#pragma unroll
                        for (int t = 0; t < K1; ++t)
                            Y[q][t] = fma(tb.w[g] * tb.own[0][h][g][t], f[q], Y[q][t]);
                }
                __builtin_amdgcn_sched_barrier(0);   // one half-edge at a time: bounds the live registers
            }
            // P_n(1) = 1; out of the frame of the side
#pragma unroll
            for (int q = 0; q < NC; ++q)
#pragma unroll
                for (int t = 0; t < K1; ++t) {
                    const double y = ht * Y[q][t], z = flip_sign(y, fn);
#pragma unroll
                    for (int n = 0; n < K1; ++n) {
                        if (!kept<K, PK>(n, t)) continue;
                        const double x = (n & 1) != (int)vecn(dir, q) ? z : y;
                        if (dir) R[q][t][n] += x;
                        else R[q][n][t] += x;
                    }
                }
        }
    }
}

// One RK stage (see the top of the file).  WPS waves per SIMD, no more: a fifth wave of
// the advection kernels, whose registers allow it, costs more in the caches than it
// hides (P3 at 512^2, three steps of RK4: 1409 us with five, 1366 with four).
template <int K, int FLUX, int TX, int TY, int WPS, bool PK>
__global__ __launch_bounds__(2 * mesh_threads(TX, TY)) __attribute__((amdgpu_waves_per_eu(WPS, WPS))) void k_stage2d(Stage2Args a) {
    using F = Flux2D<FLUX>;
    constexpr int NC = F::NC, K1 = K + 1, NM = kept_modes<K, PK>(), NE = NC * NM, LS = lds_stride(NE);
    constexpr int W = Halo2<TX, TY>::W, NCELL = Halo2<TX, TY>::N, MT = mesh_threads(TX, TY), NT = 2 * MT;
    __shared__ double tile[2 * NCELL * LS];      // [mesh][cell][entry], damped

    const int tid = threadIdx.x;
    const int tileid = tile_of_block(a.ntx * a.nty);
    const int i0 = (tileid % a.ntx) * TX, j0 = (tileid / a.ntx) * TY;
    const Stats2 *st = a.st;
    if (st->done[a.gpar]) return;

    // the tile's cells into LDS, damped on the way: a cell of either mesh per
    // thread, and the cells beyond the threads shared by the waves, PART entries
    // each.  Every load is issued before the first wait.
    constexpr int REST = 2 * NCELL - NT, PARTS = NC == 4 ? (NT >= 4 * WAVE ? 4 : 2) : 1, PART = NE / PARTS;
    static_assert(REST > 0 && REST <= WAVE && NT / WAVE >= PARTS, "one more cell per lane");
    const bool small = a.nx <= TX || a.ny <= TY;
    const int wave = tid / WAVE, lane = tid % WAVE;
    struct Cell {
        int mesh, cell;
        long long g;
    };
    auto cell_of = [&](int c) {
        Cell t;
        t.mesh = c >= NCELL;
        t.cell = c - t.mesh * NCELL;
        const int gx = wrap_idx(i0 - 1 + t.mesh + t.cell % W, a.nx, small);
        const int gy = wrap_idx(j0 - 1 + t.mesh + t.cell / W, a.ny, small);
        t.g = (long long)gy * a.nx + gx;
        return t;
    };
    const Cell c0 = cell_of(tid), c1 = cell_of(NT + (lane < REST ? lane : 0));
    const bool more = lane < REST && wave < PARTS;
    const int q1 = more ? wave * (NC / PARTS) : 0;           // first component of this wave's part
    double v0[NE], v1[PART], n0[K1 * NC], n1[K1 * NC];
    {
        const double *p = (c0.mesh ? a.inD : a.inC) + c0.g;
#pragma unroll
        for (int q = 0; q < NC; ++q)
#pragma unroll
            for (int i = 0; i < K1; ++i)
#pragma unroll
                for (int j = 0; j < K1; ++j, p += a.plane)
                    if (kept<K, PK>(i, j)) v0[q * NM + kept_index<K, PK>(i, j)] = *p;
    }
    if (more) {
        const double *p = (c1.mesh ? a.inD : a.inC) + c1.g + (long long)q1 * K1 * K1 * a.plane;
#pragma unroll
        for (int q = 0; q < NC / PARTS; ++q)
#pragma unroll
            for (int i = 0; i < K1; ++i)
#pragma unroll
                for (int j = 0; j < K1; ++j, p += a.plane)
                    if (kept<K, PK>(i, j)) v1[q * NM + kept_index<K, PK>(i, j)] = *p;
    }
    if (a.damp) {
        load_numerators<K, NC>(c0.mesh ? a.numD : a.numC, a.plane, c0.g, n0);
        if (more) load_numerators<K, NC>(c1.mesh ? a.numD : a.numC, a.plane, c1.g, n1);
    }
    {
        double f[K];
        if (a.damp) {
            damp_factors<K, NC>(n0, st, c0.mesh, f);
#pragma unroll
            for (int q = 0; q < NC; ++q)
#pragma unroll
                for (int i = 0; i < K1; ++i)
#pragma unroll
                    for (int j = 0; j < K1; ++j)
                        if (kept<K, PK>(i, j) && i + j > 0)
                            v0[q * NM + kept_index<K, PK>(i, j)] *= f[(i + j < K ? i + j : K) - 1];
        }
        double *o = tile + (c0.mesh * NCELL + c0.cell) * LS;
#pragma unroll
        for (int e = 0; e < NE; ++e) o[e] = v0[e];
    }
    if (more) {
        double f[K];
        if (a.damp) {
            damp_factors<K, NC>(n1, st, c1.mesh, f);
#pragma unroll
            for (int q = 0; q < NC / PARTS; ++q)
#pragma unroll
                for (int i = 0; i < K1; ++i)
#pragma unroll
                    for (int j = 0; j < K1; ++j)
                        if (kept<K, PK>(i, j) && i + j > 0)
                            v1[q * NM + kept_index<K, PK>(i, j)] *= f[(i + j < K ? i + j : K) - 1];
        }
        double *o = tile + (c1.mesh * NCELL + c1.cell) * LS + q1 * NM;
#pragma unroll
        for (int e = 0; e < PART; ++e) o[e] = v1[e];
    }
    __syncthreads();

    // owned cells: the first half of the threads primal, the second dual (threads
    // beyond the tile's cells take cell 0 along and store nothing)
    const int mesh = tid >= MT, rr = tid - mesh * MT < TX * TY ? tid - mesh * MT : 0;
    const int s = rr % TX, r = rr / TX;
    const int gx = i0 + s, gy = j0 + r;
    const bool valid = tid - mesh * MT < TX * TY && gx < a.nx && gy < a.ny;
    const long long gofs = valid ? (long long)gy * a.nx + gx : 0;
    const double *own = tile + (mesh * NCELL + (r + 1 - mesh) * W + s + 1 - mesh) * LS;
    const double sxx = st->fx, syy = st->fy;
    const double *oth = tile + (1 - mesh) * NCELL * LS;
    double R[NC][K1][K1];
    volume2d<K, FLUX, TX, TY, PK>(a, oth, s, r, sxx, syy, R);
    // u^n and its factors, asked for before the edges, which leave the registers for
    // them.  The undamped u^n is still there (the last stage overwrites it, each
    // cell by its own thread) and is damped again: K factors are stored instead of
    // the damped state.
    const double *UM = (mesh ? a.unD : a.unC) + gofs;
    double *OM = (mesh ? a.outD : a.outC) + gofs, *AM = (mesh ? a.AD : a.AC) + gofs;
    double *FM = a.facC ? (mesh ? a.facD : a.facC) + gofs : nullptr;
    double base[NC][K1][K1], fn[K];              // u^n
#pragma unroll
    for (int j = 0; j < K; ++j) fn[j] = 1.0;
#pragma unroll
    for (int q = 0; q < NC; ++q)
#pragma unroll
        for (int i = 0; i < K1; ++i)
#pragma unroll
            for (int j = 0; j < K1; ++j) base[q][i][j] = 0.0;
    if (a.l > 0) {                               // (lanes without a cell read cell 0)
        const double *p = UM;
#pragma unroll
        for (int q = 0; q < NC; ++q)
#pragma unroll
            for (int i = 0; i < K1; ++i)
#pragma unroll
                for (int j = 0; j < K1; ++j, p += a.plane)
                    if (kept<K, PK>(i, j)) base[q][i][j] = *p;
        if (FM) {
#pragma unroll
            for (int j = 0; j < K; ++j) fn[j] = FM[j * a.plane];
        }
    }
    edges2d<K, FLUX, TX, TY, PK>(a, oth, s, r, sxx, syy, R);
    double cn = a.rs.cn;
    if (FM && a.l > 0) {
#pragma unroll
        for (int q = 0; q < NC; ++q)
#pragma unroll
            for (int i = 0; i < K1; ++i)
#pragma unroll
                for (int j = 0; j < K1; ++j)
                    if (kept<K, PK>(i, j) && i + j > 0) base[q][i][j] *= fn[(i + j < K ? i + j : K) - 1];
    }
    if (a.rs.acc_read) {                         // classical RK4's last stage: the accumulated earlier stages
        const double *p = AM;
#pragma unroll
        for (int q = 0; q < NC; ++q)
#pragma unroll
            for (int i = 0; i < K1; ++i)
#pragma unroll
                for (int j = 0; j < K1; ++j, p += a.plane)
                    if (kept<K, PK>(i, j)) base[q][i][j] = fma(cn, base[q][i][j], *p);
        cn = 1.0;
    }

    // own part of the coupling, mass inverse, RK combination:
    // c_{ll} u + tau d_{ll} L = (c_{ll} - lam) u + lam (R scaled), lam = d_{ll} tau / tau_max
    const double lam = a.rs.d * st->ratio, own_c = a.rs.cw - lam;
    double bad = 0.0;                            // 0 times every output: 0, or NaN if one is not finite
    double *po = OM;
#pragma unroll
    for (int q = 0; q < NC; ++q)
#pragma unroll
        for (int i = 0; i < K1; ++i)
#pragma unroll
            for (int j = 0; j < K1; ++j, po += a.plane) {
                if (!kept<K, PK>(i, j)) {
                    if (valid) *po = 0.0;
                    continue;
                }
                const double s0 = own[q * NM + kept_index<K, PK>(i, j)];
                const double o = fma(cn, base[q][i][j], fma((2.0 * i + 1.0) * (2.0 * j + 1.0) / 16.0 * lam, R[q][i][j], own_c * s0));
                bad = fma(o, 0.0, bad);
                if (valid) *po = o;
                R[q][i][j] = o;
            }
    if (valid && !(bad == 0.0)) a.err[0] = 1;
    if (valid && a.rs.ca != 0.0) {               // classical RK4: the sum of the damped inputs that its last stage needs
        double *p = AM;
#pragma unroll
        for (int q = 0; q < NC; ++q)
#pragma unroll
            for (int i = 0; i < K1; ++i)
#pragma unroll
                for (int j = 0; j < K1; ++j, p += a.plane) {
                    const double s0 = kept<K, PK>(i, j) ? own[q * NM + kept_index<K, PK>(i, j)] : 0.0;
                    *p = a.rs.acc_first ? a.rs.ca * s0 : fma(a.rs.ca, s0, *p);
                }
    }
    if (valid && FM && a.l == 0) {               // the factors of the step's input, for its later stages
        double nv[K1 * NC];
        load_numerators<K, NC>(mesh ? a.numD : a.numC, a.plane, gofs, nv);
        damp_factors<K, NC>(nv, st, mesh, fn);
#pragma unroll
        for (int j = 0; j < K; ++j) FM[j * a.plane] = fn[j];
    }
    // Statistics of the output, from registers: this kernel waits on memory
    // where k_delta2d, which had them, is bound by VALU issue.
    wave_record<K, FLUX, PK>(a, mesh, valid, [&](int q, double (&m)[K1][K1]) {
#pragma unroll
        for (int i = 0; i < K1; ++i)
#pragma unroll
            for (int j = 0; j < K1; ++j) m[i][j] = R[q][i][j];
    }, a.part + ((long long)tileid * (MT / WAVE) + tid % MT / WAVE) * Rec2<NC>::N);
}

// Statistics of given data (a run's initial data, oecdg_dt): a record per 64 cells.
template <int K, int FLUX, bool PK>
__global__ __launch_bounds__(256) void k_stats2d(Stage2Args a) {
    constexpr int NC = Flux2D<FLUX>::NC, K1 = K + 1;
    const long long g = (long long)blockIdx.x * 256 + threadIdx.x;
    const bool valid = g < a.plane;
    if (g - threadIdx.x % WAVE >= a.plane) return;           // the whole wave
#pragma unroll 1
    for (int mesh = 0; mesh < 2; ++mesh) {
        const double *in = (mesh ? a.inD : a.inC) + (valid ? g : 0);
        wave_record<K, FLUX, PK>(a, mesh, valid, [&](int q, double (&m)[K1][K1]) {
#pragma unroll
            for (int i = 0; i < K1; ++i)
#pragma unroll
                for (int j = 0; j < K1; ++j) m[i][j] = kept<K, PK>(i, j) ? in[((q * K1 + i) * K1 + j) * a.plane] : 0.0;
        }, a.part + g / WAVE * Rec2<NC>::N);
    }
}

// A state damped without a stage (damp off: copied), one thread per cell; grid.y is the mesh.
template <int K, int FLUX, bool PK>
__global__ __launch_bounds__(256) void k_damp2d(Stage2Args a) {
    constexpr int NC = Flux2D<FLUX>::NC, K1 = K + 1;
    const long long g = (long long)blockIdx.x * 256 + threadIdx.x;
    const int mesh = blockIdx.y;
    if (g >= a.plane) return;
    double f[K];
#pragma unroll
    for (int j = 0; j < K; ++j) f[j] = 1.0;
    if (a.damp) {
        double nv[K1 * NC];
        load_numerators<K, NC>(mesh ? a.numD : a.numC, a.plane, g, nv);
        damp_factors<K, NC>(nv, a.st, mesh, f);
    }
    const double *in = (mesh ? a.inD : a.inC) + g;
    double *out = (mesh ? a.outD : a.outC) + g;
#pragma unroll
    for (int q = 0; q < NC; ++q)
#pragma unroll
        for (int i = 0; i < K1; ++i)
#pragma unroll
            for (int j = 0; j < K1; ++j) {
                const long long e = (long long)((q * K1 + i) * K1 + j) * a.plane;
                if (!kept<K, PK>(i, j)) out[e] = 0.0;
                else out[e] = i + j == 0 ? in[e] : in[e] * f[(i + j < K ? i + j : K) - 1];
            }
}

// ---------------------------------------------------------- reduction ---

constexpr int RED2_NT = 256;
constexpr int RED2_LDS = RED2_NT + 2;
constexpr int RED2_MAXB = 64;
constexpr int RED2_AHEAD = 8;                    // records in flight per thread

__device__ inline void set_step(const Red2Args &r, double tau, double tau_max) {
    r.st->tau = tau;
    r.st->tau_max = tau_max;
    r.st->fx = 2.0 * tau_max / r.hx;
    r.st->fy = 2.0 * tau_max / r.hy;
    r.st->ratio = tau / tau_max;
}

// Workgroup blk of r.nb folds its range of records into r.fold; the last one to
// arrive folds those and updates the step scalars.  Both in a fixed order, so the
// result does not depend on which one is last.  lds: RED2_LDS doubles.
template <int NC>
__device__ void reduce2d(const Red2Args &r, int blk, double *lds) {
    using RC = Rec2<NC>;
    constexpr int G = RC::G, N = RC::N, NM = RC::NM, SUB = RED2_NT / G;
    const int tid = threadIdx.x, row = tid % G, sub = tid / G;
    const int j = row < N ? row : 0, kind = RC::kind(j);
    Stats2 *st = r.st;
    auto op = [kind](double x, double y) { return kind == 0 ? x + y : (kind == 1 ? max_d(x, y) : min_d(x, y)); };
    auto combine = [&](double v) {               // over the subs in order: thread row < N gets row's value
        lds[tid] = v;
        __syncthreads();
        double t = lds[row];
        for (int k = 1; k < SUB; ++k) t = op(t, lds[k * G + row]);
        __syncthreads();
        return t;
    };
    if (r.mode == R2_SINGLE) {
        if (tid == 0) {
            set_step(r, r.tau_o, r.taumax_o);
            st->tau_damp = r.tau_o;
            st->done[0] = st->done[1] = 0;
        }
        return;
    }
    const int t0 = blk * r.per, t1 = min(r.nrec, t0 + r.per);
    double acc = stat_identity(kind);
    for (int t = t0 + sub; t < t1; t += SUB * RED2_AHEAD) {
        double x[RED2_AHEAD];
#pragma unroll
        for (int i = 0; i < RED2_AHEAD; ++i) x[i] = r.part[(long long)min(t + i * SUB, t1 - 1) * N + j];
#pragma unroll
        for (int i = 0; i < RED2_AHEAD; ++i) {
            const double y = op(acc, x[i]);
            acc = t + i * SUB < t1 ? y : acc;
        }
    }
    double tot = combine(acc);
    if (r.nb > 1) {
        if (sub == 0 && row < N)
            __hip_atomic_store(&r.fold[blk * N + row], tot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();                     // (the stores are the first wave's, as the arrival, which waits for them)
        unsigned *flag = (unsigned *)(lds + RED2_NT);
        if (tid == 0) {
            const unsigned n = __hip_atomic_fetch_add(r.count, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
            *flag = n == (unsigned)r.nb - 1;
        }
        __syncthreads();
        if (!*flag) return;                  // uniform over the workgroup
        if (tid == 0) __hip_atomic_store(r.count, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        acc = stat_identity(kind);
        for (int b = sub; b < r.nb; b += SUB)
            acc = op(acc, __hip_atomic_load(&r.fold[b * N + j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        tot = combine(acc);
    }
    lds[tid] = tot;
    __syncthreads();
    if (r.mode == R2_STAGE && st->done[r.gpar ^ 1]) {            // the run has ended: nothing changes but the entry of this parity
        if (tid == 0) st->done[r.gpar] = 1;
        return;
    }
    if (tid < 2 * NC) {
        const int mesh = tid / NC, q = tid % NC;
        const double *t = lds + mesh * NM + 3 * q;
        const double avg = t[0] / (double)r.ncell;
        const double sig = fmax(t[1] - avg, avg - t[2]);
        const double s[1] = {sig};
        double is[1];
        const bool any = __any(recip_sigma(s, is));   // (all in one wave)
        st->isig[mesh][q] = is[0];
        if (tid == 0) st->small = any;
    }
    if (tid != 0) return;
    const double bx = max_d(lds[3 * NC], lds[NM + 3 * NC]), by = max_d(lds[3 * NC + 1], lds[NM + 3 * NC + 1]);
    st->bx = bx;
    st->by = by;
    if (r.mode == R2_STEP || r.mode == R2_FINAL) {
        if (st->pending) {                       // complete the previous step
            st->t = st->last ? r.t_end : st->t + st->tau;
            st->nexec += 1;
            st->pending = 0;
        }
        st->tau_damp = st->tau;
    }
    if (r.mode == R2_STEP) {
        if (!(st->t < r.t_end) || st->bad) {     // (after a bad step the records are older ones')
            st->done[r.gpar] = 1;
            return;
        }
        double tm = r.dt_fixed;
        if (!(tm > 0.0)) {
            const double rate = bx / r.hx + by / r.hy;
            if (!(rate > 0.0) || !isfinite(rate)) {
                st->done[r.gpar] = 1;
                st->bad = 1;
                r.err[2] = 1;
                return;
            }
            tm = r.cfl / rate;
        }
        double tau = tm;
        int last = 0;
        if (st->t + tau >= r.t_end) {
            tau = r.t_end - st->t;
            last = 1;
        }
        set_step(r, tau, tm);
        st->last = last;
        st->done[r.gpar] = 0;
        st->pending = 1;
    } else if (r.mode == R2_STAGE) {
        st->tau_damp = st->tau;
        st->done[r.gpar] = 0;
    }
}

// ----------------------------------------------------------- delta kernel ---

// Damping numerators of a state (the undamped output of a stage): per cell and
// component q
//   N^m_q = sum_{e in {W,E,S,N}} beta_{e,K} (2m+1) h_e^(m-1) / ((2k-1) m!)
//           (1/|e|) int_e ( sum_{alpha1+alpha2=m} (d^alpha (u_K - w)_q)^2 )^(1/2) ds
// (delta^m_K = max_q N^m_q / sigma_q once sigma is known, Sec. 2.2).
//
// The two edges of a direction share beta, so N^m_q = beta_x X^m_q + beta_y Y^m_q
// with X, Y formed from component q alone: a workgroup takes one component of
// one tile, and its threads one cell of each mesh in turn.  Along a half-edge
// the traces of both meshes are polynomials in the edge coordinate; the other
// mesh's is brought to the cell's own coordinate (tb.sh), and the derivatives of
// the difference are evaluated from its coefficients.

// sqrt terms of one direction: acc[m] = sum over both edges, both halves and the
// Gauss nodes of w_g (sum_alpha (d^alpha (u_K - w))^2)^(1/2).  u[n][t]: the own
// cell's modes, normal to the edge and along it; oth: the other mesh's, of which
// cell side sn + half st (strides sn, st) overlaps each half-edge.
// The W (S) edge is evaluated as its mirror image on the E (N) edge: the odd modes
// of the normal direction change sign in both cells, the derivatives at most
// their sign.  Derivatives are scaled by the tangential (2/h_t)^m of their order m:
// the factor leaves the root and is applied to the sum at the end, and a normal
// derivative brings (h_t/h_n) each.
template <int K, bool PK, bool DIRY, int NCELL>
__device__ inline void edge_norms(const double (&u)[K + 1][K + 1], const double *oth, int sn, int st, double hn,
                                  double ht, double (&acc)[K + 1]) {
    constexpr int K1 = K + 1, Q = K + 1;
    constexpr Tab2<K> tb = make_tab2<K>();
    double kap[K1], sct[K1];
    kap[0] = sct[0] = 1.0;
#pragma unroll
    for (int d = 1; d < K1; ++d) {
        kap[d] = kap[d - 1] * (ht / hn);
        sct[d] = sct[d - 1] * (2.0 / ht);
    }
#pragma unroll
    for (int m = 0; m < K1; ++m) acc[m] = 0.0;
    // what the sums of the roots come to where every sum of squares is 0 (exactly: the
    // additions below, scaled by 2^537); a sum of larger ones does not change by it
    constexpr double none = [] {
        constexpr Tab2<K> t = make_tab2<K>();
        double x = 0.0;
        for (int i = 0; i < 4; ++i)
            for (int g = 0; g < Q; ++g) x += t.w[g];
        return x * 0x1p-537;
    }();
    double tiny = SQRT_TINY;                     // in a register: as a constant it is moved there for every sum
    asm volatile("" : "+v"(tiny));
#pragma unroll 1
    for (int side = 0; side < 2; ++side) {
        const unsigned fn = side ? 0u : 0x80000000u;
        double own[K1][K1], ks[K1];              // own trace by [normal derivative][mode along the edge], scaled
#pragma unroll
        for (int dn = 0; dn < K1; ++dn) {
            ks[dn] = (dn & 1) ? flip_sign(kap[dn], fn) : kap[dn];
#pragma unroll
            for (int t = 0; t < K1; ++t) {
                own[dn][t] = 0.0;
                if (!kept<K, PK>(dn, t)) continue;
                double ev = 0.0, od = 0.0;       // even and odd normal modes
                bool e0 = true, o0 = true;
#pragma unroll
                for (int n = dn; n < K1; ++n) {
                    if (!kept<K, PK>(n, t)) continue;
                    if (n & 1) od = o0 ? mul_c(tb.e1[dn][n], u[n][t]) : mad_c(tb.e1[dn][n], u[n][t], od), o0 = false;
                    else ev = e0 ? mul_c(tb.e1[dn][n], u[n][t]) : mad_c(tb.e1[dn][n], u[n][t], ev), e0 = false;
                }
                const double x = o0 ? ev : (e0 ? flip_sign(od, fn) : ev + flip_sign(od, fn));
                own[dn][t] = dn == 0 ? x : x * kap[dn];
            }
        }
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const double *o = oth + side * sn + half * st;
            double D[K1][K1];                    // the traces' difference, own coordinate
#pragma unroll
            for (int dn = 0; dn < K1; ++dn) {
                double r[K1];                    // derivative dn of the other trace at its centre line
#pragma unroll
                for (int t = 0; t < K1; ++t) {
                    r[t] = 0.0;
                    if (!kept<K, PK>(dn, t)) continue;
#pragma unroll
                    for (int n = dn; n < K1; n += 2)                  // (one parity)
                        if (kept<K, PK>(n, t)) {
                            const double w = o[(DIRY ? kept_index<K, PK>(t, n) : kept_index<K, PK>(n, t)) * NCELL];
                            r[t] = n == dn ? mul_c(tb.e0[dn][n], w) : mad_c(tb.e0[dn][n], w, r[t]);
                        }
                    if (dn > 0) r[t] *= ks[dn];
                }
#pragma unroll
                for (int t = 0; t < K1; ++t) {
                    double x = own[dn][t];
#pragma unroll
                    for (int j = t; j < K1; ++j)
                        if (kept<K, PK>(dn, j)) x = j == t ? x - r[j] : fma(r[j], -tb.sh[half][j][t], x);
                    D[dn][t] = x;
                }
            }
#pragma unroll
            for (int g = 0; g < Q; ++g)
#pragma unroll
                for (int m = 0; m < K1; ++m) {
                    double ss = tiny;
#pragma unroll
                    for (int dn = 0; dn <= m; ++dn) {
                        const int dt = m - dn;
                        double v = 0.0;
                        bool first = true;
#pragma unroll
                        for (int t = dt; t < K1; ++t)
                            if (kept<K, PK>(dn, t) && tb.own[dt][half][g][t] != 0.0) {
                                const double c = tb.own[dt][half][g][t];
                                v = first ? mul_c(c, D[dn][t]) : mad_c(c, D[dn][t], v);
                                first = false;
                            }
                        ss = m == 0 ? fabs(v) : fma(v, v, ss);
                    }
                    acc[m] = fma(tb.w[g], m == 0 ? ss : sqrt_nr(ss), acc[m]);   // |d| = (d^2)^(1/2) for m = 0
                }
            __builtin_amdgcn_sched_barrier(0);   // one half-edge at a time: bounds the live registers
        }
    }
#pragma unroll
    for (int m = 1; m < K1; ++m) acc[m] = min_d(acc[m] - none, INFINITY) * sct[m];
}

// A workgroup takes one mesh of one component of a tile, a cell per thread: only
// the other mesh is staged in LDS (21 KB for k = 2), the own cell is in registers,
// and registers alone limit the waves in flight.  Workgroups 0 .. nred-1 reduce
// the stage's statistics meanwhile (reduce2d): they depend on the stage kernel
// alone.
__host__ __device__ constexpr int delta_blocks(int nt) { return 2 * ((nt + 7) / 8 * 8); }   // per component

template <int K, int FLUX, int TX, int TY, bool PK>
__global__ __launch_bounds__(TX * TY, K == 3 ? 2 : 4) void k_delta2d(Stage2Args a, Red2Args red) {
    using F = Flux2D<FLUX>;
    constexpr int NC = F::NC, K1 = K + 1, NM = kept_modes<K, PK>();
    constexpr int W = Halo2<TX, TY>::W, NCELL = Halo2<TX, TY>::N, NT = TX * TY;
    constexpr Tab2<K> tb = make_tab2<K>();
    static_assert(NT == RED2_NT && NM * NCELL >= RED2_LDS, "reduce2d runs in this workgroup");
    __shared__ double tile[NM * NCELL];          // [mode][cell] of component q of the other mesh

    if (blockIdx.x < (unsigned)a.nred) {
        reduce2d<NC>(red, blockIdx.x, tile);
        return;
    }
    // component, then (per XCD) a band of tiles, both meshes of a tile next to each other
    const int tid = threadIdx.x;
    const int nt = a.ntx * a.nty, per = delta_blocks(nt), b = blockIdx.x - a.nred, q = b / per, l = b - q * per;
    const int mesh = (l >> 3) & 1, tileid = (l & 7) * (per / 16) + (l >> 4);
    if (tileid >= nt || a.st->done[a.gpar]) return;
    const int i0 = (tileid % a.ntx) * TX, j0 = (tileid / a.ntx) * TY;
    const int s = tid % TX, r = tid / TX, gx = i0 + s, gy = j0 + r;
    const bool valid = gx < a.nx && gy < a.ny;
    const long long gofs = valid ? (long long)gy * a.nx + gx : 0, qofs = (long long)q * K1 * K1 * a.plane;
    const bool small = a.nx <= TX || a.ny <= TY;

    // every load before the first wait: the own cell and its averages, the other mesh's cells
    double u[K1][K1], ub[NC];
    {
        const double *p = (mesh ? a.inD : a.inC) + gofs + qofs;
#pragma unroll
        for (int i = 0; i < K1; ++i)
#pragma unroll
            for (int j = 0; j < K1; ++j, p += a.plane) u[i][j] = kept<K, PK>(i, j) ? *p : 0.0;
        p = (mesh ? a.inD : a.inC) + gofs;
#pragma unroll
        for (int c = 0; c < NC; ++c, p += K1 * K1 * a.plane) ub[c] = *p;
    }
    constexpr int REST = NCELL - NT;
    static_assert(REST > 0 && REST <= WAVE, "one more cell per lane of the first wave");
    auto cell_ptr = [&](int c) {                 // cell c of the other mesh: primal from i0-1, dual from i0
        const int x = wrap_idx(i0 - mesh + c % W, a.nx, small), y = wrap_idx(j0 - mesh + c / W, a.ny, small);
        return (mesh ? a.inC : a.inD) + qofs + (long long)y * a.nx + x;
    };
    double v0[NM], v1[NM];
    auto load = [&](const double *p, double (&v)[NM]) {
#pragma unroll
        for (int i = 0; i < K1; ++i)
#pragma unroll
            for (int j = 0; j < K1; ++j, p += a.plane)
                if (kept<K, PK>(i, j)) v[kept_index<K, PK>(i, j)] = *p;
    };
    load(cell_ptr(tid), v0);
    if (tid < REST) load(cell_ptr(NT + tid), v1);
#pragma unroll
    for (int e = 0; e < NM; ++e) tile[e * NCELL + tid] = v0[e];
    if (tid < REST) {
#pragma unroll
        for (int e = 0; e < NM; ++e) tile[e * NCELL + NT + tid] = v1[e];
    }
    __syncthreads();

    const double *oth = tile + r * W + s;
    double X[K1], Y[K1], ut[K1][K1];
    edge_norms<K, PK, false, NCELL>(u, oth, 1, W, a.hx, a.hy, X);
#pragma unroll
    for (int i = 0; i < K1; ++i)
#pragma unroll
        for (int j = 0; j < K1; ++j) ut[i][j] = u[j][i];
    edge_norms<K, PK, true, NCELL>(ut, oth, W, 1, a.hy, a.hx, Y);
    if (!valid) return;
    double bx, by;
    F::speeds(ub, bx, by, a.fp);
    double *N = (mesh ? a.numD : a.numC) + gofs;
    double hxm = 1.0 / a.hx, hym = 1.0 / a.hy;             // h_e^(m-1)
#pragma unroll
    for (int m = 0; m < K1; ++m) {
        N[(long long)(m * NC + q) * a.plane] = 0.25 * tb.cdel[m] * (bx * hxm * X[m] + by * hym * Y[m]);
        hxm = m == 0 ? 1.0 : hxm * a.hx;
        hym = m == 0 ? 1.0 : hym * a.hy;
    }
}

// The reduction alone (before a run's first stage, at its end, with OE off).
template <int NC>
__global__ __launch_bounds__(RED2_NT) void k_reduce2d(Red2Args r) {
    __shared__ double lds[RED2_LDS];
    reduce2d<NC>(r, blockIdx.x, lds);
}

// ------------------------------------------------------------ host side ---

namespace {

// Tiles of k_stage2d in primal cells and waves per SIMD asked for.  Rows of 16 cells
// are whole 128-byte lines.  The Euler tiles are the largest of which two fit the
// 160 KB of LDS (2 x 80.5 KB for Q2 at 16 x 7: eight waves per CU and a halo of
// 1.21 cells per owned one; three of 16 x 4 left six waves on four SIMDs at 1.33,
// and 8 x 4, a wave each, measured the same or slower in every space).  Q3 needs
// 74.9 KB for 8 x 7, four waves per CU.  k_delta2d takes 16 x 16 of one component.
template <int K, int FLUX, bool PK> struct Tile2 {
    static constexpr bool EULER = FLUX == OECDG_FLUX_EULER;
    static constexpr int TX = EULER && K == 3 && !PK ? 8 : 16;
    static constexpr int TY = !EULER || K == 1 ? 4 : (K == 3 ? (PK ? 4 : 7) : (PK ? 8 : 7));
    static constexpr int WPS = !EULER ? (K == 3 && !PK ? 3 : 4) : (K == 3 ? 1 : (K == 1 ? 4 : 2));
};
constexpr int DELTA_T = 16;
struct Tiles2 {
    int tx, ty;
};

// which: 0 stage, 1 delta, 2 damp, 3 statistics of given data
template <int K, int FLUX, bool PK>
void *kernel2d_fn(int which, Tiles2 &t) {
    using T = Tile2<K, FLUX, PK>;
    t = {T::TX, T::TY};
    if (which == 1) return (void *)k_delta2d<K, FLUX, DELTA_T, DELTA_T, PK>;
    if (which == 2) return (void *)k_damp2d<K, FLUX, PK>;
    if (which == 3) return (void *)k_stats2d<K, FLUX, PK>;
    return (void *)k_stage2d<K, FLUX, T::TX, T::TY, T::WPS, PK>;
}

template <int K>
void *pick2_k(int flux, bool pk, int which, Tiles2 &t) {
    if (flux == OECDG_FLUX_EULER)
        return pk ? kernel2d_fn<K, OECDG_FLUX_EULER, true>(which, t) : kernel2d_fn<K, OECDG_FLUX_EULER, false>(which, t);
    return pk ? kernel2d_fn<K, OECDG_FLUX_ADVECTION, true>(which, t)
              : kernel2d_fn<K, OECDG_FLUX_ADVECTION, false>(which, t);
}

// Kernel of a kind, and the stage kernel's tile.
void *pick2(int k, int flux, bool pk, int which, Tiles2 &t) {
    switch (k) {
    case 1: return pick2_k<1>(flux, pk, which, t);
    case 2: return pick2_k<2>(flux, pk, which, t);
    default: return pick2_k<3>(flux, pk, which, t);
    }
}

struct Ext2D {
    int k, nc, flux, oe;
    int pk;                      // total-degree space P^k
    Tiles2 t;                    // k_stage2d: primal cells per tile and direction
    void *fn[4];                 // kernels (pick2)
    int rk, ns;                  // RK method (rk_stage) and its stages per step
    int nx, ny;
    int ntx, nty;                // k_stage2d's tiles
    int dtx, dty;                // k_delta2d's tiles
    double hx, hy, cfl;
    FPar2 fp;
    long long S1;                // doubles of one mesh
    long long SN;                // damping numerators of one mesh: (k+1) nc nx ny
    double *B[3] = {nullptr, nullptr, nullptr};   // stage states, both meshes each (run_2d)
    double *num[2] = {nullptr, nullptr};    // damping numerators of B[i], both meshes each
    double *A = nullptr;         // classical RK4: accumulated damped inputs of stages 1 and 2 (both meshes)
    double *fac = nullptr;       // damping factors of the step's input, K per cell (both meshes)
    double *part[2] = {nullptr, nullptr};
    double *fold = nullptr;      // first-level records of the reduction
    unsigned *count = nullptr;   // its arrival count
    Stats2 *st = nullptr;
    Stats2 *st_h = nullptr;      // pinned
    int *err = nullptr, *err_h = nullptr;
};

Ext2D *ext(oecdg_handle *h) { return static_cast<Ext2D *>(handle_ext2d(h)); }

#define HIPCHK2(h, expr)                                                                                      \
    do {                                                                                                      \
        hipError_t e_ = (expr);                                                                               \
        if (e_ != hipSuccess) return handle_fail((h), OECDG_EHIP, hipGetErrorString(e_));                     \
    } while (0)

hipError_t launch_stage2d(const Ext2D &x, const Stage2Args &a, hipStream_t s) {
    Stage2Args copy = a;
    copy.ntx = x.ntx;
    copy.nty = x.nty;
    void *args[] = {&copy};
    return hipLaunchKernel(x.fn[0], dim3(x.ntx * x.nty), dim3(2 * mesh_threads(x.t.tx, x.t.ty)), args, 0, s);
}

// Workgroups of the reduction of nrec records: enough for a few rounds of loads
// each (a workgroup has RED2_NT / G records in a round), at most RED2_MAXB.
int red_blocks(int nrec) { return std::min(RED2_MAXB, (nrec + 127) / 128); }

// Numerators of the state in a.inC/inD when OE is on, and (red) the reduction for
// the next stage beside them.
hipError_t launch_delta2d(const Ext2D &x, const Stage2Args &a, const Red2Args *red, hipStream_t s) {
    Stage2Args copy = a;
    Red2Args r{};
    copy.ntx = x.dtx;
    copy.nty = x.dty;
    copy.nred = 0;
    if (red) {
        r = *red;
        copy.nred = r.nb;
    }
    if (x.oe && x.k > 0) {
        void *args[] = {&copy, &r};
        return hipLaunchKernel(x.fn[1], dim3(copy.nred + delta_blocks(x.dtx * x.dty) * x.nc),
                               dim3(DELTA_T * DELTA_T), args, 0, s);
    }
    if (!red) return hipSuccess;
    void *args[] = {&r};
    void *fn = x.nc == 4 ? (void *)k_reduce2d<4> : (void *)k_reduce2d<1>;
    return hipLaunchKernel(fn, dim3(r.nb), dim3(RED2_NT), args, 0, s);
}

hipError_t launch_reduce2d(const Ext2D &x, const Red2Args &red, hipStream_t s) {
    Red2Args r = red;
    void *args[] = {&r};
    void *fn = x.nc == 4 ? (void *)k_reduce2d<4> : (void *)k_reduce2d<1>;
    return hipLaunchKernel(fn, dim3(r.nb), dim3(RED2_NT), args, 0, s);
}

hipError_t launch_stats2d(const Ext2D &x, const Stage2Args &a, hipStream_t s) {
    Stage2Args copy = a;
    void *args[] = {&copy};
    return hipLaunchKernel(x.fn[3], dim3((unsigned)((a.plane + 255) / 256)), dim3(256), args, 0, s);
}

hipError_t launch_damp2d(const Ext2D &x, const Stage2Args &a, hipStream_t s) {
    Stage2Args copy = a;
    void *args[] = {&copy};
    return hipLaunchKernel(x.fn[2], dim3((unsigned)((a.plane + 255) / 256), 2), dim3(256), args, 0, s);
}

Stage2Args stage_args(const Ext2D &x) {
    Stage2Args a;
    memset(&a, 0, sizeof(a));
    a.nx = x.nx;
    a.ny = x.ny;
    a.plane = (long long)x.nx * x.ny;
    a.hx = x.hx;
    a.hy = x.hy;
    a.fp = x.fp;
    a.st = x.st;
    a.err = x.err;
    if (x.A) {
        a.AC = x.A;
        a.AD = x.A + x.S1;
    }
    a.rs = rk_stage(x.rk, 0);
    return a;
}

// Records of a stage's output: one per wave of primal cells of k_stage2d; of given data: one per 64 cells.
int stage_records(const Ext2D &x) { return x.ntx * x.nty * (mesh_threads(x.t.tx, x.t.ty) / WAVE); }
int data_records(const Ext2D &x) { return (int)(((long long)x.nx * x.ny + 63) / 64); }

// gpar: parity of the stage that the result is for.
Red2Args red_args(const Ext2D &x, const double *part, int nrec, int mode, int gpar) {
    Red2Args r;
    memset(&r, 0, sizeof(r));
    r.part = part;
    r.nrec = nrec;
    r.nb = red_blocks(nrec);
    r.per = (nrec + r.nb - 1) / r.nb;
    r.mode = mode;
    r.gpar = gpar;
    r.ncell = (long long)x.nx * x.ny;
    r.t_end = INFINITY;
    r.cfl = x.cfl;
    r.hx = x.hx;
    r.hy = x.hy;
    r.fold = x.fold;
    r.count = x.count;
    r.st = x.st;
    r.err = x.err;
    return r;
}

// Arguments of k_delta2d for a state: its numerators into num[i].
Stage2Args delta_args(const Ext2D &x, const double *uC, const double *uD, int i, int gpar) {
    Stage2Args a = stage_args(x);
    a.gpar = gpar;
    a.inC = uC;
    a.inD = uD;
    a.numC = x.num[i];
    a.numD = x.num[i] + x.SN;
    return a;
}

hipError_t stats_of(const Ext2D &x, const double *uC, const double *uD, int i, hipStream_t s) {
    Stage2Args a = stage_args(x);
    a.inC = uC;
    a.inD = uD;
    a.part = x.part[i];
    return launch_stats2d(x, a, s);
}

int check2d(oecdg_handle *h, const Ext2D &x) {
    hipStream_t s = handle_stream(h);
    HIPCHK2(h, hipMemcpyAsync(x.err_h, x.err, 4 * sizeof(int), hipMemcpyDeviceToHost, s));
    HIPCHK2(h, hipStreamSynchronize(s));
    if (x.err_h[2]) return handle_fail(h, OECDG_ENONFINITE, "no admissible time step (wave speed zero or not finite)");
    if (x.err_h[0]) return handle_fail(h, OECDG_ENONFINITE, "non-finite coefficient produced");
    if (x.err_h[1]) return handle_fail(h, OECDG_ENONPHYSICAL, "non-positive density or pressure at a cell average");
    return OECDG_OK;
}

int reset2d(oecdg_handle *h, Ext2D &x) {
    hipStream_t s = handle_stream(h);
    memset(x.st_h, 0, sizeof(Stats2));
    HIPCHK2(h, hipMemcpyAsync(x.st, x.st_h, sizeof(Stats2), hipMemcpyHostToDevice, s));
    HIPCHK2(h, hipMemsetAsync(x.err, 0, 4 * sizeof(int), s));
    return OECDG_OK;
}

}  // namespace

int create_2d(oecdg_handle *h, const oecdg_desc *d) {
    Ext2D *x = new (std::nothrow) Ext2D();
    if (!x) return OECDG_ENOMEM;
    handle_ext2d(h) = x;
    x->k = d->k;
    x->flux = d->flux;
    x->nc = d->flux == OECDG_FLUX_EULER ? 4 : 1;
    x->oe = d->oe;
    x->pk = d->space == 1;
    x->nx = (int)d->nx;
    x->ny = (int)d->ny;
    for (int i = 0; i < 4; ++i) x->fn[i] = pick2(x->k, x->flux, x->pk, i, x->t);
    x->rk = d->rk == 0 ? 3 : d->rk;
    x->ns = rk_stages(x->rk);
    x->ntx = (x->nx + x->t.tx - 1) / x->t.tx;
    x->nty = (x->ny + x->t.ty - 1) / x->t.ty;
    x->dtx = (x->nx + DELTA_T - 1) / DELTA_T;
    x->dty = (x->ny + DELTA_T - 1) / DELTA_T;
    x->hx = (d->xhi - d->xlo) / d->nx;
    x->hy = (d->yhi - d->ylo) / d->ny;
    x->cfl = d->cfl;
    x->fp.a = d->flux_param[0];
    x->fp.b = d->flux_param[1];
    x->fp.gamma = d->flux_param[0];
    x->S1 = (long long)x->nc * (x->k + 1) * (x->k + 1) * x->nx * x->ny;
    x->SN = (long long)x->nc * (x->k + 1) * x->nx * x->ny;
    const size_t nval = x->nc == 4 ? Rec2<4>::N : Rec2<1>::N;   // doubles of a record
    const size_t nrec = std::max(stage_records(*x), data_records(*x));
    for (int i = 0; i < (x->ns > 2 ? 3 : 2); ++i) HIPCHK2(h, hipMalloc(&x->B[i], sizeof(double) * 2 * x->S1));
    HIPCHK2(h, hipMalloc(&x->fac, sizeof(double) * 2 * x->k * x->nx * x->ny));
    for (int i = 0; i < 2; ++i) {
        HIPCHK2(h, hipMalloc(&x->num[i], sizeof(double) * 2 * x->SN));
        HIPCHK2(h, hipMalloc(&x->part[i], sizeof(double) * nval * nrec));
    }
    if (x->rk == 4) HIPCHK2(h, hipMalloc(&x->A, sizeof(double) * 2 * x->S1));
    HIPCHK2(h, hipMalloc(&x->fold, sizeof(double) * nval * RED2_MAXB));
    HIPCHK2(h, hipMalloc(&x->count, sizeof(unsigned)));
    const unsigned none = 0;
    HIPCHK2(h, hipMemcpy(x->count, &none, sizeof(none), hipMemcpyHostToDevice));
    HIPCHK2(h, hipMalloc(&x->st, sizeof(Stats2)));
    HIPCHK2(h, hipHostMalloc((void **)&x->st_h, sizeof(Stats2), hipHostMallocDefault));
    HIPCHK2(h, hipMalloc(&x->err, 4 * sizeof(int)));
    HIPCHK2(h, hipHostMalloc((void **)&x->err_h, 4 * sizeof(int), hipHostMallocDefault));
    return OECDG_OK;
}

void destroy_2d(oecdg_handle *h) {
    Ext2D *x = ext(h);
    if (!x) return;
    for (double *b : x->B)
        if (b) (void)hipFree(b);
    if (x->fac) (void)hipFree(x->fac);
    for (int i = 0; i < 2; ++i) {
        if (x->num[i]) (void)hipFree(x->num[i]);
        if (x->part[i]) (void)hipFree(x->part[i]);
    }
    if (x->A) (void)hipFree(x->A);
    if (x->fold) (void)hipFree(x->fold);
    if (x->count) (void)hipFree(x->count);
    if (x->st) (void)hipFree(x->st);
    if (x->st_h) (void)hipHostFree(x->st_h);
    if (x->err) (void)hipFree(x->err);
    if (x->err_h) (void)hipHostFree(x->err_h);
    delete x;
    handle_ext2d(h) = nullptr;
}

int dt_2d(oecdg_handle *h, const double *uC, const double *uD, double *dt_out) {
    Ext2D &x = *ext(h);
    hipStream_t s = handle_stream(h);
    int rc = reset2d(h, x);
    if (rc != OECDG_OK) return rc;
    HIPCHK2(h, stats_of(x, uC, uD, 0, s));
    HIPCHK2(h, launch_reduce2d(x, red_args(x, x.part[0], data_records(x), R2_STATS, 0), s));
    HIPCHK2(h, hipMemcpyAsync(x.st_h, x.st, sizeof(Stats2), hipMemcpyDeviceToHost, s));
    HIPCHK2(h, hipStreamSynchronize(s));
    const double rate = x.st_h->bx / x.hx + x.st_h->by / x.hy;
    if (!(rate > 0.0) || !std::isfinite(rate)) return handle_fail(h, OECDG_ENONFINITE, "wave speed is zero or not finite");
    *dt_out = x.cfl / rate;
    return OECDG_OK;
}

int stage_2d(oecdg_handle *h, int stage, double dt, double tau_max, const double *uCn, const double *uDn,
             const double *uCl, const double *uDl, double *uCo, double *uDo) {
    Ext2D &x = *ext(h);
    hipStream_t s = handle_stream(h);
    int rc = reset2d(h, x);
    if (rc != OECDG_OK) return rc;
    Red2Args r = red_args(x, nullptr, 1, R2_SINGLE, 0);       // the step scalars only
    r.tau_o = dt;
    r.taumax_o = std::min(tau_max, 1e100 * dt);               // (infinite: no coupling; it is a factor of the fluxes)
    HIPCHK2(h, launch_reduce2d(x, r, s));
    Stage2Args a = stage_args(x);
    a.part = x.part[0];
    a.l = stage;
    a.rs = rk_stage(x.rk, stage);
    a.damp = 0;
    a.inC = stage == 0 ? uCn : uCl;
    a.inD = stage == 0 ? uDn : uDl;
    a.unC = uCn;
    a.unD = uDn;
    a.outC = x.B[0];
    a.outD = x.B[0] + x.S1;
    HIPCHK2(h, launch_stage2d(x, a, s));
    r = red_args(x, x.part[0], stage_records(x), R2_STAGE, 1);
    HIPCHK2(h, launch_delta2d(x, delta_args(x, x.B[0], x.B[0] + x.S1, 0, 0), &r, s));
    Stage2Args f = stage_args(x);
    f.damp = x.oe && x.k > 0;
    f.inC = x.B[0];
    f.inD = x.B[0] + x.S1;
    f.numC = x.num[0];
    f.numD = x.num[0] + x.SN;
    f.outC = uCo;
    f.outD = uDo;
    HIPCHK2(h, launch_damp2d(x, f, s));
    return check2d(h, x);
}

int run_2d(oecdg_handle *h, double *uC, double *uD, double t_end, int64_t nsteps, double dt_fixed, double *t_out,
           int64_t *steps_out) {
    Ext2D &x = *ext(h);
    hipStream_t s = handle_stream(h);
    if (nsteps < 0 && !std::isfinite(t_end)) return handle_fail(h, OECDG_EINVAL, "give a finite t_end or nsteps >= 0");
    int rc = reset2d(h, x);
    if (rc != OECDG_OK) return rc;
    // statistics of the initial data, and from them the first step
    auto reduction = [&](const double *part, int nrec, long long g, int mode) {   // for stage g of the run
        Red2Args r = red_args(x, part, nrec, mode, (int)(g & 1));
        r.t_end = t_end;
        r.dt_fixed = dt_fixed;
        return r;
    };
    HIPCHK2(h, stats_of(x, uC, uD, 0, s));
    if (nsteps != 0) HIPCHK2(h, launch_reduce2d(x, reduction(x.part[0], data_records(x), 0, R2_STEP), s));
    // Stage states.  The caller's arrays are the input of step 0 (P^k: the kernels
    // read no mode beyond k); a step's output is in B[0] and, but for forward Euler,
    // overwrites the step's input there in its last stage, which reads of it only
    // the cell it writes.  Between, the stages alternate between B[1] and B[2].
    auto buffer = [&](long long n, int l) -> double * {   // output of stage l of step n
        if (x.ns == 1) return x.B[n & 1];
        return l == x.ns - 1 ? x.B[0] : x.B[1 + (l & 1)];
    };
    const int chunk = 16;
    long long n = 0;
    while (nsteps < 0 || n < nsteps) {
        const long long m = nsteps < 0 ? chunk : std::min<long long>(chunk, nsteps - n);
        for (long long j = 0; j < m; ++j)
            for (int l = 0; l < x.ns; ++l) {
                const long long g = (long long)x.ns * (n + j) + l;
                const int ib = (int)(g & 1), ob = (int)((g + 1) & 1);
                Stage2Args a = stage_args(x);
                a.l = l;
                a.gpar = ib;
                a.rs = rk_stage(x.rk, l);
                a.damp = x.oe && x.k > 0 && g > 0;
                const bool first = n + j == 0;
                const double *un = first ? uC : buffer(n + j - 1, x.ns - 1), *in = l > 0 ? buffer(n + j, l - 1) : un;
                double *out = buffer(n + j, l);
                a.inC = in;
                a.inD = l == 0 && first ? uD : in + x.S1;
                a.unC = un;
                a.unD = first ? uD : un + x.S1;
                if (x.oe && x.k > 0 && !first) {
                    a.facC = x.fac;
                    a.facD = x.fac + (size_t)x.k * x.nx * x.ny;
                }
                a.numC = x.num[ib];
                a.numD = x.num[ib] + x.SN;
                a.outC = out;
                a.outD = out + x.S1;
                a.part = x.part[ob];
                HIPCHK2(h, launch_stage2d(x, a, s));
                // the numerators of its output and, beside them, the statistics for the next stage
                const bool end = l == x.ns - 1 && n + j + 1 == nsteps;
                const Red2Args r = reduction(x.part[ob], stage_records(x), g + 1, l == x.ns - 1 ? R2_STEP : R2_STAGE);
                HIPCHK2(h, launch_delta2d(x, delta_args(x, out, out + x.S1, ob, ib), end ? nullptr : &r, s));
            }
        n += m;
        HIPCHK2(h, hipMemcpyAsync(x.st_h, x.st, sizeof(Stats2), hipMemcpyDeviceToHost, s));
        HIPCHK2(h, hipStreamSynchronize(s));
        if (x.st_h->done[(x.ns * n) & 1]) break;           // (of the stage after the last one launched)
    }
    const long long N = x.st_h->nexec + x.st_h->pending;   // executed steps
    const int fb = (int)((x.ns * N) & 1);                  // parity of the last stage's numerators and statistics
    const double *last = N > 0 ? buffer(N - 1, x.ns - 1) : uC;   // its output
    HIPCHK2(h, launch_reduce2d(x, reduction(x.part[fb], N > 0 ? stage_records(x) : data_records(x), 0, R2_FINAL), s));
    Stage2Args f = stage_args(x);
    f.damp = x.oe && x.k > 0 && N > 0;
    f.inC = last;
    f.inD = N > 0 ? last + x.S1 : uD;
    f.numC = x.num[fb];
    f.numD = x.num[fb] + x.SN;
    f.outC = uC;
    f.outD = uD;
    HIPCHK2(h, launch_damp2d(x, f, s));
    HIPCHK2(h, hipMemcpyAsync(x.st_h, x.st, sizeof(Stats2), hipMemcpyDeviceToHost, s));
    rc = check2d(h, x);
    if (t_out) *t_out = x.st_h->t;
    if (steps_out) *steps_out = N;
    return rc;
}

}  // namespace oecdg
