// oecdg_device.h -- device helpers shared by the forward and adjoint kernels:
// flux functions, shared-state loads, order-fixed DPP reductions and the
// reduction of per-tile partial statistics.
#pragma once

#include "oecdg_internal.h"

#include <math.h>

namespace oecdg {

constexpr int WAVE = 64;

// a / b by the steps of the IEEE division without its range scaling and fix-up:
// the same bits wherever those do nothing (b and the quotient within about
// 2^+-1000 and neither 0 nor infinite), 8 instructions instead of 11.  b = 0
// gives NaN instead of an infinity; both make the output non-finite.  div_nr0 has the
// fix-up of zeros and infinities: a wave speed has to stay infinite, as a maximum drops
// a NaN.
__device__ inline double div_nr(double a, double b) {
    double r = __builtin_amdgcn_rcp(b);
    r = fma(r, fma(-b, r, 1.0), r);
    r = fma(r, fma(-b, r, 1.0), r);
    const double q = a * r;
    return fma(fma(-b, q, a), r, q);
}
__device__ inline double div_nr0(double a, double b) { return __builtin_amdgcn_div_fixup(div_nr(a, b), b, a); }

// 1 / sigma of components as the damping takes it: 0 where sigma is 0 (the component takes
// no part), and -1 / (SMALL_SCALE sigma) of a subnormal sigma, whose reciprocal may
// overflow; whether there is one.  scale_small then brings the others of the cell to that
// scale and takes it out of the exponents through tau; the damping reads the magnitudes.
constexpr double SMALL_SCALE = 0x1p64;
template <int NC>
__device__ inline bool recip_sigma(const double (&sig)[NC], double (&isig)[NC]) {
    double least = sig[0];
    bool small = false;
#pragma unroll
    for (int q = 0; q < NC; ++q) {
        isig[q] = 1.0 / sig[q];
        if (q > 0) least = fmin(least, sig[q]);
    }
    if (least < 0x1p-1022) {
#pragma unroll
        for (int q = 0; q < NC; ++q) {
            if (sig[q] == 0.0) isig[q] = 0.0;
            if (sig[q] > 0.0 && sig[q] < 0x1p-1022) {
                isig[q] = -1.0 / (SMALL_SCALE * sig[q]);
                small = true;
            }
        }
    }
    return small;
}
template <int NC>
__device__ inline bool any_small(const double (&isig)[NC]) {
    long long any = 0;
#pragma unroll
    for (int q = 0; q < NC; ++q) any |= __builtin_bit_cast(long long, isig[q]);
    return any < 0;
}
template <int NC>
__device__ inline void scale_small(double (&isig)[NC], double &tau) {
#pragma unroll
    for (int q = 0; q < NC; ++q)
        if (isig[q] > 0.0) isig[q] *= 1.0 / SMALL_SCALE;
    tau *= SMALL_SCALE;
}

// ---------------------------------------------------------------- fluxes ---

template <int FLUX> struct FluxT;

template <> struct FluxT<0> {          // linear advection f = a u
    static constexpr int NC = 1;
    __device__ static inline void f(const double *w, double *o, double a) { o[0] = a * w[0]; }
    __device__ static inline double speed(const double *, double a) { return fabs(a); }
    __device__ static inline bool physical(const double *, double) { return true; }
};

template <> struct FluxT<1> {          // Burgers f = u^2 / 2
    static constexpr int NC = 1;
    __device__ static inline void f(const double *w, double *o, double) { o[0] = 0.5 * w[0] * w[0]; }
    __device__ static inline double speed(const double *u, double) { return fabs(u[0]); }
    __device__ static inline bool physical(const double *, double) { return true; }
};

template <> struct FluxT<2> {          // Euler (rho, m, E), ideal gas
    static constexpr int NC = 3;
    __device__ static inline void f(const double *w, double *o, double g) {
        const double v = div_nr(w[1], w[0]);
        const double p = (g - 1.0) * (w[2] - 0.5 * w[1] * v);
        o[0] = w[1];
        o[1] = w[1] * v + p;
        o[2] = (w[2] + p) * v;
    }
    // |v| + sqrt(gamma |p| / rho): |v| + c for every physical state, finite
    // where a tolerated non-positive pressure sits at a cell average
    __device__ static inline double speed(const double *u, double g) {
        const double v = div_nr0(u[1], u[0]);
        const double p = (g - 1.0) * (u[2] - 0.5 * u[1] * v);
        return fabs(v) + sqrt(div_nr0(g * fabs(p), u[0]));
    }
    __device__ static inline bool physical(const double *u, double g) {
        if (!(u[0] > 0.0)) return false;
        const double p = (g - 1.0) * (u[2] - div_nr(0.5 * u[1] * u[1], u[0]));
        return p > 0.0;
    }
};

// Euler between reflective walls: the same flux; 1D kernels instantiated with
// it also carry the wall-ghost code (the others carry none).
template <> struct FluxT<3> : FluxT<2> {};

// ------------------------------------------------------ shared-state access ---
// Between kernel launches plain loads see the previous kernel's stores.  In
// the persistent launch, values written by other workgroups of the same
// launch are read with device-scope atomic loads after the grid barrier.

__device__ inline double ld_d(const double *p, bool coherent) {
    return coherent ? __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : *p;
}
__device__ inline int ld_i(const int *p, bool coherent) {
    return coherent ? __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : *p;
}
__device__ inline long long ld_ll(const long long *p, bool coherent) {
    return coherent ? __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : *p;
}
__device__ inline Slot ld_slot(const Slot *p, bool coherent) {
    Slot s;
    s.t = ld_d(&p->t, coherent);
    s.tau = ld_d(&p->tau, coherent);
    s.tau_max = ld_d(&p->tau_max, coherent);
    s.done = ld_i(&p->done, coherent);
    s.last = ld_i(&p->last, coherent);
    return s;
}

// Waits until the wave's stores are acknowledged (agent-scope atomic ones: by the memory
// that all XCDs share; plain ones: by the XCD's L2).  A workgroup barrier waits for no
// store, and a release in one thread only for those of its own wave: before other
// workgroups are told of stores of several waves, each wave waits here.
__device__ inline void wait_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// ------------------------------------------------------ tiles and XCDs ---
// Workgroup b of a launch over n tiles -> its tile (offset from the first).
// Workgroups are dealt to the 8 XCDs in turn (XCD b mod 8), so XCD x gets
// the band of consecutive tiles that starts at x*q + min(x, r) (q = n / 8,
// r = n mod 8; a bijection on [0, n)).  Neighbouring tiles read the cache
// lines at their common edge (planes whose length is not a multiple of 16
// doubles share a line at every tile edge); in one band they fetch them into
// one L2.
__device__ inline int xcd_tile(int b, int n) {
    const int x = b & 7, j = b >> 3, q = n >> 3, r = n & 7;
    return x * q + (x < r ? x : r) + j;
}

// ------------------------------------------------------------- reductions ---

__device__ inline double stat_identity(int kind) {
    return kind == 0 ? 0.0 : (kind == 1 ? -INFINITY : INFINITY);
}

// Maximum and minimum of two doubles as the bare v_max_f64 / v_min_f64.
// fmax and fmin first canonicalize each operand that the compiler cannot prove
// canonical (every DPP move and every load: one more dependent instruction per
// level of a reduction tree).  For all inputs except signalling NaNs, which no
// arithmetic here produces, the bare instruction returns what fmax and fmin
// return.
__device__ inline double max_d(double x, double y) {
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(x), "v"(y));
    return r;
}
__device__ inline double min_d(double x, double y) {
    double r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(x), "v"(y));
    return r;
}

__device__ inline double stat_op(int kind, double x, double y) {
    return kind == 0 ? x + y : (kind == 1 ? max_d(x, y) : min_d(x, y));
}

// Cross-lane data movement with DPP (plain VALU operations, no LDS round
// trip).  A 64-bit value moves as two 32-bit halves; lanes that the control
// does not write keep `old`.
template <int CTRL, int ROWMASK = 0xf>
__device__ inline double dpp_d(double v, double old) {
    const long long x = __builtin_bit_cast(long long, v), o = __builtin_bit_cast(long long, old);
    const int lo = __builtin_amdgcn_update_dpp((int)o, (int)x, CTRL, ROWMASK, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp((int)(o >> 32), (int)(x >> 32), CTRL, ROWMASK, 0xf, false);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (long long)(unsigned)lo);
}

// A lane permutation that writes every lane (quad_perm, row mirrors): no
// "old" operand, so none is copied.  Every lane of the wave must be active.
template <int CTRL>
__device__ inline double dpp_all(double v) {
    const long long x = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_mov_dpp((int)x, CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(x >> 32), CTRL, 0xf, 0xf, true);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (long long)(unsigned)lo);
}

// Value of lane k (uniform) in every lane.
__device__ inline double lane_value(double v, int k) {
    const long long x = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_readlane((int)x, k), hi = __builtin_amdgcn_readlane((int)(x >> 32), k);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (long long)(unsigned)lo);
}

// Reduction over the 64 lanes of a wave in a fixed tree (pairs, quads, half
// rows, rows, then rows 0+1 and 2+3, then all four); the result is in lane 63.
// Every lane of the wave must be active.
__device__ inline double wave_reduce(int kind, double v) {
    const double id = stat_identity(kind);
    v = stat_op(kind, v, dpp_all<0xB1>(v));            // quad_perm [1,0,3,2]
    v = stat_op(kind, v, dpp_all<0x4E>(v));            // quad_perm [2,3,0,1]
    v = stat_op(kind, v, dpp_all<0x141>(v));           // row_half_mirror
    v = stat_op(kind, v, dpp_all<0x140>(v));           // row_mirror
    v = stat_op(kind, v, dpp_d<0x142, 0xa>(v, id));    // row_bcast:15 into rows 1, 3
    v = stat_op(kind, v, dpp_d<0x143, 0xc>(v, id));    // row_bcast:31 into rows 2, 3
    return v;
}

// Per-tile partial statistics are stored [tile][NSTAT]: the NSTAT values of a
// tile are contiguous (one 160-byte record, read with 16-byte loads).
__device__ inline const double *part_tile(const double *part, long long tile) { return part + tile * NSTAT; }

// Reduction of the per-tile partial statistics of tiles [tile0, tile0+ntiles) in a
// fixed order: in blocks of PRE x 64 tiles, of which lane l of a wave takes tiles
// l, l + 64, ... in turn, then the wave's tree; the blocks in turn.  A wave of the
// workgroup reduces the rows of some of the (mesh, component) triples over all tiles
// (and wave 0 and 1 one of the wave-speed rows): with every wave reducing all 18 rows of a third of the tiles, the trees
// were the longest phase of a stage launch.  Split in two so that the loads of the
// first PRE tiles per lane are issued together with the kernel's other independent
// loads (5 x 64 tiles hold the 257 columns of a mesh that fills the chip).  More blocks
// are taken a barrier apart: every wave reads a part of each line of the records, and
// waves that drift from each other fetch the lines three times over (Euler P2 at
// 3125 tiles: 188 us per stage without it, 155 with it).
template <int NT, int NC>
struct Partials {
    static constexpr int NS = 6 * NC + 2, NW = (NT + WAVE - 1) / WAVE;
    static constexpr int PRE = NT <= 2 * WAVE ? 3 : 5;       // tiles of 32 serve meshes of up to 129 columns
    static constexpr int TPW = (2 * NC + NW - 1) / NW;       // triples per wave
    double v[PRE][3 * TPW], beta[PRE];
};

template <int NT, int NC>
__device__ inline int first_triple() {
    return __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE) * Partials<NT, NC>::TPW;
}
// Row of a triple's sum in a record (max and min follow).
template <int NC>
__device__ inline int triple_row(int tr) { return NC == 3 ? 3 * tr : 9 * tr; }

template <int NT, int NC>
__device__ __forceinline__ void load_triples(const double *rec, int tr0, double (&v)[3 * Partials<NT, NC>::TPW]) {
    constexpr int TPW = Partials<NT, NC>::TPW;
    if constexpr (NC == 3 && TPW == 2) {             // 48 bytes, 16-byte aligned
        const double2 *q = reinterpret_cast<const double2 *>(rec + 3 * tr0);
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const double2 x = q[j];
            v[2 * j] = x.x;
            v[2 * j + 1] = x.y;
        }
    } else {
#pragma unroll
        for (int k = 0; k < TPW; ++k)
#pragma unroll
            for (int j = 0; j < 3; ++j) v[3 * k + j] = rec[triple_row<NC>(min(tr0 + k, 2 * NC - 1)) + j];
    }
}

template <int NT, int NC>
__device__ __forceinline__ void load_partials(const double *part, int tile0, int ntiles, bool beta, Partials<NT, NC> &p) {
    using P = Partials<NT, NC>;
    const int lane = threadIdx.x % WAVE, tr0 = first_triple<NT, NC>();
    const int brow = ST_BETA + (tr0 > 0);
#pragma unroll
    for (int i = 0; i < P::PRE; ++i) {
        if (i * WAVE >= ntiles || tr0 >= 2 * NC) break;      // uniform
        const double *rec = part_tile(part, tile0 + min(lane + i * WAVE, ntiles - 1));
        load_triples<NT, NC>(rec, tr0, p.v[i]);
        if (beta) p.beta[i] = rec[brow];
    }
}

// The rest of the reduction; the rows (triples in order, then the wave speeds when
// beta) are in out[0 .. NS) (LDS) after the barrier that ends it.
template <int NT, int NC>
__device__ __forceinline__ void finish_partials(Partials<NT, NC> &p, const double *part, int tile0, int ntiles, bool beta,
                                                double *out) {
    using P = Partials<NT, NC>;
    constexpr int TPW = P::TPW, BLOCK = P::PRE * WAVE;
    const int lane = threadIdx.x % WAVE, tr0 = first_triple<NT, NC>();
    if (tr0 < 2 * NC) {                                      // uniform
        double tot[3 * TPW], totb = -INFINITY;               // (in lane 63)
#pragma unroll
        for (int r = 0; r < 3 * TPW; ++r) tot[r] = stat_identity(r % 3);
        for (int t0 = 0;;) {
            double acc[3 * TPW], b = -INFINITY;
#pragma unroll
            for (int r = 0; r < 3 * TPW; ++r) acc[r] = stat_identity(r % 3);
#pragma unroll
            for (int i = 0; i < P::PRE; ++i) {
                if (i * WAVE >= ntiles - t0) break;          // uniform
                const bool in = lane + i * WAVE < ntiles - t0;
#pragma unroll
                for (int r = 0; r < 3 * TPW; ++r)
                    acc[r] = stat_op(r % 3, acc[r], in ? p.v[i][r] : stat_identity(r % 3));
                if (beta) b = max_d(b, in ? p.beta[i] : -INFINITY);
            }
#pragma unroll
            for (int r = 0; r < 3 * TPW; ++r) {
                acc[r] = wave_reduce(r % 3, acc[r]);
                tot[r] = t0 == 0 ? acc[r] : stat_op(r % 3, tot[r], acc[r]);
            }
            if (beta) totb = max_d(totb, wave_reduce(1, b));
            t0 += BLOCK;
            if (t0 >= ntiles) break;                         // uniform
            __syncthreads();
            load_partials<NT, NC>(part, tile0 + t0, ntiles - t0, beta, p);
        }
        if (lane == WAVE - 1) {
#pragma unroll
            for (int r = 0; r < 3 * TPW; ++r)
                if (tr0 + r / 3 < 2 * NC) out[3 * tr0 + r] = tot[r];
            if (beta && tr0 <= TPW) out[6 * NC + (tr0 > 0)] = totb;
        }
    } else {
        for (int t0 = BLOCK; t0 < ntiles; t0 += BLOCK) __syncthreads();
    }
    __syncthreads();
}

template <int NT, int NC>
__device__ __forceinline__ void reduce_instance(const double *part, int tile0, int ntiles, bool beta, double *out) {
    Partials<NT, NC> p;
    load_partials<NT, NC>(part, tile0, ntiles, beta, p);
    finish_partials<NT, NC>(p, part, tile0, ntiles, beta, out);
}

}  // namespace oecdg
