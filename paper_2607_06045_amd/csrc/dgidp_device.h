// Device code that the two files of stage kernels share: dgidp_kernels.hip (positivity) and
// dgidp_local.hip (local bounds), which keeps an arithmetic of its own.  R, where it is a
// parameter, is the file's reciprocal (R::rcp) and its operator tables (R::tab): constant
// memory belongs to one file, so each has its own.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>

#include "dgidp_internal.h"

namespace dgidp {
namespace {

// Workgroups are dispatched round-robin over the 8 XCDs; give each XCD a
// contiguous range of element batches so that face neighbours share its L2.
__device__ __forceinline__ int xcd_batch(int bid, int nb)
{
    const int q = nb >> 3, r = nb & 7;
    const int x = bid & 7, j = bid >> 3;
    return (x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q) + j;
}
// the same ranges walked from their ends: a kernel that reads what the
// previous one wrote takes the most recently written batches, the ones most
// likely still held by the memory-side cache, first
__device__ __forceinline__ int xcd_batch_rev(int bid, int nb)
{
    const int q = nb >> 3, r = nb & 7;
    const int x = bid & 7, j = bid >> 3;
    const int len = x < r ? q + 1 : q;
    return (x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q) + len - 1 - j;
}

// ---------------------------------------------------------------------------
// arithmetic helpers
// ---------------------------------------------------------------------------
// 1/y from the hardware estimate r (relative error e = 1 - y r of about 2^-23)
// and the third-order step r (1 + e + e^2), whose own error is e^3 (about 1 ulp
// after rounding); used on the paths every node takes, where y > 0.  For 2^-1022 <=
// |y| <= 2^1022 only: below, r is infinite and e NaN, so a quotient by an increment,
// which may be subnormal, is a division instead
struct Rcp3 {
    static __device__ __forceinline__ double rcp(double y)
    {
        const double r = __builtin_amdgcn_rcp(y);
        const double e = fma(-y, r, 1.0);
        return fma(r, fma(e, e, e), r);
    }
};

// the same from the estimate and two Newton steps (the local modes' arithmetic)
struct Rcp2 {
    static __device__ __forceinline__ double rcp(double y)
    {
        double r = __builtin_amdgcn_rcp(y);
        double e = fma(-y, r, 1.0);
        r = fma(r, e, r);
        e = fma(-y, r, 1.0);
        return fma(r, e, r);
    }
};

// sqrt(y) for y >= 0 (normal or zero): the hardware reciprocal square root,
// one step of the coupled Newton iteration for sqrt y and 1 / (2 sqrt y), then
// a Newton correction of the root (about 1 ulp).  y = 0 gives 0, y < 0 or NaN
// gives NaN.
__device__ __forceinline__ double fsqrt(double y)
{
    const double r = __builtin_amdgcn_rsq(y);
    double g = y * r, h = 0.5 * r;
    const double e = fma(-g, h, 0.5);
    g = fma(g, e, g);
    h = fma(h, e, h);
    g = fma(fma(-g, g, y), h, g);
    return y == 0.0 ? 0.0 : g;
}

// two FP32 values in one FP64 LDS slot (register moves only)
struct F2 {
    float x, y;
};
__device__ __forceinline__ double pack2(float x, float y)
{
    return __hiloint2double(__float_as_int(y), __float_as_int(x));
}
__device__ __forceinline__ F2 unpack2(double d)
{
    return F2{__int_as_float(__double2loint(d)), __int_as_float(__double2hiint(d))};
}

struct NodeP {
    double u[4];
    double r, v1, v2, p, c;
};

template <class R>
__device__ __forceinline__ void make_node(NodeP& s, double g)
{
    const double ir = R::rcp(s.u[0]);
    s.r = s.u[0];
    s.v1 = s.u[1] * ir;
    s.v2 = s.u[2] * ir;
    s.p = (g - 1.0) * (s.u[3] - 0.5 * (s.u[1] * s.v1 + s.u[2] * s.v2));
    s.c = fsqrt(g * s.p * ir);
}

// Ghost state across a boundary face f (0 x-, 1 x+, 2 y-, 3 y+) of the interior
// node s; the outward normal is the axis f / 2, negative on even faces.  Wall:
// the normal momentum reversed.  Characteristic, by the outward normal velocity
// vn and sound speed c of s: the exterior state x if vn <= -c; x's density and
// velocity with s's pressure if vn <= 0; s's density and velocity with x's
// pressure if vn < c; else s.  Outflow: s.
__device__ __forceinline__ void boundary_ghost(int kind, const double* x, const NodeP& s, int f,
                                               double g, double* gu)
{
    const int d = f >> 1;
#pragma unroll
    for (int v = 0; v < 4; ++v) gu[v] = s.u[v];
    if (kind == DGIDP_BC_WALL) {  // (constant indices keep gu in registers)
        if (d == 0) gu[1] = -s.u[1];
        else gu[2] = -s.u[2];
        return;
    }
    if (kind != DGIDP_BC_CHARACTERISTIC) return;
    const double vn = (f & 1) ? (d == 0 ? s.v1 : s.v2) : -(d == 0 ? s.v1 : s.v2);
    if (vn >= s.c) return;
    if (vn <= -s.c) {
#pragma unroll
        for (int v = 0; v < 4; ++v) gu[v] = x[v];
        return;
    }
    const double ixr = 1.0 / x[0], xv1 = x[1] * ixr, xv2 = x[2] * ixr;
    if (vn <= 0.0) {
        gu[0] = x[0];
        gu[1] = x[0] * xv1;
        gu[2] = x[0] * xv2;
        gu[3] = s.p / (g - 1.0) + 0.5 * x[0] * (xv1 * xv1 + xv2 * xv2);
    } else {
        const double xp = (g - 1.0) * (x[3] - 0.5 * (x[1] * xv1 + x[2] * xv2));
        gu[3] = xp / (g - 1.0) + 0.5 * s.r * (s.v1 * s.v1 + s.v2 * s.v2);
    }
}

template <class R>
__device__ __forceinline__ double pressure(const double* u, double g)
{
    return (g - 1.0) * (u[3] - 0.5 * (u[1] * u[1] + u[2] * u[2]) * R::rcp(u[0]));
}

// local Lax-Friedrichs flux across a face (eq. FVmethod): 1/2 (f_n(u_L) + f_n(u_R)) -
// 1/2 lambda (u_R - u_L), lambda = max(|v_n| + c) of the two states.
// Normal direction d and side are run-time values (lanes of a wave hold
// different faces): this element's state `own`, the other side's state `o`,
// own_low = this element is on the low side.  Branch free, so a wave evaluates
// one flux body whatever mix of faces its lanes hold.
__device__ __forceinline__ void llf_face(int d, bool own_low, const NodeP& own, const NodeP& o,
                                         double* F)
{
    const bool dx = d == 0;
    const double va = dx ? own.v1 : own.v2, vb = dx ? o.v1 : o.v2;
    const double lam = fmax(fabs(va) + own.c, fabs(vb) + o.c);
    const double hl = own_low ? 0.5 * lam : -0.5 * lam;
    double fa[4], fb[4];
    fa[0] = own.r * va;
    fa[1] = own.u[1] * va + (dx ? own.p : 0.0);
    fa[2] = own.u[2] * va + (dx ? 0.0 : own.p);
    fa[3] = (own.u[3] + own.p) * va;
    fb[0] = o.r * vb;
    fb[1] = o.u[1] * vb + (dx ? o.p : 0.0);
    fb[2] = o.u[2] * vb + (dx ? 0.0 : o.p);
    fb[3] = (o.u[3] + o.p) * vb;
#pragma unroll
    for (int v = 0; v < 4; ++v) F[v] = 0.5 * (fa[v] + fb[v]) - hl * (o.u[v] - own.u[v]);
}

// LLF flux on a mortar node between the interpolated large-face state ui and
// the small-face state us.  An interpolated state outside the admissible set
// leaves the high-order mortar flux undefined (NaN); the mortar limiter then
// keeps the low-order flux for the whole mortar.
__device__ __forceinline__ void mortar_flux(int d, bool large_low, const NodeP& ui, const NodeP& us,
                                            double* F)
{
    if (!(ui.r > 0.0) || !(ui.p > 0.0)) {
        const double nan = __builtin_nan("");
        F[0] = F[1] = F[2] = F[3] = nan;
        return;
    }
    llf_face(d, large_low, ui, us, F);
}

__device__ __forceinline__ float lnmeanf(float x, float y, float lx, float ly)
{
    const float s = x + y, d = x - y;
    if (d * d < 1e-2f * (s * s)) {
        const float is = __builtin_amdgcn_rcpf(s);
        const float f2 = d * d * is * is;
        return s * __builtin_amdgcn_rcpf(2.0f + f2 * (2.0f / 3.0f + f2 * (2.0f / 5.0f + f2 * (2.0f / 7.0f))));
    }
    return d * __builtin_amdgcn_rcpf(lx - ly);
}

__device__ __forceinline__ float inv_lnmeanf(float x, float y, float lx, float ly)
{
    const float s = x + y, d = x - y;
    if (d * d < 1e-2f * (s * s)) {
        const float is = __builtin_amdgcn_rcpf(s);
        const float f2 = d * d * is * is;
        return (2.0f + f2 * (2.0f / 3.0f + f2 * (2.0f / 5.0f + f2 * (2.0f / 7.0f)))) * is;
    }
    return (lx - ly) * __builtin_amdgcn_rcpf(d);
}

// ---------------------------------------------------------------------------
// pressure blending factor: largest theta in [0,1] with rho(u0 + theta dc) > 0
// and p(u0 + theta dc) >= pt.  For rho > 0, p >= pt is
// g(theta) = (E - pt/(gamma-1)) rho - |m|^2 / 2 >= 0, a quadratic in theta whose
// admissible set along the ray is an interval [0, theta*] (p is concave).
// ---------------------------------------------------------------------------
// The ray's direction is S c (S = Gamma = 4 for the volume faces' increments,
// 1 otherwise): a power of two, so that S c is formed exactly inside the
// fused multiply-adds.
template <int S = 1>
__device__ __forceinline__ double theta_p(const double* u0, const double* c, double pt, double ig1)
{
    const double e0 = u0[3] - pt * ig1;
    const double g0 = u0[0] * e0 - 0.5 * (u0[1] * u0[1] + u0[2] * u0[2]);
    if (!(g0 > 0.0) || !(u0[0] > 0.0)) return 0.0;
    // full step admissible: the interval contains [0, 1]
    const double r1 = fma((double)S, c[0], u0[0]);
    if (r1 > 0.0) {
        const double m1 = fma((double)S, c[1], u0[1]), m2 = fma((double)S, c[2], u0[2]);
        const double g1v = fma((double)S, c[3], e0) * r1 - 0.5 * (m1 * m1 + m2 * m2);
        if (g1v >= 0.0) return 1.0;
    }
    const double dc[4] = {S * c[0], S * c[1], S * c[2], S * c[3]};
    const double g1 = dc[0] * e0 + u0[0] * dc[3] - (u0[1] * dc[1] + u0[2] * dc[2]);
    const double g2 = dc[0] * dc[3] - 0.5 * (dc[1] * dc[1] + dc[2] * dc[2]);
    double root = 1.0;
    if (g2 == 0.0) {
        if (g1 < 0.0) root = fmin(root, -g0 / g1);
    } else {
        const double disc = g1 * g1 - 4.0 * g2 * g0;
        if (disc >= 0.0) {
            const double sq = sqrt(disc);
            const double qq = -0.5 * (g1 + (g1 >= 0.0 ? sq : -sq));
            const double ra = qq / g2, rb = g0 / qq;
            if (ra > 0.0) root = fmin(root, ra);
            if (rb > 0.0) root = fmin(root, rb);
        }
    }
    if (dc[0] < 0.0) root = fmin(root, -u0[0] / dc[0]);
    return root;
}

// the limiter aims at the bounds raised by this relative margin so that the
// rounding of the final sums cannot cross the bounds themselves
constexpr double kMargin = 1.0 + 0x1p-40;
// the mortar correction aims at half that margin: a node that the volume
// limiter left on its target keeps 2^-41 of room, instead of a zero or one
// mortar factor decided by the sign of a rounding error
constexpr double kMarginMortar = 1.0 + 0x1p-41;
// the local bounds hold for the low-order state only up to rounding (it is a
// convex combination of bar states in exact arithmetic): the bound check allows
// this relative slack for them
constexpr double kLocalTol = 1e-12;

// ---------------------------------------------------------------------------
// statistics
// ---------------------------------------------------------------------------
template <typename TT>
__device__ __forceinline__ TT wave_sum(TT v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

__device__ __forceinline__ double wave_min(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o, 64));
    return v;
}

__device__ __forceinline__ double wave_max(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    return v;
}

// accumulation of per-thread statistics; every lane of the wave must call it.
// Counts are taken from lane masks (per lane: inad and viol 0 or 1); the two
// floating-point reductions run only in waves where some lane has a value to
// contribute, and only such waves touch memory, at the accumulator of their
// block.  The number of faces and mortars, by which the means divide, follows
// from the mesh and is not counted here.  Bound: the device-scope atomics that
// meet at one address are served one after another, about 10 ns each; with one
// accumulator and two counts per wave the 22,156-leaf N = 3 stage took 142 us
// with statistics against 20 us without, with them spread and the counts gone
// 21.4 us; the blended stage of the 22,732-leaf jet 157 and 43 us, the N = 4
// local one of the 20,480-element double Mach reflection 305 and 74 us.
__device__ __forceinline__ void push_stats(DevStats* st, unsigned long long inad,
                                           unsigned long long viol, double thmin, double asum, bool mortar)
{
    const unsigned long long ninad = __popcll(__ballot(inad != 0));
    const unsigned long long nviol = __popcll(__ballot(viol != 0));
    const bool any_a = __ballot(asum != 0.0) != 0, any_t = __ballot(thmin < 1.0) != 0;
    if (any_a) asum = wave_sum(asum);
    if (any_t) thmin = wave_min(thmin);
    if ((threadIdx.x & 63) == 0) {
        DevStats* s = st + blockIdx.x % kStatSpread;
        if (ninad) atomicAdd(&s->fv_inadmissible, ninad);
        if (nviol) atomicAdd(&s->violations, nviol);
        if (any_a) atomicAdd(mortar ? &s->alpha_mort_sum : &s->alpha_vol_sum, asum);
        if (any_t) {
            unsigned long long bits = __double_as_longlong(fmax(thmin, 0.0));
            atomicMin(mortar ? &s->theta_mort_min_bits : &s->theta_vol_min_bits, bits);
        }
    }
}

// ---------------------------------------------------------------------------
// mortar corrections: one thread per slot, after the stage's mortar elements are
// written: a launch of their own (k_mortar), or the first blocks of the second launch of a
// positivity-limited stage.
// ---------------------------------------------------------------------------
struct MortarArgs {
    const double* slot;
    const int* snode;
    const int* spart;
    int M;
    double* uout;
    double b;
    double gamma;
    int limiter;
    DevStats* st;
};

// factor of mortar S: the minimum of its slots' node factors; combined
// limiting blends the positivity and the local minimum with the largest
// indicator of the mortar's three elements.  LOC: one of the modes with local bounds
template <int N, bool LOC>
__device__ __forceinline__ double mortar_theta(const double* __restrict__ slot, int S, int limiter)
{
    constexpr int NS = 3 * (N + 1);
    const bool comb = LOC && limiter == DGIDP_LIMIT_COMBINED;
    double t = 1.0, tl = 1.0, w = 0.0;
#pragma unroll
    for (int j = 0; j < NS; ++j) {
        const double* R = slot + ((size_t)S * NS + j) * kSlotW;
        t = fmin(t, R[8]);
        if (comb) {
            tl = fmin(tl, R[13]);
            w = fmax(w, R[14]);
        }
    }
    return comb ? (1.0 - w) * t + w * tl : t;
}

// correction of slot s (past the last slot: none); all lanes of a wave call it
template <int N, class R, bool LOC>
__device__ __forceinline__ void mortar_slot(const MortarArgs& A, int s)
{
    constexpr int n = N + 1, NN = n * n, NS = 3 * n;
    const double* __restrict__ slot = A.slot;
    double* uout = A.uout;
    unsigned long long viol = 0;
    double asum = 0.0, thmin = 1.0;
    if (s < A.M * NS) {
        const int S = s / NS;
        // every load that needs no other load first: slot factors of the
        // mortar, this slot's record, its node and its partner
        const double* own = slot + (size_t)s * kSlotW;
        const int part = A.spart[s];
        const int node = A.snode[s];
        double rec[11];
#pragma unroll
        for (int i = 0; i < 11; ++i) rec[i] = own[i];
        double t = mortar_theta<N, LOC>(slot, S, A.limiter);
        const int e = node / NN, q = node - e * NN;
        double uo[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) uo[v] = uout[((size_t)e * 4 + v) * NN + q];
        if (s == S * NS) {
            asum = 1.0 - t;
            thmin = t;
        }
        bool apply = true;
        double corr[4] = {0, 0, 0, 0};
        if (t != 0.0)
#pragma unroll
            for (int v = 0; v < 4; ++v) corr[v] = t * rec[4 + v];
        if (part >= 0) {
            const int S2 = part / NS;
            if (S2 < S) {
                apply = false;  // the lower-numbered mortar applies both corrections
            } else {
                const double t2 = mortar_theta<N, LOC>(slot, S2, A.limiter);
                if (t2 != 0.0)
#pragma unroll
                    for (int v = 0; v < 4; ++v) corr[v] += t2 * slot[(size_t)part * kSlotW + 4 + v];
            }
        }
        if (apply) {
            double w[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                uout[((size_t)e * 4 + v) * NN + q] = uo[v] + A.b * corr[v];
                w[v] = rec[v] + corr[v];
            }
            if (LOC && A.limiter != DGIDP_LIMIT_COMBINED) {
                const double rhi = own[11], lsm = own[12];
                const double pw = pressure<R>(w, A.gamma);
                if (!(w[0] >= rec[9] * (1.0 - kLocalTol)) || w[0] > rhi * (1.0 + kLocalTol) ||
                    pw < rec[10] || !(log(pw) - A.gamma * log(w[0]) >= lsm - kLocalTol))
                    viol = 1;
            } else if (A.limiter != DGIDP_LIMIT_NONE &&
                       (w[0] < rec[9] || pressure<R>(w, A.gamma) < rec[10] || w[0] != w[0])) {
                viol = 1;
            }
        }
    }
    if (A.st) push_stats(A.st, 0, viol, thmin, asum, true);
}

template <int N, class R, bool LOC>
__global__ __launch_bounds__(256) void k_mortar(MortarArgs A)
{
    mortar_slot<N, R, LOC>(A, blockIdx.x * blockDim.x + threadIdx.x);
}

// the launch of k_mortar (mortars > 0)
template <class R, bool LOC>
int run_mortar(int N, const MortarArgs& A, hipStream_t s)
{
    const dim3 grid((A.M * 3 * (N + 1) + 255) / 256);
    if (N == 3) hipLaunchKernelGGL((k_mortar<3, R, LOC>), grid, dim3(256), 0, s, A);
    else if (N == 4) hipLaunchKernelGGL((k_mortar<4, R, LOC>), grid, dim3(256), 0, s, A);
    else return -1;
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// ---------------------------------------------------------------------------
// what both stage kernels are given: the common members of their arguments
// ---------------------------------------------------------------------------
template <class Args>
void set_stage(Args& A, const DevMesh& m, const KernelParams& kp, const double* uin, const double* un, double* uout,
               double a, double b, const DtSource& dt, DevStats* st)
{
    A.uin = uin;
    A.un = un;
    A.uout = uout;
    A.a = a;
    A.b = b;
    A.dt = dt.dt;
    A.dtmax = dt.dtmax;
    A.cfl = dt.cfl;
    A.dt_out = dt.dt_out;
    A.fnbr = m.fnbr;
    A.fnbr2 = m.fnbr2;
    A.fmort = m.fmort;
    A.mort = m.mort;
    A.h = m.h;
    A.slot = m.slot;
    A.bkind = m.bkind;
    A.bext = m.bext;
    A.E = m.E;
    A.gamma = kp.gamma;
    A.beta = kp.beta;
    A.ig1 = 1.0 / (kp.gamma - 1.0);
    A.rev = 0;
    A.limiter = kp.limiter;
    A.vflux = kp.vflux;
    A.st = st;
}

// node (a, b) at position k along face f
template <int N>
__device__ __forceinline__ int face_q(int f, int k)
{
    constexpr int n = N + 1;
    // x faces (0, 1) run along a column, y faces (2, 3) along a row; the odd
    // face of each pair is N columns or N rows further on
    const int hi = f & 1;
    return f < 2 ? k * n + hi * N : k + hi * (N * n);
}

template <int N>
__device__ __forceinline__ void load_u(const double* u, int e, int q, double* w)
{
    constexpr int NN = (N + 1) * (N + 1);
    // one address per node; the variables at constant offsets (index < 2^30, mesh limit)
    const double* p = u + ((unsigned)e * 4u * NN + (unsigned)q);
#pragma unroll
    for (int v = 0; v < 4; ++v) w[v] = p[v * NN];
}

template <int N, class R>
__device__ __forceinline__ void load_node(const double* u, int e, int q, NodeP& s, double g)
{
    load_u<N>(u, e, q, s.u);
    make_node<R>(s, g);
}

// ---------------------------------------------------------------------------
// time step: per node sum_j 2 d_ij / m_i (or the low-order estimate), block max
// ---------------------------------------------------------------------------
struct DtArgs {
    const double* u;
    const int* fnbr;
    const int* fnbr2;
    const int* fmort;
    const double* h;
    const int8_t* bkind;
    const double* bext;
    int E;
    double gamma;
    int mode;
    unsigned long long* acc;    // running maximum, bits of a non-negative double
    unsigned long long* other;  // the other accumulator, cleared for the next step
};

__device__ __forceinline__ double wave_speed(const NodeP& s, int d)
{
    return fabs(d == 0 ? s.v1 : s.v2) + s.c;
}

// the block's maximum (of its waves' in red) into one of the accumulators
template <int NW>
__device__ __forceinline__ void dt_merge(const DtArgs& A, const double* red)
{
    if (threadIdx.x == 0) {
        // non-negative doubles order like their bit patterns; NaN and zero
        // maxima are left out, as fmax would
        double m = red[0];
#pragma unroll
        for (int w = 1; w < NW; ++w) m = fmax(m, red[w]);
        if (m > 0.0)
            atomicMax(A.acc + (blockIdx.x % kDtSpread) * kDtStride,
                      (unsigned long long)__double_as_longlong(m));
    }
    if (blockIdx.x == 0 && threadIdx.x < kDtSpread) A.other[threadIdx.x * kDtStride] = 0ull;
}

// the dt kernel: kDtBlock = 256-thread blocks (16 elements at N = 3, 10 at N = 4), fewer
// blocks and so fewer atomics than the stage kernel's geometry
// threads per block of the dt kernel (whole elements per block)
constexpr int kDtBlock = 256;

template <int N>
struct DtGeo {
    static constexpr int n = N + 1, NN = n * n, NFN = 4 * n;
    static constexpr int BS = kDtBlock, EPB = BS / NN, NT = EPB * NN;
};

template <int N, class R>
__global__ __launch_bounds__(kDtBlock) void k_dt(DtArgs A)
{
    using G = DtGeo<N>;
    constexpr int n = G::n, NN = G::NN, EPB = G::EPB, NT = G::NT, NFN = G::NFN;
    __shared__ double sL[EPB][2][NN];
    __shared__ double sF[EPB][NFN];
    __shared__ double sMl[EPB][8 * n];  // wave speeds across mortars, staged per position
    constexpr int NW = G::BS / 64;  // waves per block
    __shared__ double sRed[NW];
    __shared__ double sTw[2][n];  // LGL weights and their reciprocals, read per lane
    const Tab<N>& tb = R::template tab<N>();
    const double g = A.gamma;
    const int tid = threadIdx.x;
    const int le = tid / NN, q = tid - le * NN, a = q % n, b = q / n;
    // (contiguous element ranges per XCD, as in the stage kernel: the face
    // neighbours' traces are then mostly in the same L2; each range from its
    // end, where the stage before this kernel finished writing)
    const int e = xcd_batch_rev(blockIdx.x, gridDim.x) * EPB + le;
    const bool act = tid < NT && e < A.E;
    if (tid < n) {
        sTw[0][tid] = tb.w[tid];
        sTw[1][tid] = tb.winv[tid];
    }
    const bool idp = A.mode != DGIDP_DT_LOWORDER;
    const bool fnode = act && idp && q < NFN;
    const int ff = q / n, fk = q - (q / n) * n, dff = ff >> 1;
    double hx = 1.0, hy = 1.0, lo_nb = 0.0;
    int code = -1, nb = 0, nb2 = -1;
    if (act) {
        if (fnode) {  // face tables first: the neighbour loads depend on them
            code = A.fmort[e * 4 + ff];
            nb = A.fnbr[e * 4 + ff];
            nb2 = A.fnbr2[e * 4 + ff];
        }
        NodeP me;
        load_node<N, R>(A.u, e, q, me, g);
        hx = A.h[2 * e];
        hy = A.h[2 * e + 1];
        sL[le][0][q] = wave_speed(me, 0);
        sL[le][1][q] = wave_speed(me, 1);
        if (fnode) {
            NodeP o;
            if (code >= -1) {
                load_node<N, R>(A.u, nb, face_q<N>(ff ^ 1, fk), o, g);
            } else {  // boundary: the ghost state of the face node
                const int j = (-2 - code) * n + fk;
                double x[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) x[v] = A.bext[(size_t)j * 4 + v];
                NodeP s;
                load_node<N, R>(A.u, e, face_q<N>(ff, fk), s, g);
                boundary_ghost(A.bkind[j], x, s, ff, g, o.u);
                make_node<R>(o, g);
            }
            lo_nb = wave_speed(o, dff);
            if (code >= 0) {
                // mortar: stage the wave speeds of the other side at position fk
                // (large side: both small elements; small side: the large one)
                sMl[le][(ff * 2) * n + fk] = lo_nb;
                if (!fm_small(code)) {
                    NodeP o2;
                    load_node<N, R>(A.u, nb2, face_q<N>(ff ^ 1, fk), o2, g);
                    sMl[le][(ff * 2 + 1) * n + fk] = wave_speed(o2, dff);
                }
            }
        }
    }
    __syncthreads();
    if (fnode) {
        // edges across face ff at position fk: 2 |c_ij| lambda_ij
        const double hf = ff < 2 ? hy : hx;
        const double lm = sL[le][dff][face_q<N>(ff, fk)];
        double sum = 0.0;
        if (code < 0) {
            sum = 0.5 * sTw[0][fk] * hf * fmax(lm, lo_nb);
        } else if (!fm_small(code)) {
#pragma unroll
            for (int hh = 0; hh < 2; ++hh)
#pragma unroll
                for (int l = 0; l < n; ++l) {
                    const double wt = tb.Wt[fk][hh * n + l];
                    if (wt == 0.0) continue;
                    sum += 2.0 * wt * hf * 0.25 * fmax(lm, sMl[le][(ff * 2 + hh) * n + l]);
                }
        } else {
            const int hh = fm_half(code);
#pragma unroll
            for (int j = 0; j < n; ++j) {
                const double wt = tb.Wt[j][hh * n + fk];
                if (wt == 0.0) continue;
                sum += 2.0 * wt * (2.0 * hf) * 0.25 * fmax(lm, sMl[le][(ff * 2) * n + j]);
            }
        }
        sF[le][q] = sum;
    }
    __syncthreads();
    double s = 0.0;
    if (act) {
        const double lx = sL[le][0][q], ly = sL[le][1][q];
        if (!idp) {
            s = (N + 1) * (lx * R::rcp(hx) + ly * R::rcp(hy));
        } else {
            // edges along x carry 2 |c| = w_b h_y / 2, along y w_a h_x / 2
            const double cx = 0.5 * sTw[0][b] * hy, cy = 0.5 * sTw[0][a] * hx;
            double sum = 0.0;
            if (a > 0) sum += cx * fmax(lx, sL[le][0][q - 1]);
            if (a < N) sum += cx * fmax(lx, sL[le][0][q + 1]);
            if (b > 0) sum += cy * fmax(ly, sL[le][1][q - n]);
            if (b < N) sum += cy * fmax(ly, sL[le][1][q + n]);
            if (a == 0) sum += sF[le][0 * n + b];
            if (a == N) sum += sF[le][1 * n + b];
            if (b == 0) sum += sF[le][2 * n + a];
            if (b == N) sum += sF[le][3 * n + a];
            s = sum * (4.0 * R::rcp(hx * hy)) * sTw[1][a] * sTw[1][b];
        }
    }
    s = wave_max(s);
    if ((tid & 63) == 0) sRed[tid >> 6] = s;
    __syncthreads();
    dt_merge<NW>(A, sRed);
}

inline DtArgs dt_args(const DevMesh& m, const KernelParams& kp, const double* u, int mode, unsigned long long* acc,
                      unsigned long long* other)
{
    DtArgs A;
    A.u = u;
    A.fnbr = m.fnbr;
    A.fnbr2 = m.fnbr2;
    A.fmort = m.fmort;
    A.bkind = m.bkind;
    A.bext = m.bext;
    A.h = m.h;
    A.E = m.E;
    A.gamma = kp.gamma;
    A.mode = mode;
    A.acc = acc;
    A.other = other;
    return A;
}

// the launch of k_dt
template <class R>
int run_dt(int N, const DtArgs& A, hipStream_t s)
{
    if (N == 3)
        hipLaunchKernelGGL((k_dt<3, R>), dim3((A.E + DtGeo<3>::EPB - 1) / DtGeo<3>::EPB), dim3(kDtBlock), 0, s, A);
    else if (N == 4)
        hipLaunchKernelGGL((k_dt<4, R>), dim3((A.E + DtGeo<4>::EPB - 1) / DtGeo<4>::EPB), dim3(kDtBlock), 0, s, A);
    else return -1;
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// dt = cfl / (the maximum over the dt kernel's accumulators), once per step:
// one wave reads the kDtSpread accumulators; the stage kernels then read the
// stored value (a per-wave reduction in every block of the first stage would
// read the kDtSpread cache lines once per wave).  On a small mesh, of fewer than kFinalMin
// element batches, the extra launch costs more than that reduction.
constexpr int kFinalMin = 16384;
static_assert(kDtSpread == 64, "one wave reduces the dt accumulators");
__global__ __launch_bounds__(64) void k_dt_final(const unsigned long long* dtmax, double cfl, double* dt_out,
                                                 DevStats* st)
{
    const double m = wave_max(__longlong_as_double((long long)dtmax[threadIdx.x * kDtStride]));
    if (threadIdx.x == 0) {
        const double dt = cfl / m;
        *dt_out = dt;
        if (st) st->dt = dt;
    }
}

}  // namespace
}  // namespace dgidp
