// HIP kernels of the limiting modes with local bounds (from bar states or from the low-order
// solution, alone or blended with positivity).
//
// These modes keep an arithmetic of their own, operation by operation, apart from
// dgidp_kernels.hip's.  Where the density or the entropy is constant along a
// direction, a node's local bounds have no width, its antidiffusive increment there
// is a rounding error, and their quotient, the node's factor, is anywhere in [0, 1]; that
// factor also multiplies the node's increments in the other direction.  So any other order
// of the operations, though as accurate, gives other solutions: with the forms of
// dgidp_kernels.hip a shear layer's transverse momentum changed by up to 5e-3 of
// its largest value in five steps with local bounds alone; with the blend, whose weights
// are above zero at shocks only, a top-hat blast in gas of constant density by up to 4e-5
// and a pressure jump beside a shear by 8e-8, though blasts, quadrants and the jet only by
// 1e-13; the FP32 fluxes' rounding by 1e-7 in the jet.  The faster forms were left out for
// that.  Timed in turn: five steps of the 22,156-leaf blast 715 us with them and 940 here
// with bar states, 812 and 1,350 with the low-order solution (1,222 since, see MODE_LOWSOL);
// three of the blended 22,732-leaf jet 570 and 680.
//
// k_stage is as described in dgidp_kernels.hip, with these differences: logarithms of
// density and rho / p per node, the pair fluxes telescoped through LDS, the library's
// logarithm, exponential and roots.  k_dt and k_shock_indicator belong to the same
// arithmetic, since a stage's rounding errors follow from dt and the weights too.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "dgidp_device.h"

namespace dgidp {
namespace local {

__constant__ Tab<3> c_tab3;
__constant__ Tab<4> c_tab4;

template <int N>
__device__ __forceinline__ const Tab<N>& T();
template <>
__device__ __forceinline__ const Tab<3>& T<3>() { return c_tab3; }
template <>
__device__ __forceinline__ const Tab<4>& T<4>() { return c_tab4; }

int upload_tables(int N, const void* host_tab, size_t bytes)
{
    hipError_t e = hipErrorInvalidValue;
    if (N == 3 && bytes == sizeof(Tab<3>)) e = hipMemcpyToSymbol(HIP_SYMBOL(c_tab3), host_tab, bytes);
    if (N == 4 && bytes == sizeof(Tab<4>)) e = hipMemcpyToSymbol(HIP_SYMBOL(c_tab4), host_tab, bytes);
    return e == hipSuccess ? 0 : -1;
}

// this file's arithmetic
struct Rc : Rcp2 {
    template <int N>
    static __device__ __forceinline__ const Tab<N>& tab()
    {
        return T<N>();
    }
};

// launch geometry per degree: one-wave blocks of 4 elements at N = 3 (the
// phase barriers stay inside a wave and a late block holds less work),
// two-wave blocks of 5 elements at N = 4 (125 of 128 lanes busy; a block
// needs 19.6 KB of LDS, so eight blocks, sixteen waves, fill a compute unit
// to the four waves per SIMD that the conforming variant's registers allow).
// Three-wave blocks of 7 elements (175 of 192 lanes, 40 KB of LDS with all
// pairs stored at once, four blocks per CU) took 410.9 against 385.4 us per
// launch on the 246,736-leaf workload.
template <int N>
struct Geo {
    static constexpr int n = N + 1, NN = n * n;
    static constexpr int BS = N == 3 ? 64 : 128;   // block size
    static constexpr int EPB = BS / NN;            // 4 for N = 3, 5 for N = 4
    static_assert(EPB == stage_block_elems(N), "host element order assumes this block size");
    static constexpr int NT = EPB * NN;            // active threads
    static constexpr int NFN = 4 * n;              // face nodes per element
    static constexpr int NPL = n * (n - 1) / 2;    // node pairs per line
    static constexpr int NP = 2 * n * NPL;         // node pairs per element
    static constexpr int NF = 2 * N * n;           // interior subcell faces per element
    // LDS variable stride of the primitive array: unpadded.  At N = 3 padding
    // to an odd element stride cost blocks per compute unit, more than the
    // bank conflicts it saved; at N = 4 a pad of one made no difference
    // (288.7 against 289.8 us per stage on the 246,736-leaf workload).
    static constexpr int PR = NN;  // sR variable stride
    // x and y pairs in two passes where the x pairs fill whole thread rounds
    // (N = 4); the pair buffer then needs the larger of the mortar staging
    // (12 n) and half the pairs with the x lines' telescoped fluxes.  The
    // low-order subcell fluxes go to the primitive rows once those are read,
    // so the pair buffer no longer holds them.
    static constexpr bool SPLIT = (n * NPL) % NN == 0;
    static constexpr int XH = n * NPL;  // SPLIT: the x lines' telescoped fluxes follow the pair slots
    // (one pad slot at N = 4: an odd stride keeps the elements sharing a wave
    // out of step with the 256-byte bank period)
    static constexpr int PP = SPLIT ? (XH + n * N > 12 * n ? XH + n * N : 12 * n) + 1 : NP;  // sPair variable stride
    // free pair slots after the telescoping (the slots N..NPL-1 of every line
    // whose first N slots hold its telescoped fluxes) carry the surface terms
    // of the face nodes: face f, position k in line f L + k / FR, slot N + k % FR
    static constexpr int FR = NPL - N;
    static constexpr int FL = (n + FR - 1) / FR;
    static_assert(FR >= 1 && FL <= 2 && 4 * FL <= (SPLIT ? n : 2 * n), "surface-term slots");
    static __device__ __forceinline__ int fslot(int f, int k)
    {
        if constexpr (FL == 1) return f * NPL + N + k;
        else return (f * 2 + (k >= FR ? 1 : 0)) * NPL + N + (k >= FR ? k - FR : k);
    }
};

// (l, k) of the node pairs l < k of a line, 6 bits per pair in line order
template <int N>
constexpr unsigned long long pair_code()
{
    unsigned long long c = 0;
    int i = 0;
    for (int l = 0; l <= N; ++l)
        for (int k = l + 1; k <= N; ++k) {
            c |= (unsigned long long)(l | (k << 3)) << (6 * i);
            ++i;
        }
    return c;
}

// The node pairs of an element, N per thread: thread q evaluates the pairs
// q + i NN (i < N) of the list "x lines, then y lines; in each line the pairs
// (l, k), l < k, in order" (N NN pairs in all, 2 n n(n-1)/2).  Entry
// ql | qk << 5 | d << 10 | l << 11 | k << 14: the two nodes (element-local
// indices), the direction and their positions along the line.
template <int N>
struct PairMap {
    static constexpr int n = N + 1, NN = n * n, NPL = n * (n - 1) / 2;
    unsigned int code[NN][N];
    constexpr PairMap() : code()
    {
        for (int q = 0; q < NN; ++q)
            for (int i = 0; i < N; ++i) {
                const int p = q + i * NN;
                const int d = p / (n * NPL), rem = p % (n * NPL), line = rem / NPL;
                int l = 0, r = rem % NPL;
                while (r >= n - 1 - l) {
                    r -= n - 1 - l;
                    ++l;
                }
                const int k = l + 1 + r;
                const int ql = d == 0 ? line * n + l : l * n + line;
                const int qk = d == 0 ? line * n + k : k * n + line;
                code[q][i] = (unsigned)(ql | qk << 5 | d << 10 | l << 11 | k << 14);
            }
    }
};
__constant__ PairMap<3> c_pm3 = PairMap<3>();
__constant__ PairMap<4> c_pm4 = PairMap<4>();
template <int N>
__device__ __forceinline__ unsigned pair_entry(int q, int i);
template <>
__device__ __forceinline__ unsigned pair_entry<3>(int q, int i) { return c_pm3.code[q][i]; }
template <>
__device__ __forceinline__ unsigned pair_entry<4>(int q, int i) { return c_pm4.code[q][i]; }

// ---------------------------------------------------------------------------
// arithmetic helpers
// ---------------------------------------------------------------------------
// logarithmic mean x^ln = (x - y) / (ln x - ln y) from the logarithms lx, ly.
// Where |f| = |x - y| / (x + y) < 1e-2 (f^2 < 1e-4) the series
// x^ln = (x + y)/2 f / atanh f = (x + y)/2 (1 - f^2/3 - 4 f^4/45 - 44 f^6/945 - ...)
// (from the series of 2 atanh, as in Ismail & Roe 2009), whose next term is
// below 4e-18 relative there.  Branch free: one reciprocal serves whichever
// form applies.
__device__ __forceinline__ double lnmean(double x, double y, double lx, double ly)
{
    const double s = x + y, d = x - y;
    const bool ser = fabs(d) < 1e-2 * s;
    const double r = Rc::rcp(ser ? s : lx - ly);
    const double f = d * r, f2 = f * f;
    // 1/3 + f2 (4/45 + f2 44/945) = 44/945 (945/132 + f2 (21/11 + f2)): one
    // literal per instruction
    const double t = fma(f2, f2 + 21.0 / 11.0, 945.0 / 132.0) * f2;
    const double sv = 0.5 * s * fma(-44.0 / 945.0, t, 1.0);
    return ser ? sv : f;
}

// 1 / x^ln = (ln x - ln y) / (x - y); series (2 + f^2 (2/3 + f^2 (2/5 + f^2 2/7))) / (x + y)
__device__ __forceinline__ double inv_lnmean(double x, double y, double lx, double ly)
{
    const double s = x + y, d = x - y;
    const bool ser = fabs(d) < 1e-2 * s;
    const double r = Rc::rcp(ser ? s : d);
    const double f = d * r, f2 = f * f;
    // 2/3 + f2 (2/5 + f2 2/7) = 2/7 (7/3 + f2 (7/5 + f2))
    const double t = fma(f2, f2 + 7.0 / 5.0, 7.0 / 3.0) * f2;
    const double sv = fma(2.0 / 7.0, t, 2.0) * r;
    return ser ? sv : (lx - ly) * r;
}

// Natural logarithm for x > 0 normal (NaN for x <= 0 or NaN): x = m 2^k with
// m in [sqrt(1/2), sqrt(2)), f = m - 1 (exact), s = f / (2 + f), so that
// ln m = 2 atanh s = 2 s + T, T = 2 s^3/3 + 2 s^5/5 + ... (|s| < 0.172, the
// series to s^21 leaves less than 2^-56 of ln m), and 2 s = f - s f gives
// ln m = f - s (f - T / s) with T / s a polynomial in s^2; ln x = k ln 2 +
// ln m with ln 2 split into a head whose product with k is exact and a tail.
// About 1 ulp, thirty instructions (the run-time library's logarithm takes
// about eighty).
__device__ __forceinline__ double flog(double x)
{
    double m = __builtin_amdgcn_frexp_mant(x);  // [0.5, 1)
    int k = __builtin_amdgcn_frexp_exp(x);
    if (m < 0x1.6a09e667f3bcdp-1) {
        m *= 2.0;
        k -= 1;
    }
    const double f = m - 1.0;
    const double sf = f * Rc::rcp(2.0 + f);
    const double z = sf * sf;
    const double t = z * (2.0 / 3.0 + z * (2.0 / 5.0 + z * (2.0 / 7.0 + z * (2.0 / 9.0 + z * (2.0 / 11.0 +
                     z * (2.0 / 13.0 + z * (2.0 / 15.0 + z * (2.0 / 17.0 + z * (2.0 / 19.0 + z * (2.0 / 21.0))))))))));
    const double lm = f - sf * (f - t);
    const double kd = (double)k;
    const double r = fma(kd, 0x1.62e42fefp-1, fma(kd, 0x1.473de6af278edp-34, lm));
    return x > 0.0 ? r : __builtin_nan("");
}

// upper bounds are aimed at from below by the same margins
constexpr double kMarginHi = 1.0 - 0x1p-40;
constexpr double kMarginMortarHi = 1.0 - 0x1p-41;
// density increments (per node and step) this small relative to the density are
// not limited against the local density bounds
constexpr double kLocalNegl = 1e-14;

// ---------------------------------------------------------------------------
// local bounds (eq. Bounds_Barstates)
// ---------------------------------------------------------------------------
// Density and log specific entropy ln(p rho^-gamma) of the bar state of the
// low-order graph edge between this element's node `own` and the node `o`
// across a face of direction d (own_low: `own` on the low side).  The bar state
// (u_i + u_j)/2 - c_ij . (f_j - f_i) / (2 d_ij) with d_ij = |c_ij| lambda_ij is
// (u_L + u_R)/2 - (f(u_R) - f(u_L)) / (2 lambda), lambda as in llf_face.  A bar
// state outside the admissible set (only by rounding) gives -inf: no entropy
// bound from it.
__device__ __forceinline__ void bar_bounds(int d, bool own_low, const NodeP& own, const NodeP& o,
                                           double g, double& rb, double& lsb)
{
    const bool dx = d == 0;
    const double va = dx ? own.v1 : own.v2, vb = dx ? o.v1 : o.v2;
    const double lam = fmax(fabs(va) + own.c, fabs(vb) + o.c);
    const double k = (own_low ? 0.5 : -0.5) * Rc::rcp(lam);
    double fa[4], fb[4];
    fa[0] = own.r * va;
    fa[1] = own.u[1] * va + (dx ? own.p : 0.0);
    fa[2] = own.u[2] * va + (dx ? 0.0 : own.p);
    fa[3] = (own.u[3] + own.p) * va;
    fb[0] = o.r * vb;
    fb[1] = o.u[1] * vb + (dx ? o.p : 0.0);
    fb[2] = o.u[2] * vb + (dx ? 0.0 : o.p);
    fb[3] = (o.u[3] + o.p) * vb;
    double ub[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) ub[v] = 0.5 * (own.u[v] + o.u[v]) - k * (fb[v] - fa[v]);
    rb = ub[0];
    const double pb = (g - 1.0) * (ub[3] - 0.5 * (ub[1] * ub[1] + ub[2] * ub[2]) / ub[0]);
    lsb = (rb > 0.0 && pb > 0.0) ? log(pb) - g * log(rb) : -__builtin_inf();
}

// psi(theta) = p(u0 + theta dc) - exp(lst + gamma ln rho(theta)) and its
// derivative: psi >= 0 with rho > 0 is p rho^-gamma >= exp(lst).  p is concave
// in the conserved variables and rho^gamma convex, so psi is concave on the ray.
__device__ __forceinline__ double psi_s(const double* u0, const double* dc, double th, double lst,
                                        double g, double& dpsi)
{
    const double q0 = u0[0] + th * dc[0], q1 = u0[1] + th * dc[1];
    const double q2 = u0[2] + th * dc[2], q3 = u0[3] + th * dc[3];
    if (!(q0 > 0.0)) {
        dpsi = 0.0;
        return -__builtin_inf();
    }
    const double ir = 1.0 / q0;
    const double v1 = q1 * ir, v2 = q2 * ir;
    const double p = (g - 1.0) * (q3 - 0.5 * (q1 * v1 + q2 * v2));
    const double rg = exp(lst + g * log(q0));
    const double dp = (g - 1.0) * (dc[3] - v1 * dc[1] - v2 * dc[2] + 0.5 * (v1 * v1 + v2 * v2) * dc[0]);
    dpsi = dp - g * rg * ir * dc[0];
    return p - rg;
}

// Largest theta in [0, thi] with p rho^-gamma >= exp(lst) at u0 + theta dc, on
// a ray where rho stays positive up to thi.  The admissible set of the concave
// psi is an interval [0, theta*] when psi(0) >= 0.  The root is bracketed from
// both sides: the chord through the feasible and the infeasible end cuts the
// axis at or below theta* (concavity), the Newton step from the infeasible end
// at or above it (the tangent lies above psi); the two-sided iteration of
// convex limiting (Guermond, Nazarov, Popov and Tomas, SIAM J. Sci. Comput.
// 2018).  When the two estimates are within 1e-14 (or cross by rounding) it
// returns the chord point, theta* up to rounding; otherwise it stops when the
// bracket is that narrow, at most 16 rounds, and returns the feasible end;
// psi(0) <= 0 returns 0.
__device__ double theta_s(const double* u0, const double* dc, double lst, double g, double thi)
{
    if (!(thi > 0.0)) return 0.0;
    double dh, dl, dx;
    double ph = psi_s(u0, dc, thi, lst, g, dh);
    if (ph >= 0.0) return thi;
    double pl = psi_s(u0, dc, 0.0, lst, g, dl);
    if (!(pl > 0.0)) return 0.0;
    double lo = 0.0, hi = thi;
#pragma unroll 1
    for (int it = 0; it < 16; ++it) {
        double c = lo + pl * (hi - lo) / (pl - ph);
        double nw = dh < 0.0 ? hi - ph / dh : hi;
        if (!(c > lo)) c = lo;
        if (!(c < hi)) c = hi;
        if (!(nw < hi)) nw = hi;
        if (nw < c) nw = c;
        const double pc = psi_s(u0, dc, c, lst, g, dx);
        if (pc >= 0.0) {
            lo = c;
            pl = pc;
        } else {
            hi = c;
            ph = pc;
            dh = dx;
        }
        // the estimates meet: c is theta* up to rounding
        if (nw - c <= 1e-14) return c;
        const double pn = psi_s(u0, dc, nw, lst, g, dx);
        if (pn >= 0.0) {
            if (nw > lo) {
                lo = nw;
                pl = pn;
            }
        } else if (nw < hi) {
            hi = nw;
            ph = pn;
            dh = dx;
        }
        if (hi - lo <= 1e-14) break;
    }
    return lo;
}

// Node factor of the volume limiter from the node's four face increments cf
// (dt/m_i-scaled, zero for missing faces): Zalesak factors for the density
// floor rfl (and, with local bounds, the ceiling rce), the pressure root per
// face and, with local bounds, the entropy root per face on [0, theta] (log
// entropy floor lsm); the last two on Gamma = 4-scaled increments.
template <bool LOCB>
__device__ __forceinline__ double volume_factor(const double* uFV, const double (&cf)[4][4], double rfl,
                                                double pfl, double rce, double lsm, double lsi, double g,
                                                double ig1)
{
    const double rt = rfl * kMargin, pt = pfl * kMargin;
    // Zalesak: the sum of the negative (positive) density increments may use at
    // most the distance to the floor (ceiling)
    double P = 0.0, Pp = 0.0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        P += fmin(cf[j][0], 0.0);
        if (LOCB) Pp += fmax(cf[j][0], 0.0);
    }
    // local bounds: increments below kLocalNegl of the density are rounding
    // noise and are not limited (a node whose density interval has zero width
    // would otherwise switch between theta = 0 and 1 on the sign of a rounding
    // error)
    if (LOCB && P > -kLocalNegl * uFV[0]) P = 0.0;
    if (LOCB && Pp < kLocalNegl * uFV[0]) Pp = 0.0;
    double th = 1.0;
    if (P < 0.0) th = fmax(fmin((rt - uFV[0]) * Rc::rcp(P), 1.0), 0.0);
    if (LOCB && Pp > 0.0) th = fmin(th, fmax((rce * kMarginHi - uFV[0]) / Pp, 0.0));
    // pressure: each face's increment scaled by Gamma = 2d = 4 (a zero
    // increment, as on a missing face, admits theta = 1 at an admissible uFV)
#pragma unroll
    for (int j = 0; j < 4; ++j) th = fmin(th, theta_p<4>(uFV, cf[j], pt, ig1));
    // specific entropy: per face on [0, th].  The target ln(s_min (1 + 2^-40))
    // is capped at lsi lowered by 2^-41: with bounds from the low-order solution
    // lsi is the node's own low-order log entropy (where the node itself is the
    // minimum of its neighbourhood, the raised bound would lie above the state
    // the limiter starts from); with bar states lsi = +inf (no cap)
    if (LOCB) {
        const double lst = fmin(lsm + 0x1p-40, lsi - 0x1p-41);
#pragma unroll 1
        for (int j = 0; j < 4; ++j) {
            const double dc[4] = {4.0 * cf[j][0], 4.0 * cf[j][1], 4.0 * cf[j][2], 4.0 * cf[j][3]};
            if (dc[0] == 0.0 && dc[1] == 0.0 && dc[2] == 0.0 && dc[3] == 0.0) continue;
            th = theta_s(uFV, dc, lst, g, th);
        }
    }
    return th;
}

// Factor of one mortar node for its n_i-scaled increment dc on top of u^vol:
// density floor (and ceiling), pressure root, entropy root, all against half
// the volume margin.
template <bool LOCB>
__device__ __forceinline__ double mortar_factor(const double* uvol, const double* dc, double rfl, double pfl,
                                                double rce, double lsm, double lsi, double g, double ig1)
{
    const double rt = rfl * kMarginMortar, pt = pfl * kMarginMortar;
    double ts = 1.0;
    const bool negl = LOCB && fabs(dc[0]) <= kLocalNegl * uvol[0];
    if (dc[0] < 0.0 && !negl) ts = fmin(ts, fmax((rt - uvol[0]) / dc[0], 0.0));
    if (LOCB && dc[0] > 0.0 && !negl) ts = fmin(ts, fmax((rce * kMarginMortarHi - uvol[0]) / dc[0], 0.0));
    ts = fmin(ts, theta_p(uvol, dc, pt, ig1));
    if (LOCB) ts = theta_s(uvol, dc, fmin(lsm + 0x1p-41, lsi - 0x1p-40), g, ts);
    return ts;
}

// ---------------------------------------------------------------------------
// element kernel
// ---------------------------------------------------------------------------
// Local bounds from the low-order solution (eq. Bounds_LowOrder): per node the density
// range over u^FV = u + dt R_LO / m of the node and its low-order neighbours (subcell
// neighbours; the matching node across a conforming face; the nodes with a nonzero
// sparse weight across a mortar; none across a boundary), and the smallest
// ln(p rho^-gamma) among those with rho, p > 0.
// MODE_LOWSOL: each node's low-order density and log entropy (+inf where rho or p <= 0),
// without the pair fluxes; the stage gathers them through LDS and its face lanes.  On the
// 22,156-leaf blast the bounds took a residual with pair fluxes (15.9 us of a stage), a
// pass over it (6.4) and a gather (11.7); five steps 1,494 us, without the pair fluxes and
// the pass 1,366, without the gather's kernel 1,245; results are the same bits.
enum { MODE_STAGE = 0, MODE_LOWSOL = 1 };

struct StageArgs {
    const double* uin;
    const double* un;
    double* uout;
    double a, b;
    const double* dt;
    const double* ind;  // combined limiting: shock indicator per element, in [0, 1]
    const double* lsv;  // bounds from the low-order solution: [E][2][NN] its density and log entropy
    // when set, dt = cfl / max over the accumulator set dtmax (bits of
    // non-negative doubles); block 0 stores it in dt_out
    const unsigned long long* dtmax;
    double cfl;
    double* dt_out;
    const int* fnbr;
    const int* fnbr2;
    const int* fmort;
    const int* mort;  // (not read; see dgidp_kernels.hip)
    const double* h;
    double* slot;
    const int8_t* bkind;  // boundary nodes: condition and exterior state
    const double* bext;
    int E;
    double gamma, beta;
    double ig1;  // 1 / (gamma - 1)
    int rev;     // walk the XCD batch ranges from their ends (conforming variant only)
    int limiter;
    int vflux;  // two-point volume flux: DGIDP_FLUX_RANOCHA or DGIDP_FLUX_CHANDRASHEKAR
    DevStats* st;
};

// node qq of the block's element le from its LDS primitives; the conserved
// state is formed again from them (rho v = rho * v, E = p / (gamma - 1) +
// (rho v . v) / 2: within a few ulp of the stored state, the same for every
// reader of a node, so that equal states still meet in a zero flux difference)
#define LDS_NODE(X, qq)                                                    \
    do {                                                                   \
        X.r = sR[le][0][qq];                                               \
        X.v1 = sR[le][1][qq];                                              \
        X.v2 = sR[le][2][qq];                                              \
        X.p = sR[le][3][qq];                                               \
        X.c = sR[le][4][qq];                                               \
        X.u[0] = X.r;                                                      \
        X.u[1] = X.r * X.v1;                                               \
        X.u[2] = X.r * X.v2;                                               \
        X.u[3] = fma(X.p, ig1, 0.5 * (X.u[1] * X.v1 + X.u[2] * X.v2));     \
    } while (0)

// LIMK: 0 positivity (or none, at run time), 1 local bounds from bar states,
// 2 the blend of positivity and bar-state local factors by the per-element
// shock indicator A.ind (eq. combination_posLim_local), 3 local bounds from the
// low-order solution (eq. Bounds_LowOrder), read from A.lsv
// MORT: the launch over the element batches that hold a mortar element (the
// surface phase with Kopriva's mortar and the sparse low-order mortar flux,
// mortar slot records); the batches without one run the MORT = false variant,
// which has no mortar code, fewer registers and four waves per SIMD.
template <int N, int MODE, bool MIXED, int LIMK, bool MORT>
// at least three waves per SIMD: the local-limiting variant would otherwise
// take 172 registers and run two (63.3 against 67.7 us on the 22,156-leaf
// blast with a few spilled registers; the other variants fit anyway); the
// conforming positivity variant fits 128 registers, four waves
__global__ __launch_bounds__(Geo<N>::BS) __attribute__((amdgpu_waves_per_eu((!MORT && LIMK == 0) ? 4 : 3)))
void k_stage(StageArgs A)
{
    using G = Geo<N>;
    // LOC: local bounds enforced; COMB: blended with positivity; BAR: the bounds
    // come from bar states (computed here), otherwise from the low-order
    // solution (read from A.lsv); PURE: local factors only
    constexpr bool LOC = LIMK >= 1, COMB = LIMK == 2, BAR = LIMK == 1 || LIMK == 2;
    constexpr bool PURE = LIMK == 1 || LIMK == 3;
    constexpr bool PAIRS = MODE == MODE_STAGE;
    constexpr int n = G::n, NN = G::NN, EPB = G::EPB, NT = G::NT, NFN = G::NFN;
    constexpr int NPL = G::NPL, NP = G::NP, NF = G::NF, PPT = NP / NN, PP = G::PP;
    static_assert(NP % NN == 0, "pair split");
    constexpr bool DSTAT = (n * NPL) % NN == 0, SPLIT = G::SPLIT;
    constexpr int XH = n * NPL;  // SPLIT: the x lines' telescoped fluxes follow the pair slots
    static_assert(!SPLIT || (DSTAT && XH + n * N <= G::PP), "two-pass pair buffer");
    static_assert(G::PP >= 12 * n, "mortar buffers reuse the pair buffer");
    static_assert(G::PR == NN && 4 * NF + NN <= 8 * NN, "subcell fluxes and node factors reuse sR");
    constexpr int MB = 4 * n;  // offset of the mortar-node fluxes in the pair buffer

    // variable-major (see Geo)
    __shared__ double sR[EPB][8][G::PR];     // rho, v1, v2, p, c, ln rho, z = rho/p, ln z
    __shared__ double sPair[EPB][4][G::PP];  // pair fluxes, then telescoped fluxes and surface terms
    // bar states of local limiting: rows 0-3 the subcell faces owned by a node
    // (x: density, log entropy; y: the same), rows 4-6 the face lanes' range
    // across the element face; row 0 later the local node factors of the blend
    // (from the low-order solution: rows 0 and 1 its density and log entropy per node)
    __shared__ double sB[LOC ? EPB : 1][7][LOC ? NN : 1];
    __shared__ double sTw[2][n];              // LGL weights and their reciprocals, read per lane
    __shared__ double sS[n][n];               // Sbar, read per pair
    // After phase 5b the primitive rows of sR are read no more: they take the
    // low-order subcell fluxes, variable-major over the NF faces (x faces
    // b N + a, y faces N n + a N + b), and after them the node factors.
#define sFV(v, fi) sRe[(v) * NF + (fi)]
#define sTh(qq) sRe[4 * NF + (qq)]

    const Tab<N>& tb = T<N>();
    const double g = A.gamma, ig1 = A.ig1;
    const int tid = threadIdx.x;
    const int le = tid / NN, q = tid - le * NN, a = q % n, b = q / n;
    const int xb = !MORT && A.rev ? xcd_batch_rev(blockIdx.x, gridDim.x) : xcd_batch(blockIdx.x, gridDim.x);
    const int e = xb * EPB + le;
    double* const sRe = &sR[0][0][0] + le * 8 * NN;  // element le's rows, flat
    double* const sPe = &sPair[0][0][0] + le * 4 * PP;  // element le's pair buffer, flat
    const bool act = tid < NT && e < A.E;
    if (tid < n) {
        sTw[0][tid] = tb.w[tid];
        sTw[1][tid] = tb.winv[tid];
    }
    if (tid < NN) (&sS[0][0])[tid] = (&tb.S[0][0])[tid];

    // ---- phase 1: own node into LDS; face-node role and its remote loads ----
    double hx = 1.0, hy = 1.0;
    int fcode[4] = {-1, -1, -1, -1};
    const bool fnode = act && q < NFN;       // this lane also evaluates one face node
    const int ff = q / n, fk = q - (q / n) * n;  // its face and position
    const int qfo = face_q<N>(ff, fk), qfn = face_q<N>(ff ^ 1, fk);  // the face node, its neighbour's
    int fcode_f = -1, fnb = 0, fnb2 = -1, bk = 0;
    double onb[4];  // conforming neighbour state (boundary: exterior state) across face ff at fk
    double us1[4];  // large side: the second small element's trace at position fk
    // u^n of this node for the SSP combination, loaded where it is needed (so
    // that it occupies no registers through the flux phases), and this node's
    // state (uin)
    double un4[4] = {0, 0, 0, 0};
    double u0[4] = {0, 0, 0, 0};
    // the low-order surface term of this lane's face node, kept in registers
    // until phase 5 frees pair slots, which then carry it to the node's own thread
    double fterm[4] = {0, 0, 0, 0};
    // local bounds: own log entropy; for face lanes the density range and the
    // smallest log entropy of the bar states across this lane's face node
    double ls_own = 0.0;
    double w_e = 0.0;  // combined limiting: weight of the local factors
    bool need_loc = false;  // this element computes bounds and local factors (uniform per element)
    double fb_lo = __builtin_inf(), fb_hi = -__builtin_inf(), fb_ls = __builtin_inf();
    const double dtpart =
        A.dtmax ? __longlong_as_double((long long)A.dtmax[(tid & 63) * kDtStride]) : 0.0;
    // this thread's node pairs (the pair map), loaded with the state
    unsigned pcode[PPT];
#pragma unroll
    for (int i = 0; i < PPT; ++i) pcode[i] = act ? pair_entry<N>(q, i) : 0u;
    if (act) {
        // issue the independent global loads first
#pragma unroll
        for (int f = 0; f < 4; ++f) fcode[f] = A.fmort[e * 4 + f];
        if (fnode) {
            fnb = A.fnbr[e * 4 + ff];
            fnb2 = A.fnbr2[e * 4 + ff];
        }
        NodeP me;
        load_node<N, Rc>(A.uin, e, q, me, g);
        hx = A.h[2 * e];
        hy = A.h[2 * e + 1];
        if (COMB) w_e = A.ind[e];
#pragma unroll
        for (int v = 0; v < 4; ++v) u0[v] = me.u[v];
        // the logarithms feed only the two-point volume fluxes: FP32 in the
        // mixed mode, where rows 5-7 hold the FP32 operands of those fluxes in
        // pairs (rho, p), (ln rho, z), (ln z, 0)
        const double z = me.r * Rc::rcp(me.p);
        sR[le][0][q] = me.r;
        sR[le][1][q] = me.v1;
        sR[le][2][q] = me.v2;
        sR[le][3][q] = me.p;
        sR[le][4][q] = me.c;
        double lr, lz;
        if (MIXED) {
            const float lrf = __logf((float)me.r), lzf = __logf((float)z);
            lr = lrf;
            lz = lzf;
            sR[le][5][q] = pack2((float)me.r, (float)me.p);
            sR[le][6][q] = pack2(lrf, (float)z);
            sR[le][7][q] = pack2(lzf, 0.0f);
        } else {
            lr = PAIRS ? flog(me.r) : 0.0;
            lz = PAIRS ? flog(z) : 0.0;
            sR[le][5][q] = lr;
            sR[le][6][q] = z;
            sR[le][7][q] = lz;
        }
        // the blend needs local factors only where the indicator fires, and at
        // mortar nodes (their mortar may blend with another element's weight)
        need_loc = LOC && (!COMB || w_e > 0.0 || fcode[0] >= 0 || fcode[1] >= 0 || fcode[2] >= 0 ||
                           fcode[3] >= 0);
        // ln(p rho^-gamma) of the node itself, the bar state (i, i)
        if (need_loc) ls_own = MIXED ? log(me.p) - g * log(me.r) : (1.0 - g) * lr - lz;
        if (fnode) {
            fcode_f = fcode[ff];
            if (fcode_f == -1) {
                load_u<N>(A.uin, fnb, qfn, onb);
            } else if (fcode_f < -1) {
                const int j = (-2 - fcode_f) * n + fk;
                bk = A.bkind[j];
#pragma unroll
                for (int v = 0; v < 4; ++v) onb[v] = A.bext[(size_t)j * 4 + v];
            } else if (MORT && !fm_small(fcode_f)) {
                // large side: both small traces at position fk, kept in
                // registers for the mortar-node fluxes and staged for the
                // sparse low-order pairs of the other positions
                load_u<N>(A.uin, fnb, qfn, onb);
                load_u<N>(A.uin, fnb2, qfn, us1);
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    sPair[le][v][MB + (ff * 2 + 0) * n + fk] = onb[v];
                    sPair[le][v][MB + (ff * 2 + 1) * n + fk] = us1[v];
                }
            } else if (MORT) {
                // small side: stage the large face trace for the interpolation
                double w[4];
                load_u<N>(A.uin, fnb, qfn, w);
#pragma unroll
                for (int v = 0; v < 4; ++v) sPair[le][v][ff * n + fk] = w[v];
            }
        }
        if (LIMK == 3) {
            // the low-order solution at the node and across this lane's face node (the
            // matching node of a conforming face, the nodes with a nonzero sparse
            // weight across a mortar, none across a boundary)
            const double* own = A.lsv + ((unsigned)e * 2u * NN + (unsigned)q);
            sB[le][0][q] = own[0];
            sB[le][1][q] = own[NN];
            auto gather = [&](int el, int node) {
                const double* o = A.lsv + ((unsigned)el * 2u * NN + (unsigned)node);
                fb_lo = fmin(fb_lo, o[0]);
                fb_hi = fmax(fb_hi, o[0]);
                fb_ls = fmin(fb_ls, o[NN]);
            };
            if (fnode) {
                if (fcode_f == -1) {
                    gather(fnb, qfn);
                } else if (MORT && fcode_f >= 0) {
                    const bool small = fm_small(fcode_f);
                    const int hh = fm_half(fcode_f);
                    const int nz = small ? tb.snc[hh][fk] : tb.lnc[fk];
#pragma unroll 1
                    for (int i = 0; i < nz; ++i) {
                        const int col = small ? tb.snz[hh][fk][i] : tb.lnz[fk][i];  // large side: h n + l
                        gather(small || col < n ? fnb : fnb2, face_q<N>(ff ^ 1, col < n ? col : col - n));
                    }
                }
                sB[le][4][q] = fb_lo;
                sB[le][5][q] = fb_hi;
                sB[le][6][q] = fb_ls;
            }
        }
    }
    __syncthreads();
    double dt;
    if (A.dtmax) {
        const double m = wave_max(dtpart);
        dt = A.cfl / m;
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            *A.dt_out = dt;
            if (A.st) A.st->dt = dt;
        }
    } else {
        dt = A.dt ? *A.dt : 0.0;
    }

    // ---- phase 2: one surface flux per face node ----
    const int dff = ff >> 1;
    const bool lowf = ff & 1;                    // element on the low side of face ff
    const double sgf = lowf ? -1.0 : 1.0;
    const double hff = ff < 2 ? hy : hx;
    if (fnode) {
        NodeP own;  // the face node's state
        LDS_NODE(own, qfo);
        if (fcode_f < 0) {
            NodeP o;
            if (fcode_f == -1) {
#pragma unroll
                for (int v = 0; v < 4; ++v) o.u[v] = onb[v];
            } else {
                boundary_ghost(bk, onb, own, ff, g, o.u);
            }
            make_node<Rc>(o, g);
            double F[4];
            llf_face(dff, lowf, own, o, F);
            if (BAR && need_loc) {
                bar_bounds(dff, lowf, own, o, g, fb_lo, fb_ls);
                fb_hi = fb_lo;
            }
            const double W = sgf * sTw[0][fk] * hff * 0.5;
#pragma unroll
            for (int v = 0; v < 4; ++v) fterm[v] = W * F[v];
        } else if (MORT && !fm_small(fcode_f)) {
            // large side: mortar-node fluxes at position fk of both halves
            // (kept in registers until every lane has read the staged small
            // traces), and the sparse low-order pairs of this node
            for (int hh = 0; hh < 2; ++hh) {
                NodeP ui, us;
#pragma unroll
                for (int v = 0; v < 4; ++v) us.u[v] = hh == 0 ? onb[v] : us1[v];
                make_node<Rc>(us, g);
                // the large face interpolated to half hh, from the face nodes'
                // conserved states formed as LDS_NODE does
                double ia[4] = {0, 0, 0, 0};
#pragma unroll
                for (int j = 0; j < n; ++j) {
                    const int qj = face_q<N>(ff, j);
                    const double r = sR[le][0][qj], v1 = sR[le][1][qj], v2 = sR[le][2][qj];
                    const double m1 = r * v1, m2 = r * v2;
                    const double uj[4] = {r, m1, m2, fma(sR[le][3][qj], ig1, 0.5 * (m1 * v1 + m2 * v2))};
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        if (MIXED) ia[v] = (float)ia[v] + tb.If[hh][fk][j] * (float)uj[v];
                        else ia[v] += tb.I[hh][fk][j] * uj[v];
                    }
                }
#pragma unroll
                for (int v = 0; v < 4; ++v) ui.u[v] = ia[v];
                make_node<Rc>(ui, g);
                double F[4];
                mortar_flux(dff, lowf, ui, us, F);
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    if (hh == 0) onb[v] = F[v];
                    else us1[v] = F[v];
                }
            }
            // (over this node's nonzero weights only: a wave runs as many
            // rounds as its busiest lane)
            double lo[4] = {0, 0, 0, 0};
            const int nz = tb.lnc[fk];
#pragma unroll 1
            for (int i = 0; i < nz; ++i) {
                const int col = tb.lnz[fk][i];  // h n + l
                const double wt = tb.Wt[fk][col];
                NodeP us;
#pragma unroll
                for (int v = 0; v < 4; ++v) us.u[v] = sPair[le][v][MB + ff * 2 * n + col];
                make_node<Rc>(us, g);
                double Gf[4];
                llf_face(dff, lowf, own, us, Gf);
                if (BAR && need_loc) {
                    double rb, lb;
                    bar_bounds(dff, lowf, own, us, g, rb, lb);
                    fb_lo = fmin(fb_lo, rb);
                    fb_hi = fmax(fb_hi, rb);
                    fb_ls = fmin(fb_ls, lb);
                }
                const double W = sgf * wt * hff * 0.5;
#pragma unroll
                for (int v = 0; v < 4; ++v) lo[v] += W * Gf[v];
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) fterm[v] = lo[v];
        } else if (MORT) {
            // small side: interpolate the large face, LLF on the mortar = this face
            const int hh = fm_half(fcode_f);
            NodeP ui;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                if (MIXED) {
                    float acc = 0.0f;
#pragma unroll
                    for (int j = 0; j < n; ++j) acc += tb.If[hh][fk][j] * (float)sPair[le][v][ff * n + j];
                    ui.u[v] = acc;
                } else {
                    double acc = 0.0;
#pragma unroll
                    for (int j = 0; j < n; ++j) acc += tb.I[hh][fk][j] * sPair[le][v][ff * n + j];
                    ui.u[v] = acc;
                }
            }
            make_node<Rc>(ui, g);
            double F[4], ho[4], lo[4] = {0, 0, 0, 0};
            mortar_flux(dff, !lowf, ui, own, F);
#pragma unroll
            for (int v = 0; v < 4; ++v) ho[v] = sgf * sTw[0][fk] * hff * 0.5 * F[v];
            const int nz = tb.snc[hh][fk];
#pragma unroll 1
            for (int i = 0; i < nz; ++i) {
                const int j = tb.snz[hh][fk][i];
                const double wt = tb.Wt[j][hh * n + fk];
                NodeP uj;
#pragma unroll
                for (int v = 0; v < 4; ++v) uj.u[v] = sPair[le][v][ff * n + j];
                make_node<Rc>(uj, g);
                double Gf[4];
                llf_face(dff, lowf, own, uj, Gf);
                if (BAR && need_loc) {
                    double rb, lb;
                    bar_bounds(dff, lowf, own, uj, g, rb, lb);
                    fb_lo = fmin(fb_lo, rb);
                    fb_hi = fmax(fb_hi, rb);
                    fb_ls = fmin(fb_ls, lb);
                }
                const double W = sgf * wt * hff;  // wt * h_L / 2 with h_L = 2 h
#pragma unroll
                for (int v = 0; v < 4; ++v) lo[v] += W * Gf[v];
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) fterm[v] = lo[v];
            {
                const int S = fm_mortar(fcode_f);
                double* R = A.slot + (size_t)(S * 3 * n + n + fm_half(fcode_f) * n + fk) * kSlotW;
#pragma unroll
                for (int v = 0; v < 4; ++v) R[4 + v] = ho[v] - lo[v];
            }
        }
    }
    if constexpr (MORT) {  // (every batch of the mortar launch holds a mortar element)
        __syncthreads();
        // ---- phase 3: large sides publish and project the mortar fluxes ----
        const bool large = fnode && fcode_f >= 0 && !fm_small(fcode_f);
        if (large) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                sPair[le][v][MB + (ff * 2 + 0) * n + fk] = onb[v];
                sPair[le][v][MB + (ff * 2 + 1) * n + fk] = us1[v];
            }
        }
        __syncthreads();
        if (large) {
            const int S = fm_mortar(fcode_f);
            double ho[4];
#pragma unroll 1
            for (int v = 0; v < 4; ++v) {
                double acc = 0.0;
                if (MIXED) {
                    float accf = 0.0f;
#pragma unroll
                    for (int hh = 0; hh < 2; ++hh)
#pragma unroll
                        for (int l = 0; l < n; ++l)
                            accf += tb.Pf[hh][fk][l] * (float)sPair[le][v][MB + (ff * 2 + hh) * n + l];
                    acc = accf;
                } else {
#pragma unroll
                    for (int hh = 0; hh < 2; ++hh)
#pragma unroll
                        for (int l = 0; l < n; ++l)
                            acc += tb.P[hh][fk][l] * sPair[le][v][MB + (ff * 2 + hh) * n + l];
                }
                ho[v] = sgf * sTw[0][fk] * hff * 0.5 * acc;
            }
            double* R = A.slot + (size_t)(S * 3 * n + fk) * kSlotW;
#pragma unroll
            for (int v = 0; v < 4; ++v) R[4 + v] = ho[v] - fterm[v];
        }
        __syncthreads();
    }

    // ---- phase 4: two-point volume fluxes, once per node pair of each line ----
    // Each flux is evaluated in the frame of its pair's direction d: the normal
    // velocity is read from LDS row 1 + d and the tangential one from row 2 - d,
    // and the two momentum components are stored back to rows 1 + d and 2 - d,
    // so that lanes holding x and y pairs run the same instructions.
    // pair p = q + i NN: the x pairs are slots below n NPL.  Where NN divides that
    // count (N = 4) the direction of round i is a constant, and the x and y pairs
    // are evaluated in two passes (SPLIT): the x lines are telescoped into the
    // slots after the x pairs, then the y pairs take the x pairs' slots, so the
    // pair buffer holds half the pairs at a time.
    const double hhx = 0.5 * hy, hhy = 0.5 * hx;  // pair scale of x and y lines
    auto pair_rounds = [&](auto i0c, auto i1c, int slot_off) {
        constexpr int i0 = decltype(i0c)::value, i1 = decltype(i1c)::value;
        if (!act) return;
#pragma unroll
        for (int i = i0; i < i1; ++i) {
            const unsigned c = pcode[i];
            const int ql = c & 31, qk = (c >> 5) & 31;
            // a round wholly below or above the x pairs' n NPL slots has a constant
            // direction; only a round that straddles them (N = 3: the second) decodes it
            const int d = (i + 1) * NN <= n * NPL ? 0 : (i * NN >= n * NPL ? 1 : (int)((c >> 10) & 1));
            const int p = q + i * NN - slot_off;
            const int rn = 1 + d, rt = 2 - d;
            const double scale = sS[(c >> 11) & 7][(c >> 14) & 7] * (d ? hhy : hhx);
            const double Ln = sR[le][rn][ql], Lt = sR[le][rt][ql];
            const double Rn = sR[le][rn][qk], Rt = sR[le][rt][qk];
            double f0, fn, ft, f3;
            if (!MIXED) {
                const double L0 = sR[le][0][ql], L3 = sR[le][3][ql];
                const double L5 = sR[le][5][ql], L6 = sR[le][6][ql], L7 = sR[le][7][ql];
                const double R0 = sR[le][0][qk], R3 = sR[le][3][qk];
                const double R5 = sR[le][5][qk], R6 = sR[le][6][qk], R7 = sR[le][7][qk];
                const double iz_ln = inv_lnmean(L6, R6, L7, R7);
                const double vna = 0.5 * (Ln + Rn), vta = 0.5 * (Lt + Rt);
                const double fr = lnmean(L0, R0, L5, R5) * vna;
                f0 = fr;
                if (A.vflux == DGIDP_FLUX_CHANDRASHEKAR) {
                    // Chandrashekar: beta = z / 2, so p~ = rho-bar / (2 beta-bar) =
                    // (rho_L + rho_R) / (z_L + z_R) and 1 / (2 beta^ln) = 1 / z^ln
                    const double pt = (L0 + R0) * Rc::rcp(L6 + R6);
                    fn = fr * vna + pt;
                    ft = fr * vta;
                    f3 = fr * (ig1 * iz_ln - 0.25 * (Ln * Ln + Lt * Lt + Rn * Rn + Rt * Rt)) + vna * fn + vta * ft;
                } else {
                    fn = fr * vna + 0.5 * (L3 + R3);
                    ft = fr * vta;
                    f3 = fr * (0.5 * (Ln * Rn + Lt * Rt) + ig1 * iz_ln) + 0.5 * (L3 * Rn + R3 * Ln);
                }
            } else {
                const F2 L5 = unpack2(sR[le][5][ql]), L6 = unpack2(sR[le][6][ql]);
                const F2 R5 = unpack2(sR[le][5][qk]), R6 = unpack2(sR[le][6][qk]);
                const float L7 = unpack2(sR[le][7][ql]).x, R7 = unpack2(sR[le][7][qk]).x;
                const float rL = L5.x, rR = R5.x, pL = L5.y, pR = R5.y, zL = L6.y, zR = R6.y;
                const float iz_ln = inv_lnmeanf(zL, zR, L7, R7);
                const float vnL = (float)Ln, vnR = (float)Rn, vtL = (float)Lt, vtR = (float)Rt;
                const float vna = 0.5f * (vnL + vnR), vta = 0.5f * (vtL + vtR);
                const float fr = lnmeanf(rL, rR, L6.x, R6.x) * vna;
                f0 = fr;
                if (A.vflux == DGIDP_FLUX_CHANDRASHEKAR) {
                    const float pt = (rL + rR) / (zL + zR);
                    const float fnf = fr * vna + pt, ftf = fr * vta;
                    fn = fnf;
                    ft = ftf;
                    f3 = fr * ((float)ig1 * iz_ln - 0.25f * (vnL * vnL + vtL * vtL + vnR * vnR + vtR * vtR)) +
                         vna * fnf + vta * ftf;
                } else {
                    fn = fr * vna + 0.5f * (pL + pR);
                    ft = fr * vta;
                    f3 = fr * (0.5f * (vnL * vnR + vtL * vtR) + (float)ig1 * iz_ln) + 0.5f * (pL * vnR + pR * vnL);
                }
            }
            sPair[le][0][p] = scale * f0;
            sPair[le][rn][p] = scale * fn;
            sPair[le][rt][p] = scale * ft;
            sPair[le][3][p] = scale * f3;
        }
    };
    // telescoped high-order subcell fluxes of one line and variable: the flux
    // through the subcell face after position pos is the sum of the line's pair
    // fluxes (l, k) with l <= pos < k; with the position a loop constant every
    // pair index is static.  P: the line's pair slots; the N sums go to H.
    auto telescope = [&](const double* P, double* H) {
        double hof[N];
#pragma unroll
        for (int pos = 0; pos < N; ++pos) {
            double acc = 0.0;
#pragma unroll
            for (int l = 0; l <= pos; ++l)
#pragma unroll
                for (int k = pos + 1; k < n; ++k) acc += P[l * (2 * n - l - 1) / 2 + (k - l - 1)];
            hof[pos] = acc;
        }
#pragma unroll
        for (int pos = 0; pos < N; ++pos) H[pos] = hof[pos];
    };
    if constexpr (!PAIRS) {
    } else if constexpr (SPLIT) {
        // ---- phase 4 and 5a in two passes: one task per line and variable ----
        pair_rounds(std::integral_constant<int, 0>(), std::integral_constant<int, PPT / 2>(), 0);
        __syncthreads();
        if (act && q < 4 * n) telescope(&sPair[le][q & 3][(q >> 2) * NPL], &sPair[le][q & 3][XH + (q >> 2) * N]);
        __syncthreads();
        pair_rounds(std::integral_constant<int, PPT / 2>(), std::integral_constant<int, PPT>(), n * NPL);
        __syncthreads();
        if (act && q < 4 * n) {
            double* P = &sPair[le][q & 3][(q >> 2) * NPL];
            telescope(P, P);
        }
    } else {
        pair_rounds(std::integral_constant<int, 0>(), std::integral_constant<int, PPT>(), 0);
        __syncthreads();

        // ---- phase 5a: telescoped high-order subcell fluxes ----
        // One task per line and variable (x lines first, then y lines; 8n tasks,
        // task t = q + j NN for j = 0, 1).  The N sums replace the line's first N
        // pair slots of that variable, which no other task reads.
        static_assert(8 * n <= 2 * NN, "two telescoping tasks per lane at most");
        if (act) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int t = q + j * NN;
                if (t < 8 * n) {
                    double* P = &sPair[le][t & 3][(t >> 2) * NPL];
                    telescope(P, P);
                }
            }
        }
    }
    // ---- phase 5b: low-order subcell fluxes of the faces owned by this node,
    // x (a|a+1) and y (b|b+1) ----
    double FVo[2][4];
    double brb[2] = {0.0, 0.0}, bls[2] = {0.0, 0.0};  // bar state of each owned subcell face
    if (act) {
        NodeP me;
        LDS_NODE(me, q);
#pragma unroll
        for (int d = 0; d < 2; ++d) {
            const int pos = d == 0 ? a : b;
            if (pos >= N) continue;
            const int qn = d == 0 ? q + 1 : q + n;
            NodeP o;
            LDS_NODE(o, qn);
            double F[4];
            llf_face(d, true, me, o, F);
            if (BAR && need_loc) bar_bounds(d, true, me, o, g, brb[d], bls[d]);
            const double hs = 0.5 * (d == 0 ? hy : hx);
#pragma unroll
            for (int v = 0; v < 4; ++v) FVo[d][v] = hs * F[v];
        }
    }
    // every read of the primitives (and of the pairs, by the telescoping) is done
    __syncthreads();
    if (act) {
        if (a < N) {
#pragma unroll
            for (int v = 0; v < 4; ++v) sFV(v, b * N + a) = FVo[0][v];
        }
        if (b < N) {
#pragma unroll
            for (int v = 0; v < 4; ++v) sFV(v, N * n + a * N + b) = FVo[1][v];
        }
    }
    // the face lanes' surface terms go to the free pair slots
    if (fnode) {
        const int fs = G::fslot(ff, fk);
#pragma unroll
        for (int v = 0; v < 4; ++v) sPair[le][v][fs] = fterm[v];
    }
    if (BAR && need_loc) {
        if (a < N) {
            sB[le][0][q] = brb[0];
            sB[le][1][q] = bls[0];
        }
        if (b < N) {
            sB[le][2][q] = brb[1];
            sB[le][3][q] = bls[1];
        }
        if (fnode) {
            sB[le][4][q] = fb_lo;
            sB[le][5][q] = fb_hi;
            sB[le][6][q] = fb_ls;
        }
    }
    __syncthreads();

    // ---- phase 6: low-order residual, bounds, node factors ----
    if (act && MODE == MODE_STAGE && A.a != 0.0) load_u<N>(A.un, e, q, un4);
    const bool onf[4] = {a == 0, a == N, b == 0, b == N};
    // the four subcell faces j of the node (left, right, below, above), each
    // taken at a clamped in-range position of the node's own line; a missing
    // face (on the element boundary) has weight 0.  Face index (x faces
    // b N + pos, y faces N n + a N + pos), slot of the telescoped high-order
    // flux (x faces on line b, y faces on line a) and signed weight (+w on the
    // left / lower face, -w on the right / upper one), formed where used.
    auto fpos = [&](int j) {
        return j == 0 ? (a > 0 ? a - 1 : 0) : j == 1 ? (a < N ? a : N - 1) : j == 2 ? (b > 0 ? b - 1 : 0)
                                                                             : (b < N ? b : N - 1);
    };
    auto fidx = [&](int j) { return j < 2 ? b * N + fpos(j) : N * n + a * N + fpos(j); };
    auto hslot = [&](int j) {
        if (SPLIT) return j < 2 ? XH + b * N + fpos(j) : a * NPL + fpos(j);
        return j < 2 ? b * NPL + fpos(j) : (n + a) * NPL + fpos(j);
    };
    auto fweight = [&](int j) {
        const double w = sTw[0][j < 2 ? b : a];
        const bool has = j == 0 ? a > 0 : j == 1 ? a < N : j == 2 ? b > 0 : b < N;
        return has ? ((j & 1) ? -w : w) : 0.0;
    };
    double RLO[4], dS0[4] = {0, 0, 0, 0}, dS1[4] = {0, 0, 0, 0};
    int slot0 = -1, slot1 = -1, nmf = 0;
    double im = 1.0;  // 1 / m_i
    if (act) {
        im = 4.0 * Rc::rcp(hx * hy) * sTw[1][a] * sTw[1][b];
        const double cw[4] = {fweight(0), fweight(1), fweight(2), fweight(3)};
        const int fi[4] = {fidx(0), fidx(1), fidx(2), fidx(3)};
        // the surface terms of the element faces the node lies on: at most one
        // x face (0 or 1) and one y face (2 or 3), weight 0 where it lies on none
        const double csx = onf[0] || onf[1] ? 1.0 : 0.0, csy = onf[2] || onf[3] ? 1.0 : 0.0;
        const int fsx = G::fslot(a == 0 ? 0 : 1, b), fsy = G::fslot(b == 0 ? 2 : 3, a);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            double r = 0.0;
#pragma unroll
            for (int j = 0; j < 4; ++j) r = fma(cw[j], sFV(v, fi[j]), r);
            r = fma(csx, sPe[v * PP + fsx], r);
            r = fma(csy, sPe[v * PP + fsy], r);
            RLO[v] = r;
        }
        if constexpr (MORT) {
            // a node lies on at most one x face (a = 0 or N) and one y face (b = 0 or
            // N): slot 0 takes the mortar of its x face, slot 1 that of its y face
            const int cx = onf[0] ? fcode[0] : (onf[1] ? fcode[1] : -1);
            const int cy = onf[2] ? fcode[2] : (onf[3] ? fcode[3] : -1);
            auto slot_of = [&](int code, int k) {
                const int S3 = fm_mortar(code) * 3 * n;
                return fm_small(code) ? S3 + n + fm_half(code) * n + k : S3 + k;
            };
            if (cx >= 0) {
                slot0 = slot_of(cx, b);
#pragma unroll
                for (int v = 0; v < 4; ++v) dS0[v] = A.slot[(size_t)slot0 * kSlotW + 4 + v];
            }
            if (cy >= 0) {
                slot1 = slot_of(cy, a);
#pragma unroll
                for (int v = 0; v < 4; ++v) dS1[v] = A.slot[(size_t)slot1 * kSlotW + 4 + v];
            }
            nmf = (cx >= 0) + (cy >= 0);
        }
    }
    if (MODE == MODE_LOWSOL) {
        // (products and sums as a stored residual would round them)
        double w[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) w[v] = u0[v] + dt * (RLO[v] * im);
        const double p = pressure<Rc>(w, g);
        if (act) {
            double* o = A.uout + ((unsigned)e * 2u * NN + (unsigned)q);
            o[0] = w[0];
            o[NN] = w[0] > 0.0 && p > 0.0 ? log(p) - g * log(w[0]) : __builtin_inf();
        }
        return;
    }

    const double dtm = dt * im;
    double uFV[4], cf[4][4];
    double rmin = 0.0, pmin = 0.0, th = 1.0;
    // local bounds: density floor (the larger of the local and the positivity
    // floor), ceiling, log entropy floor; thl the local node factor of the blend
    double rlf = 0.0, rhi = 0.0, lsm = 0.0, thl = 1.0;
    double lsi = 0.0;  // local bounds: the node's own low-order log entropy (cap of the entropy target)
    unsigned long long inad = 0;
    if (act) {
#pragma unroll
        for (int v = 0; v < 4; ++v) uFV[v] = u0[v] + dtm * RLO[v];
        const double pFV = pressure<Rc>(uFV, g);
        if (!(uFV[0] > 0.0) || !(pFV > 0.0)) inad = 1;
        rmin = A.beta * uFV[0];
        pmin = A.beta * pFV;
        if (need_loc && !BAR) {
            // bounds from the low-order solution over the node and its low-order
            // neighbours; the node's own low-order state, as computed here, is inside
            // them by definition (its stored copy may differ in the last bit)
            double rlo = uFV[0];
            rhi = uFV[0];
            lsi = uFV[0] > 0.0 && pFV > 0.0 ? log(pFV) - g * log(uFV[0]) : -__builtin_inf();
            lsm = lsi;
            auto take = [&](double lo, double hi, double ls) {
                rlo = fmin(rlo, lo);
                rhi = fmax(rhi, hi);
                lsm = fmin(lsm, ls);
            };
            // (at the element's edge the node itself once more, and its faces)
            const int nq[5] = {q, a > 0 ? q - 1 : q, a < N ? q + 1 : q, b > 0 ? q - n : q, b < N ? q + n : q};
#pragma unroll
            for (int j = 0; j < 5; ++j) take(sB[le][0][nq[j]], sB[le][0][nq[j]], sB[le][1][nq[j]]);
            if (onf[0] || onf[1]) {
                const int i = (onf[0] ? 0 : n) + b;
                take(sB[le][4][i], sB[le][5][i], sB[le][6][i]);
            }
            if (onf[2] || onf[3]) {
                const int i = (onf[2] ? 2 * n : 3 * n) + a;
                take(sB[le][4][i], sB[le][5][i], sB[le][6][i]);
            }
            rlf = fmax(rmin, rlo);
        } else if (need_loc) {
            // bounds over the node and the bar states of its low-order neighbours
            // (the node's own bar state is its input state: no cap)
            lsi = __builtin_inf();
            double rlo = u0[0];
            rhi = u0[0];
            lsm = ls_own;
            if (a > 0) {
                rlo = fmin(rlo, sB[le][0][q - 1]);
                rhi = fmax(rhi, sB[le][0][q - 1]);
                lsm = fmin(lsm, sB[le][1][q - 1]);
            }
            if (a < N) {
                rlo = fmin(rlo, sB[le][0][q]);
                rhi = fmax(rhi, sB[le][0][q]);
                lsm = fmin(lsm, sB[le][1][q]);
            }
            if (b > 0) {
                rlo = fmin(rlo, sB[le][2][q - n]);
                rhi = fmax(rhi, sB[le][2][q - n]);
                lsm = fmin(lsm, sB[le][3][q - n]);
            }
            if (b < N) {
                rlo = fmin(rlo, sB[le][2][q]);
                rhi = fmax(rhi, sB[le][2][q]);
                lsm = fmin(lsm, sB[le][3][q]);
            }
            const int fnq[4] = {0 * n + b, 1 * n + b, 2 * n + a, 3 * n + a};  // face lane of each face
#pragma unroll
            for (int f = 0; f < 4; ++f) {
                if (!onf[f]) continue;
                rlo = fmin(rlo, sB[le][4][fnq[f]]);
                rhi = fmax(rhi, sB[le][5][fnq[f]]);
                lsm = fmin(lsm, sB[le][6][fnq[f]]);
            }
            // the positivity floor stays: the density floor is the larger one
            rlf = fmax(rmin, rlo);
        }
        // the faces' increments dt / m_i w (f^HO - f^FV), signed (zero for missing faces)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const double wd = dtm * fweight(j);
#pragma unroll
            for (int v = 0; v < 4; ++v) cf[j][v] = wd * (sPe[v * PP + hslot(j)] - sFV(v, fidx(j)));
        }
        if (A.limiter != DGIDP_LIMIT_NONE) {
            if (PURE) {
                th = volume_factor<true>(uFV, cf, rlf, pmin, rhi, lsm, lsi, g, ig1);
            } else {
                th = volume_factor<false>(uFV, cf, rmin, pmin, 0.0, 0.0, 0.0, g, ig1);
                if (COMB && need_loc) thl = volume_factor<true>(uFV, cf, rlf, pmin, rhi, lsm, lsi, g, ig1);
            }
        }
    }
    // the blend keeps its local node factors in the first bar-state row, read
    // above for the bounds
    if (COMB) __syncthreads();
    if (act) {
        sTh(q) = th;
        if (COMB) sB[le][0][q] = thl;
    }
    __syncthreads();

    // ---- phase 7: limited volume update, SSP combination, mortar slots ----
    double asum = 0.0, thmin = 1.0;
    unsigned long long viol = 0;
    if (act) {
        double uvol[4];
        double tf[4];
        // face factor: the smaller of its two node factors; blended:
        // (1 - w) theta_pos + w theta_local
        // (a missing face reads the node itself; its increment is zero)
        const int qn4[4] = {a > 0 ? q - 1 : q, a < N ? q + 1 : q, b > 0 ? q - n : q, b < N ? q + n : q};
#pragma unroll
        for (int j = 0; j < 4; ++j)
            tf[j] = COMB ? (1.0 - w_e) * fmin(th, sTh(qn4[j])) + w_e * fmin(thl, sB[le][0][qn4[j]])
                         : fmin(th, sTh(qn4[j]));
#pragma unroll
        for (int v = 0; v < 4; ++v)
            uvol[v] = uFV[v] + tf[0] * cf[0][v] + tf[1] * cf[1][v] + tf[2] * cf[2][v] + tf[3] * cf[3][v];
        if (a < N) {
            asum += 1.0 - tf[1];
            thmin = fmin(thmin, tf[1]);
        }
        if (b < N) {
            asum += 1.0 - tf[3];
            thmin = fmin(thmin, tf[3]);
        }
        double* po = A.uout + ((unsigned)e * 4u * NN + (unsigned)q);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            // (un4 is zero where a = 0: the first stage's input is u^n itself)
            po[v * NN] = fma(A.a, un4[v], A.b * uvol[v]);
        }
        if (nmf == 0) {
            if (PURE) {
                if (A.st && (!(uvol[0] >= rlf * (1.0 - kLocalTol)) || uvol[0] > rhi * (1.0 + kLocalTol) ||
                             pressure<Rc>(uvol, g) < pmin ||
                             !(log(pressure<Rc>(uvol, g)) - g * log(uvol[0]) >= lsm - kLocalTol)))
                    viol = 1;
            } else if (A.limiter != DGIDP_LIMIT_NONE) {
                // p(uvol) >= pmin as 2 rho (E - pmin / (gamma - 1)) >= |m|^2 (rho >= rmin > 0)
                const double gp = 2.0 * uvol[0] * (uvol[3] - pmin * ig1) - (uvol[1] * uvol[1] + uvol[2] * uvol[2]);
                if (!(uvol[0] >= rmin) || !(gp >= 0.0)) viol = 1;
            }
        } else {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                if ((j == 0 ? slot0 : slot1) < 0) continue;
                const double* dS = j == 0 ? dS0 : dS1;
                double c[4], dc[4];
                bool fin = true;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    c[v] = dtm * dS[v];
                    dc[v] = nmf * c[v];
                    fin = fin && isfinite(dc[v]);
                }
                double ts = 1.0, tsl = 1.0;
                if (A.limiter != DGIDP_LIMIT_NONE) {
                    // an undefined high-order mortar flux keeps the low-order flux
                    if (!fin) {
                        ts = tsl = 0.0;
                    } else if (PURE) {
                        ts = mortar_factor<true>(uvol, dc, rlf, pmin, rhi, lsm, lsi, g, ig1);
                    } else {
                        ts = mortar_factor<false>(uvol, dc, rmin, pmin, 0.0, 0.0, 0.0, g, ig1);
                        if (COMB) tsl = mortar_factor<true>(uvol, dc, rlf, pmin, rhi, lsm, lsi, g, ig1);
                    }
                }
                double* S = A.slot + (size_t)(j == 0 ? slot0 : slot1) * kSlotW;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    S[v] = uvol[v];
                    S[4 + v] = c[v];
                }
                S[8] = ts;
                S[9] = PURE ? rlf : rmin;
                S[10] = pmin;
                if (PURE) {
                    S[11] = rhi;
                    S[12] = lsm;
                }
                if (COMB) {
                    S[13] = tsl;
                    S[14] = w_e;
                }
            }
        }
    }
    if (A.st) push_stats(A.st, inad, viol, thmin, asum, false);
}

// ---------------------------------------------------------------------------
// shock indicator of combined limiting (Sec. 3.5): the Hennemann indicator on
// the pressure, not capped, FP64, one value per element in internal order.
// One thread per node stages p, one thread per mode (i, j) forms its squared
// orthonormal-Legendre coefficient (the two passes of modal_x and modal_y_sq),
// thread 0 of the element reduces.
// ---------------------------------------------------------------------------
template <int N>
__device__ __forceinline__ double modal_x(const Tab<N>& tb, const double* Q, int a, int b)
{
    constexpr int n = N + 1;
    double r = 0.0;
#pragma unroll
    for (int aa = 0; aa < n; ++aa) r += tb.Vinv[a][aa] * Q[b * n + aa];
    return r;
}

template <int N>
__device__ __forceinline__ double modal_y_sq(const Tab<N>& tb, const double* Rx, int a, int b)
{
    constexpr int n = N + 1;
    double m = 0.0;
#pragma unroll
    for (int bb = 0; bb < n; ++bb) m += tb.Vinv[b][bb] * Rx[bb * n + a];
    return m * m;
}

template <int N>
__global__ __launch_bounds__(128) void k_shock_indicator(const double* __restrict__ u, int E, double gamma,
                                                         double* __restrict__ ind)
{
    constexpr int n = N + 1, NN = n * n, EPB = 128 / NN;
    __shared__ double sP[EPB][NN];
    __shared__ double sR[EPB][NN];
    const Tab<N>& tb = T<N>();
    const int tid = threadIdx.x;
    const int le = tid / NN, q = tid - le * NN, a = q % n, b = q / n;
    const int e = blockIdx.x * EPB + le;
    const bool act = tid < EPB * NN && e < E;
    if (act) {
        double w[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) w[v] = u[((size_t)e * 4 + v) * NN + q];
        sP[le][q] = (gamma - 1.0) * (w[3] - 0.5 * (w[1] * w[1] + w[2] * w[2]) / w[0]);
    }
    __syncthreads();
    if (act) sR[le][q] = modal_x<N>(tb, sP[le], a, b);
    __syncthreads();
    if (act) sP[le][q] = modal_y_sq<N>(tb, sR[le], a, b);  // sP now holds m^2
    __syncthreads();
    if (!act || q != 0) return;
    double all = 0.0, low1 = 0.0, low2 = 0.0;
    for (int j = 0; j < n; ++j)
        for (int i = 0; i < n; ++i) {
            const double m2 = sP[le][j * n + i];
            all += m2;
            if (i < N && j < N) low1 += m2;
            if (i < N - 1 && j < N - 1) low2 += m2;
        }
    const double en = fmax((all - low1) / all, (low1 - low2) / low1);
    const double T = 0.5 * pow(10.0, -1.8 * sqrt(sqrt((double)(N + 1))));
    const double s = log((1.0 - 1e-4) / 1e-4);
    const double al = 1.0 / (1.0 + exp(-(s / T) * (en - T)));
    ind[e] = al < 1e-3 ? 0.0 : al;
}

int launch_shock_indicator(int N, const DevMesh& m, const double* u, double gamma, hipStream_t s)
{
    if (m.E <= 0) return 0;
    const int EPB = 128 / ((N + 1) * (N + 1));
    const int grid = (m.E + EPB - 1) / EPB;
    if (N == 3) hipLaunchKernelGGL(k_shock_indicator<3>, dim3(grid), dim3(128), 0, s, u, m.E, gamma, m.shock_ind);
    else if (N == 4) hipLaunchKernelGGL(k_shock_indicator<4>, dim3(grid), dim3(128), 0, s, u, m.E, gamma, m.shock_ind);
    else return -1;
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
template <int N>
static int stage_N(const DevMesh& m, const KernelParams& kp, const double* uin, const double* un,
                   double* uout, double a, double b, const DtSource& dt, DevStats* st, int mode,
                   hipStream_t s, bool rev = false)
{
    using G = Geo<N>;
    StageArgs A;
    set_stage(A, m, kp, uin, un, uout, a, b, dt, st);
    A.ind = m.shock_ind;
    A.lsv = m.lsv;
    const int nb = (m.E + G::EPB - 1) / G::EPB;
    // on a large mesh dt is reduced once, and the stage reads it
    if (dt.dtmax && dt.dt_out && mode == MODE_STAGE && nb >= kFinalMin) {
        hipLaunchKernelGGL(k_dt_final, dim3(1), dim3(64), 0, s, dt.dtmax, dt.cfl, dt.dt_out, st);
        A.dt = dt.dt_out;
        A.dtmax = nullptr;
    }
    const bool mixed = kp.precision == DGIDP_MIXED;
    const int lk = kp.limiter == DGIDP_LIMIT_LOCAL ? 1
                   : kp.limiter == DGIDP_LIMIT_COMBINED ? 2
                   : kp.limiter == DGIDP_LIMIT_LOCAL_LOWORDER ? 3 : 0;
    // one launch of the mortar variant over all batches, or of the conforming one on a
    // mesh without mortars: its conforming variant keeps three waves per SIMD too, so
    // two launches would only add a tail
    auto go = [&](auto modec, auto mixc, auto lkc) {
        constexpr int MD = decltype(modec)::value, LK = decltype(lkc)::value;
        constexpr bool MX = decltype(mixc)::value;
        if (m.nbm > 0) hipLaunchKernelGGL((k_stage<N, MD, MX, LK, true>), dim3(nb), dim3(G::BS), 0, s, A);
        else {
            A.rev = rev ? 1 : 0;
            hipLaunchKernelGGL((k_stage<N, MD, MX, LK, false>), dim3(nb), dim3(G::BS), 0, s, A);
        }
    };
    using I0 = std::integral_constant<int, 0>;
    using BT = std::true_type;
    using BF = std::false_type;
    using MS = std::integral_constant<int, MODE_STAGE>;
    if (mode == MODE_LOWSOL) {
        go(std::integral_constant<int, MODE_LOWSOL>(), BF(), I0());
    } else if (lk == 3) {
        if (mixed) go(MS(), BT(), std::integral_constant<int, 3>());
        else go(MS(), BF(), std::integral_constant<int, 3>());
    } else if (lk == 1) {
        if (mixed) go(MS(), BT(), std::integral_constant<int, 1>());
        else go(MS(), BF(), std::integral_constant<int, 1>());
    } else if (lk == 2) {
        if (mixed) go(MS(), BT(), std::integral_constant<int, 2>());
        else go(MS(), BF(), std::integral_constant<int, 2>());
    } else {
        return -1;
    }
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_stage(int N, const DevMesh& m, const KernelParams& kp, const double* uin,
                 const double* un, double* uout, double a, double b, const DtSource& dt,
                 DevStats* st, hipStream_t s, bool rev)
{
    if (m.E == 0) return 0;
    if (N == 3) return stage_N<3>(m, kp, uin, un, uout, a, b, dt, st, MODE_STAGE, s, rev);
    if (N == 4) return stage_N<4>(m, kp, uin, un, uout, a, b, dt, st, MODE_STAGE, s, rev);
    return -1;
}

int launch_lowsol(int N, const DevMesh& m, const KernelParams& kp, const double* u, const DtSource& dt, hipStream_t s)
{
    if (m.E == 0) return 0;
    if (N == 3) return stage_N<3>(m, kp, u, nullptr, m.lsv, 0.0, 1.0, dt, nullptr, MODE_LOWSOL, s);
    if (N == 4) return stage_N<4>(m, kp, u, nullptr, m.lsv, 0.0, 1.0, dt, nullptr, MODE_LOWSOL, s);
    return -1;
}

int launch_dt(int N, const DevMesh& m, const KernelParams& kp, const double* u, int mode,
              unsigned long long* acc, unsigned long long* other, hipStream_t s)
{
    return run_dt<Rc>(N, dt_args(m, kp, u, mode, acc, other), s);
}

int launch_mortar(int N, const DevMesh& m, const KernelParams& kp, double* uout, double b, DevStats* st, hipStream_t s)
{
    return run_mortar<Rc, true>(N, {m.slot, m.slot_node, m.slot_partner, m.M, uout, b, kp.gamma, kp.limiter, st}, s);
}

}  // namespace local
}  // namespace dgidp
