// HIP kernels of dgidp for gfx950 (MI355X).
//
// One SSP-RK3 stage (Sec. 2.3 and Sec. 3 intro of the paper) is two parts:
//   k_stage   one thread per LGL node; a block holds 4 elements in one wave
//             (N = 3) or 5 elements in two waves (N = 4).  It stages the element in LDS,
//             evaluates the surface fluxes with one lane per face node
//             (conforming LLF, Kopriva's L2 mortar, the sparse IDP mortar flux
//             of eq. interfaceflux_local), the Ranocha two-point fluxes once per
//             node pair of every line, sums them to high-order subcell
//             fluxes (eq. fluxdifferencingform), evaluates the LLF subcell
//             fluxes (eq. FVmethod), forms the low-order update and the
//             positivity bounds (eq. Bounds_Positivity), limits the volume
//             antidiffusive fluxes per subcell face and writes a u^n + b u^vol.
//             Nodes on mortars also leave a slot record with their mortar
//             antidiffusive increment and their own admissible fraction of it.
//   k_mortar  one thread per mortar slot: the mortar's factor is the minimum
//             over its slots (one factor per mortar keeps the flux conservative,
//             Sec. 2.3); corrections are added in ascending mortar order.  On large
//             meshes the first blocks of k_stage's second launch do this.
// The time step (eq. timestep_restriction) is a per-block max (k_dt, on large meshes
// k_dt_rows) merged by one 64-bit atomic max per block into one of kDtSpread accumulators; the first
// stage kernel of the step reduces those and takes dt = cfl / max.
// k_mortar, k_dt and what else dgidp_local.hip has in common are in dgidp_device.h.
#include <hip/hip_runtime.h>

#include <cmath>
#include <type_traits>

#include "dgidp_device.h"
#include "dgidp_mlp_dev.h"

namespace dgidp {

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
struct Rc : Rcp3 {
    template <int N>
    static __device__ __forceinline__ const Tab<N>& tab()
    {
        return T<N>();
    }
};

// launch geometry per degree: one-wave blocks of 4 elements at N = 3 (the
// phase barriers stay inside a wave and a late block holds less work),
// two-wave blocks of 5 elements at N = 4 (125 of 128 lanes busy; a block of the
// conforming variant takes 18.3 KB of LDS, so eight blocks, sixteen waves, fill a
// compute unit to the four waves per SIMD that its 128 registers allow).  An earlier
// form of the kernel took 410.9 us per launch on the 246,736-leaf workload in
// three-wave blocks of 7 elements (175 of 192 lanes, four blocks per unit), and
// 385.4 in two-wave blocks.
template <int N>
struct Geo {
    static constexpr int n = N + 1, NN = n * n;
    static constexpr int BS = N == 3 ? 64 : 128;   // block size
    static constexpr int EPB = BS / NN;            // 4 for N = 3, 5 for N = 4
    static_assert(EPB == stage_block_elems(N), "host element order assumes this block size");
    static constexpr int NT = EPB * NN;            // active threads
    static constexpr int NFN = 4 * n;              // face nodes per element
    // LDS per element: 8 rows of primitives, one value per node, and per variable
    // the pair buffer.  It takes the pair fluxes that other threads need (see
    // the pair phase), then the antidiffusive fluxes of the x faces at the node
    // on their left and of the y faces at the node below (rounds of NN); the
    // mortar variant first stages the mortar traces there (12 n).  A LDS access
    // serves 16 lanes a cycle where their doubles differ modulo 16, so the
    // element strides are 9 modulo 16 at N = 4: consecutive threads, 25 to an
    // element, then meet no conflict.
    static constexpr int PV = N == 4 ? 2 * NN + 2 * n : 2 * NN;  // sPair variable stride
    static constexpr int pp(bool mort) { return mort && 12 * n > PV ? 12 * n : PV; }
    static constexpr int pad9(int x) { return N == 4 ? x + (25 - x % 16) % 16 : x; }
    static constexpr int ES = pad9(8 * NN);                        // sR element stride
    static constexpr int es(bool mort) { return pad9(4 * pp(mort)); }  // sPair element stride
};

// The node pairs of an element, N per thread: each of thread (a, b)'s pairs holds
// its own node, whose primitives it then reads once per pass.  At N = 4 the
// partners are a + 1 and a + 2 (modulo n) on its x line, then the same on its y
// line; at N = 3 a + 1, b + 1 and, in a last round, a + 2 where a / 2 + b / 2 is
// even and b + 2 where it is odd.  Every pair of every line occurs once.  Entry,
// 16 bits: the partner's node | (l n + k) << 5 | d << 10 | own << 11 with l < k
// the positions along the line (the entry of Sbar), d the direction, own = 1
// where this thread's node is k.
template <int N>
struct PairMap {
    static constexpr int n = N + 1, NN = n * n;
    unsigned int code[NN][(N + 1) / 2];
    constexpr PairMap() : code()
    {
        for (int q = 0; q < NN; ++q)
            for (int i = 0; i < N; ++i) {
                const int a = q % n, b = q / n;
                int d = 0, step = 0;
                if (N == 4) {
                    d = i / 2;
                    step = 1 + i % 2;
                } else {
                    d = i < 2 ? i : (a / 2 + b / 2) % 2;
                    step = i < 2 ? 1 : 2;
                }
                const int me = d == 0 ? a : b, other = (me + step) % n;
                const int qo = d == 0 ? b * n + other : other * n + a;
                const int l = me < other ? me : other, k = me < other ? other : me;
                code[q][i / 2] |= (unsigned)(qo | (l * n + k) << 5 | d << 10 | (me == k ? 1 : 0) << 11)
                                  << (16 * (i % 2));
            }
    }
};

// The face node that the thread of node q = (a, b) evaluates: a node of an x
// face its own x face, an inner node of a y face its own y face; the y faces at
// the four corners go to the four interior nodes next to them.  So all but those
// four hold a face's surface term on the thread that adds it.  Entry
// f | k << 2 | qo << 5 | qn << 10 | own << 15 | corner << 16: the face, the
// position along it, its node and the node across a conforming face; own: the
// face's node is q; corner: the term goes to a corner node.  Neither is set for
// the threads without a face (N = 4: the middle cross), which repeat another's.
template <int N>
struct FaceMap {
    static constexpr int n = N + 1, NN = n * n;
    unsigned int code[NN];
    static constexpr int node(int f, int k)
    {
        return f < 2 ? k * n + (f & 1) * N : k + (f & 1) * N * n;
    }
    constexpr FaceMap() : code()
    {
        for (int q = 0; q < NN; ++q) {
            const int a = q % n, b = q / n;
            const bool xf = a == 0 || a == N, yf = b == 0 || b == N;
            const bool corner = !xf && !yf && (a == 1 || a == N - 1) && (b == 1 || b == N - 1);
            const int f = xf ? (a == N ? 1 : 0) : yf ? (b == N ? 3 : 2) : corner ? (b == N - 1 ? 3 : 2) : 0;
            const int k = xf ? b : yf ? a : corner ? (a == N - 1 ? N : 0) : b;
            code[q] = (unsigned)(f | k << 2 | node(f, k) << 5 | node(f ^ 1, k) << 10 | (xf || yf ? 1 : 0) << 15 |
                                 (corner ? 1 : 0) << 16);
        }
    }
};
__constant__ FaceMap<3> c_fm3 = FaceMap<3>();
__constant__ FaceMap<4> c_fm4 = FaceMap<4>();
template <int N>
__device__ __forceinline__ unsigned face_entry(int q);
template <>
__device__ __forceinline__ unsigned face_entry<3>(int q) { return c_fm3.code[q]; }
template <>
__device__ __forceinline__ unsigned face_entry<4>(int q) { return c_fm4.code[q]; }
__constant__ PairMap<3> c_pm3 = PairMap<3>();
__constant__ PairMap<4> c_pm4 = PairMap<4>();
template <int N>
__device__ __forceinline__ unsigned pair_entry(int q, int i);  // pairs 2 i and 2 i + 1
template <>
__device__ __forceinline__ unsigned pair_entry<3>(int q, int i) { return c_pm3.code[q][i]; }
template <>
__device__ __forceinline__ unsigned pair_entry<4>(int q, int i) { return c_pm4.code[q][i]; }

// ---------------------------------------------------------------------------
// arithmetic helpers
// ---------------------------------------------------------------------------
// Half the logarithmic mean, x^ln / 2 with x^ln = (x - y) / (ln x - ln y), and
// the inverse one, 1 / x^ln.  With s = x + y, d = x - y, f = d / s, z = f^2
//   x^ln / 2 = (s/4) f / atanh f,   1 / x^ln = (2 / s) atanh f / f
// (ln x - ln y = 2 atanh f, as in Ismail & Roe 2009), both analytic in z:
//   z < 1e-4: the series
//     s (1/4 - (11/945) z (945/132 + z (21/11 + z))) and (2 + (2/7) z (7/3 + z (7/5 + z))) / s
//     (the next terms are at most 3.1e-18 and 1.2e-17 relative there; monic, so that an
//     instruction has one literal at most)
//   z < kLnPoly, x / y between 0.71 and 1.41: polynomials of seven coefficients with the least
//     largest error (4.2e-19 and 1.8e-18 relative as rounded to doubles), so that a pair
//     needs no logarithms of its nodes
//   beyond: the logarithm of the ratio.
constexpr double kLnSeries = 1e-4;
constexpr double kLnPoly = 0.0294;
__device__ __forceinline__ double half_lnmean_series(double s, double z)
{
    const double t = fma(z, z + 21.0 / 11.0, 945.0 / 132.0) * z;
    return s * fma(-11.0 / 945.0, t, 0.25);
}
__device__ __forceinline__ double inv_lnmean_series(double r, double z)
{
    const double t = fma(z, z + 7.0 / 5.0, 7.0 / 3.0) * z;
    return fma(2.0 / 7.0, t, 2.0) * r;
}
__device__ __forceinline__ double half_lnmean_poly(double s, double z)
{
    double t = fma(z, -0x1.e7f35bc2ef6bbp-9, -0x1.11f376d9b629ap-8);
    t = fma(z, t, -0x1.65255cdd70460p-8);
    t = fma(z, t, -0x1.eeb2bc5db1c99p-8);
    t = fma(z, t, -0x1.7d6d2c3e58a33p-7);
    t = fma(z, t, -0x1.6c16c16c0d016p-6);
    t = fma(z, t, -0x1.5555555555561p-4);
    return s * fma(z, t, 0.25);
}
// (2 atanh f / f - 2) / z, |f| < 0.1716: also the logarithm's polynomial
__device__ __forceinline__ double atanh_poly(double z)
{
    double t = fma(z, 0x1.2f056395f5a67p-3, 0x1.39a1bab2e7e3cp-3);
    t = fma(z, t, 0x1.74663ee8bc916p-3);
    t = fma(z, t, 0x1.c71c52095abb5p-3);
    t = fma(z, t, 0x1.24924941f1295p-2);
    t = fma(z, t, 0x1.999999997fdb7p-2);
    return fma(z, t, 0x1.5555555555592p-1);
}
__device__ __forceinline__ double inv_lnmean_poly(double r, double z) { return fma(z, atanh_poly(z), 2.0) * r; }

// Natural logarithms of x and y, both normal (NaN for an argument <= 0 or NaN):
// x = m 2^k with m in [sqrt(1/2), sqrt(2)), f = m - 1 (exact), s = f / (2 + f), so
// that ln m = 2 atanh s = 2 s + T, T = 2 s^3/3 + 2 s^5/5 + ..., and 2 s = f - s f
// gives ln m = f - s (f - T / s) with T / s = z (2/3 + 2 z/5 + ...) in z = s^2 < 0.0295
// (here the polynomial of seven coefficients with the least largest error, 2.2e-18
// of ln m); ln x = k ln 2 + ln m with ln 2 split into a head whose product
// with k is exact and a tail.  About 1 ulp; the two share one reciprocal, of
// (2 + f_x)(2 + f_y) between 2.9 and 5.9.
struct LogParts {
    double f, k;
};
__device__ __forceinline__ LogParts log_split(double x)
{
    const double m = __builtin_amdgcn_frexp_mant(x);  // [0.5, 1)
    const int k = __builtin_amdgcn_frexp_exp(x);
    const bool low = m < 0x1.6a09e667f3bcdp-1;
    return LogParts{low ? fma(2.0, m, -1.0) : m - 1.0, (double)(low ? k - 1 : k)};
}
__device__ __forceinline__ double log_join(const LogParts& p, double r, double x)
{
    const double sf = p.f * r;
    const double z = sf * sf;
    const double lm = fma(-sf, fma(-z, atanh_poly(z), p.f), p.f);
    const double l = fma(p.k, 0x1.62e42fefp-1, fma(p.k, 0x1.473de6af278edp-34, lm));
    return x > 0.0 ? l : __builtin_nan("");
}
__device__ __forceinline__ void flog2(double x, double y, double& lx, double& ly)
{
    const LogParts px = log_split(x), py = log_split(y);
    const double dx = 2.0 + px.f, dy = 2.0 + py.f;
    const double r = Rc::rcp(dx * dy);
    lx = log_join(px, dy * r, x);
    ly = log_join(py, dx * r, y);
}

// Node factor of the volume limiter from the node's four face increments cf
// (dt/m_i-scaled, zero for missing faces): the Zalesak factor for the density
// floor rfl and the pressure root per face, this on Gamma = 4-scaled increments.
__device__ __forceinline__ double volume_factor(const double* uFV, const double (&cf)[4][4], double rfl,
                                                double pfl, double ig1)
{
    const double rt = rfl * kMargin, pt = pfl * kMargin;
    // Zalesak: the sum of the negative density increments may use at most the
    // distance to the floor
    double P = 0.0;
#pragma unroll
    for (int j = 0; j < 4; ++j) P += fmin(cf[j][0], 0.0);
    double th = 1.0;
    if (P < 0.0) th = fmax(fmin((rt - uFV[0]) * Rc::rcp(P), 1.0), 0.0);
    // pressure: each face's increment scaled by Gamma = 2d = 4 (a zero
    // increment, as on a missing face, admits theta = 1 at an admissible uFV).
    // All four full steps are tested first, without a branch; only a wave with a
    // node that fails one runs the roots
    bool full = true;
    {
        const double e0 = uFV[3] - pt * ig1;
        const double g0 = uFV[0] * e0 - 0.5 * (uFV[1] * uFV[1] + uFV[2] * uFV[2]);
        full = g0 > 0.0 && uFV[0] > 0.0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const double r1 = fma(4.0, cf[j][0], uFV[0]);
            const double m1 = fma(4.0, cf[j][1], uFV[1]), m2 = fma(4.0, cf[j][2], uFV[2]);
            const double g1v = fma(4.0, cf[j][3], e0) * r1 - 0.5 * (m1 * m1 + m2 * m2);
            full = full && r1 > 0.0 && g1v >= 0.0;
        }
    }
    if (!full) {
#pragma unroll
        for (int j = 0; j < 4; ++j) th = fmin(th, theta_p<4>(uFV, cf[j], pt, ig1));
    }
    return th;
}

// Factor of one mortar node for its n_i-scaled increment dc on top of u^vol:
// density floor and pressure root, both against half the volume margin.
__device__ __forceinline__ double mortar_factor(const double* uvol, const double* dc, double rfl, double pfl,
                                                double ig1)
{
    const double rt = rfl * kMarginMortar, pt = pfl * kMarginMortar;
    double ts = 1.0;
    if (dc[0] < 0.0) ts = fmin(ts, fmax((rt - uvol[0]) / dc[0], 0.0));
    return fmin(ts, theta_p(uvol, dc, pt, ig1));
}

// ---------------------------------------------------------------------------
// element kernel
// ---------------------------------------------------------------------------
// The low-order residual skips the pair fluxes.
enum { MODE_STAGE = 0, MODE_RHS_HIGH = 1, MODE_RHS_LOW = 2 };

struct StageArgs {
    const double* uin;
    const double* un;
    double* uout;
    double a, b;
    const double* dt;
    // when set, dt = cfl / max over the accumulator set dtmax (bits of
    // non-negative doubles); block 0 stores it in dt_out
    const unsigned long long* dtmax;
    double cfl;
    double* dt_out;
    const int* fnbr;
    const int* fnbr2;
    const int* fmort;
    // (not read; it keeps the members' places: without it the compiler groups the loads of
    // the arguments otherwise, and five steps of the 304-leaf mesh take 222 us for 219)
    const int* mort;
    const double* h;
    double* slot;
    const int8_t* bkind;  // boundary nodes: condition and exterior state
    const double* bext;
    // element batches of this launch: blist[boff + i], i < gridDim.x (the
    // batches holding a mortar element and the others are separate launches)
    const int* blist;
    int boff;
    int E;
    double gamma, beta;
    double ig1;  // 1 / (gamma - 1)
    int rev;     // walk the XCD batch ranges from their ends (conforming variant only)
    int limiter;
    int vflux;  // two-point volume flux: DGIDP_FLUX_RANOCHA or DGIDP_FLUX_CHANDRASHEKAR
    DevStats* st;
    // the first mblocks blocks of a conforming launch, a multiple of 8, correct the
    // mortars of the launch before it instead: neither reads what the other writes, and
    // most of a launch of little work is hidden.  On the 246,736-leaf mesh the corrections
    // take 8.6 to 10.5 us in a launch of their own and lengthen the conforming launch by
    // 4 us; five steps 3,780 us before, 3,729 now (with the time step taken by the mortar
    // elements' launch).
    int mblocks;
    MortarArgs mo;
};

// node qq of the block's element le from its LDS rows; the momenta are formed
// again from the primitives (rho v = rho * v: within an ulp of the stored
// state, the same for every reader of a node, so that equal states still meet
// in a zero flux difference), in the mixed mode also the energy
// (E = p / (gamma - 1) + (rho v . v) / 2)
#define LDS_NODE(X, qq)                                                    \
    do {                                                                   \
        X.r = sRe[0 * NN + (qq)];                                           \
        X.v1 = sRe[1 * NN + (qq)];                                          \
        X.v2 = sRe[2 * NN + (qq)];                                          \
        X.p = sRe[3 * NN + (qq)];                                           \
        X.c = sRe[4 * NN + (qq)];                                           \
        X.u[0] = X.r;                                                      \
        X.u[1] = X.r * X.v1;                                               \
        X.u[2] = X.r * X.v2;                                               \
        X.u[3] = MIXED ? fma(X.p, ig1, 0.5 * (X.u[1] * X.v1 + X.u[2] * X.v2)) : sRe[5 * NN + (qq)]; \
    } while (0)

// The positivity bounds (or none, at run time); the modes with local bounds have a
// kernel of their own (dgidp_local.hip, which says why).
// MORT: the launch over the element batches that hold a mortar element (the
// surface phase with Kopriva's mortar and the sparse low-order mortar flux,
// mortar slot records), or over all; the other batches of a stage of two launches
// run the MORT = false variant, which has no mortar code.
// Bound: vector instructions and LDS accesses, each busy for about two thirds of
// the time (the HBM floor is a third), so every phase is written for few of both:
// pairs on their series or polynomial without logarithms, fluxes in their
// face's frame with the weight folded into the wave speeds, one reciprocal for
// several quotients, the faces' roles from a table, lanes that repeat a node
// instead of being switched off, a thread's pairs around its own node with
// its share of the face sums in registers, and strides without bank conflicts.
// Conforming launch of the 246,736-leaf N = 4 mesh, per wave: 799 vector and 92
// LDS instructions (748 LDS cycles, 186 of them conflicts), from 1,119 and 112
// (1,121, 393); 182 us of the stage, from 229.  More waves do not help: at 92
// registers and 16.3 KB of LDS per block, five per SIMD instead of four, the same
// instructions took the same time.
template <int N, int MODE, bool MIXED, bool MORT>
// waves per SIMD: four (128 registers), but for the FP64 N = 3 variant with mortars (148
// registers, three waves, see LATE)
__global__ __launch_bounds__(Geo<N>::BS) __attribute__((amdgpu_waves_per_eu((!MORT || N == 4 || MIXED) ? 4 : 3)))
void k_stage(StageArgs A)
{
    using G = Geo<N>;
    // PAIRS: the pair fluxes and antidiffusive fluxes are needed
    constexpr bool PAIRS = MODE == MODE_STAGE || MODE == MODE_RHS_HIGH;
    constexpr int n = G::n, NN = G::NN, EPB = G::EPB, NT = G::NT;
    constexpr int PP = G::pp(MORT);
    static_assert(N == 3 || N == 4, "pair map and face sums");
    constexpr int MB = 4 * n;  // offset of the mortar-node fluxes in the pair buffer
    // LATE: the large sides form their high-order mortar fluxes after every lane
    // has read the staged traces, in place of them, and u^n, the state and the mortar
    // increments are read where they are used: 128 registers instead of 148,
    // four waves per SIMD.  Early, they are formed beside the low-order pairs and held
    // over the barrier, at three: a shorter chain, which counts where a mesh does not fill
    // those waves.  At N = 4 the 14,871-leaf blast took 414 us early and 402 late, five
    // steps.  At N = 3 the line lies at some 40,000 leaves, but a variant is early or
    // late for all sizes, FP64 early and mixed late.  FP64, early and late: 304
    // leaves 219 and 222, 22,156 352 and 353, 44,788 556 and 554, 50,160 585 and 564, 59,392
    // 664 and 650; mixed: 304 220 and 224, 22,156 341 and 347, 59,392 662 and 647.
    constexpr bool LATE = MORT && (N == 4 || MIXED);

    // per node: rho, v1, v2, p, c, E, z = rho / p (mixed: FP32 pairs in rows 5-7)
    __shared__ double sR[EPB * G::ES];
    __shared__ double sPair[EPB * G::es(MORT)];  // pair fluxes, then antidiffusive fluxes and corner terms
    __shared__ double sTw[2][n];              // LGL weights and their reciprocals, read per lane
    __shared__ double sS[n][n];               // Sbar / 2, read per pair
    // After phase 5b the primitive rows of sR are read no more: they take the
    // low-order subcell fluxes, rows of N n (the x faces b N + a in rows 0-3, the
    // y faces b n + a in rows 4-7), and after them the node factors.
    constexpr int NFH = N * n;
    static_assert(8 * NFH + NN <= 8 * NN, "subcell fluxes and node factors reuse sR");

    const Tab<N>& tb = T<N>();
    const double g = A.gamma, ig1 = A.ig1;
    // every lane runs every phase: the lanes past the block's nodes repeat
    // nodes of their own wave, those past the mesh's last element repeat it in
    // LDS rows of their own; act masks what goes to memory
    static_assert(NT <= G::BS && G::BS - NT <= NN && (G::BS - NT == 0 || NT - NN >= G::BS - 64),
                  "the last lanes repeat nodes of their own wave");
    const int tid = threadIdx.x;
    int bid = blockIdx.x, nblk = gridDim.x;
    if constexpr (!MORT && MODE == MODE_STAGE) {
        if (bid < A.mblocks) {
            mortar_slot<N, Rc, false>(A.mo, bid * G::BS + tid);
            return;
        }
        bid -= A.mblocks;
        nblk -= A.mblocks;
    }
    const int tl = tid < NT ? tid : tid - NN;
    const int le = tl / NN, q = tl - le * NN, a = q % n, b = q / n;
    const int xb = !MORT && A.rev ? xcd_batch_rev(bid, nblk) : xcd_batch(bid, nblk);
    const int e0 = (A.blist ? A.blist[A.boff + xb] : xb) * EPB;
    const bool act = tid < NT && e0 + le < A.E;
    const int e = e0 + le < A.E ? e0 + le : A.E - 1;
    double* const sRe = sR + le * G::ES;           // the element's rows
    double* const sPe = sPair + le * G::es(MORT);  // and its pair buffer
    double* const sT = sRe + 8 * NFH;      // node factors
    const unsigned role = face_entry<N>(q);
    unsigned pcode[(N + 1) / 2];  // this thread's node pairs (the pair map)
#pragma unroll
    for (int i = 0; i < (N + 1) / 2; ++i) pcode[i] = pair_entry<N>(q, i);
    if (tid < n) {
        sTw[0][tid] = tb.w[tid];
        sTw[1][tid] = tb.winv[tid];
    }
    if (tid < NN) (&sS[0][0])[tid] = 0.5 * (&tb.S[0][0])[tid];

    // ---- phase 1: own node into LDS; face-node role and its remote loads ----
    // the face node this lane also evaluates: its face, position, node, the node across
    const int ff = role & 3, fk = (role >> 2) & 7, qfo = (role >> 5) & 31, qfn = (role >> 10) & 31;
    const bool fown = (role >> 15) & 1, fcor = (role >> 16) & 1;
    const int dff = ff >> 1;
    const bool lowf = ff & 1;                    // element on the low side of face ff
    // issue the independent global loads first
    const int fcode_f = A.fmort[e * 4 + ff];
    const int fnb = A.fnbr[e * 4 + ff];
    int fcode[4];  // the element's face codes (mortar slots)
    if (MORT)
#pragma unroll
        for (int f = 0; f < 4; ++f) fcode[f] = A.fmort[e * 4 + f];
    const int fnb2 = MORT ? A.fnbr2[e * 4 + ff] : -1;
    // conforming neighbour state (boundary: exterior state) across face ff at fk
    // in the face's frame: density, normal and tangential momentum, energy
    // (large side: the first small element's trace in the x, y frame)
    double onb[4];
    double us1[4];  // large side: the second small element's trace at position fk
    int bk = 0;
    const double dtpart =
        A.dtmax ? __longlong_as_double((long long)A.dtmax[(tid & 63) * kDtStride]) : 0.0;
    double u0[4];  // this node's state
    {
        NodeP me;
        load_node<N, Rc>(A.uin, e, q, me, g);
#pragma unroll
        for (int v = 0; v < 4; ++v) u0[v] = me.u[v];
        // mixed mode: rows 5-7 hold the FP32 operands of the two-point volume
        // fluxes in pairs (rho, p), (ln rho, z), (ln z, 0)
        const double z = PAIRS ? me.r * Rc::rcp(me.p) : 0.0;
        sRe[(0) * NN + q] = me.r;
        sRe[(1) * NN + q] = me.v1;
        sRe[(2) * NN + q] = me.v2;
        sRe[(3) * NN + q] = me.p;
        sRe[(4) * NN + q] = me.c;
        if (MIXED) {
            sRe[5 * NN + q] = pack2((float)me.r, (float)me.p);
            sRe[6 * NN + q] = pack2(__logf((float)me.r), (float)z);
            sRe[7 * NN + q] = pack2(__logf((float)z), 0.0f);
        } else {
            sRe[5 * NN + q] = me.u[3];
            // (a negative density, which only the unlimited scheme can reach, leaves
            // its pair fluxes undefined)
            if (PAIRS) sRe[6 * NN + q] = me.r > 0.0 ? z : __builtin_nan("");
        }
    }
    const double hx = A.h[2 * e], hy = A.h[2 * e + 1];
    if (MORT && fcode_f >= 0) {
        if (!fm_small(fcode_f)) {
            // large side: stage both small traces at position fk
            load_u<N>(A.uin, fnb, qfn, onb);
            load_u<N>(A.uin, fnb2, qfn, us1);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                sPe[v * PP + MB + (ff * 2 + 0) * n + fk] = onb[v];
                sPe[v * PP + MB + (ff * 2 + 1) * n + fk] = us1[v];
            }
        } else {
            // small side: stage the large face trace for the interpolation
            double w[4];
            load_u<N>(A.uin, fnb, qfn, w);
#pragma unroll
            for (int v = 0; v < 4; ++v) sPe[v * PP + ff * n + fk] = w[v];
        }
    } else if (fcode_f < -1) {
        const int j = (-2 - fcode_f) * n + fk;
        bk = A.bkind[j];
#pragma unroll
        for (int v = 0; v < 4; ++v) onb[v] = A.bext[(size_t)j * 4 + v];
    } else {
        const double* p = A.uin + ((unsigned)fnb * 4u * NN + (unsigned)qfn);
        const double* pn = p + (1 + dff) * NN;
        const double* pt = p + (2 - dff) * NN;
        onb[0] = p[0];
        onb[1] = pn[0];
        onb[2] = pt[0];
        onb[3] = p[3 * NN];
    }
    __syncthreads();
    double dt;
    if (A.dtmax) {
        const double m = wave_max(dtpart);
        dt = A.cfl / m;
        if (bid == 0 && threadIdx.x == 0) {
            *A.dt_out = dt;
            if (A.st) A.st->dt = dt;
        }
    } else {
        dt = A.dt ? *A.dt : 0.0;
    }

    // high-order flux on the mortar of a large side, at position fk of half hh, between
    // the face interpolated to it (its nodes' conserved states formed as
    // LDS_NODE does) and the small side's trace u, which the flux replaces
    auto mortar_ho = [&](int hh, double (&u)[4]) {
        NodeP ui, us;
#pragma unroll
        for (int v = 0; v < 4; ++v) us.u[v] = u[v];
        make_node<Rc>(us, g);
        double ia[4] = {0, 0, 0, 0};
#pragma unroll
        for (int j = 0; j < n; ++j) {
            const int qj = face_q<N>(ff, j);
            const double r = sRe[0 * NN + qj], v1 = sRe[1 * NN + qj], v2 = sRe[2 * NN + qj];
            const double m1 = r * v1, m2 = r * v2;
            const double E = MIXED ? fma(sRe[3 * NN + qj], ig1, 0.5 * (m1 * v1 + m2 * v2)) : sRe[5 * NN + qj];
            const double uj[4] = {r, m1, m2, E};
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                if (MIXED) ia[v] = (float)ia[v] + tb.If[hh][fk][j] * (float)uj[v];
                else ia[v] += tb.I[hh][fk][j] * uj[v];
            }
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) ui.u[v] = ia[v];
        make_node<Rc>(ui, g);
        mortar_flux(dff, lowf, ui, us, u);
    };
    // ---- phase 2: one surface flux per face node: the low-order surface term ----
    const double sgf = lowf ? -1.0 : 1.0;
    const double hff = ff < 2 ? hy : hx;
    double fterm[4];
    {
        NodeP own;  // the face node's state (mortars)
        if (MORT) LDS_NODE(own, qfo);
        if (fcode_f < 0) {
            if (fcode_f < -1) {
                NodeP me;
                LDS_NODE(me, qfo);
                double gu[4];
                boundary_ghost(bk, onb, me, ff, g, gu);
                onb[0] = gu[0];
                onb[1] = dff == 0 ? gu[1] : gu[2];
                onb[2] = dff == 0 ? gu[2] : gu[1];
                onb[3] = gu[3];
            }
            // LLF in the face's frame, the face node from its LDS rows (the
            // arithmetic of LDS_NODE).  With W = +-w h / 2 (minus on the low side),
            // W F = W/2 (f_own + f_o) + |W|/2 lambda (u_o - u_own) on either side
            const double r = sRe[(0) * NN + qfo], vn = sRe[(1 + dff) * NN + qfo], vt = sRe[(2 - dff) * NN + qfo];
            const double p = sRe[(3) * NN + qfo], c = sRe[(4) * NN + qfo];
            const double mn = r * vn, mt = r * vt;
            const double E = MIXED ? fma(p, ig1, 0.5 * fma(mn, vn, mt * vt)) : sRe[5 * NN + qfo];
            const double ir = Rc::rcp(onb[0]);
            const double on = onb[1] * ir, ot = onb[2] * ir;
            const double op = (g - 1.0) * (onb[3] - 0.5 * fma(onb[1], on, onb[2] * ot));
            const double oc = fsqrt(g * op * ir);
            const double W = 0.25 * hff * sTw[0][fk];
            const double K = W * fmax(fabs(vn) + c, fabs(on) + oc);
            const double Ws = sgf * W, wa = Ws * vn, wb = Ws * on;
            double F[4];
            F[0] = fma(K, onb[0] - r, fma(onb[0], wb, r * wa));
            F[1] = fma(K, onb[1] - mn, fma(onb[1], wb, mn * wa));
            F[2] = fma(K, onb[2] - mt, fma(onb[2], wb, mt * wa));
            F[3] = fma(K, onb[3] - E, fma(onb[3], wb, E * wa));
            F[1] = fma(Ws, p + op, F[1]);
            F[3] += fma(op, wb, p * wa);
            fterm[0] = F[0];
            fterm[1] = dff == 0 ? F[1] : F[2];
            fterm[2] = dff == 0 ? F[2] : F[1];
            fterm[3] = F[3];
        } else if (MORT && !fm_small(fcode_f)) {
            // large side: the high-order mortar fluxes (LATE: in phase 3), then the
            // sparse low-order pairs of this node with the staged traces
            if (PAIRS && !LATE) {
                mortar_ho(0, onb);
                mortar_ho(1, us1);
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
                for (int v = 0; v < 4; ++v) us.u[v] = sPe[v * PP + MB + ff * 2 * n + col];
                make_node<Rc>(us, g);
                double Gf[4];
                llf_face(dff, lowf, own, us, Gf);
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
                    for (int j = 0; j < n; ++j) acc += tb.If[hh][fk][j] * (float)sPe[v * PP + ff * n + j];
                    ui.u[v] = acc;
                } else {
                    double acc = 0.0;
#pragma unroll
                    for (int j = 0; j < n; ++j) acc += tb.I[hh][fk][j] * sPe[v * PP + ff * n + j];
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
                for (int v = 0; v < 4; ++v) uj.u[v] = sPe[v * PP + ff * n + j];
                make_node<Rc>(uj, g);
                double Gf[4];
                llf_face(dff, lowf, own, uj, Gf);
                const double W = sgf * wt * hff;  // wt * h_L / 2 with h_L = 2 h
#pragma unroll
                for (int v = 0; v < 4; ++v) lo[v] += W * Gf[v];
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) fterm[v] = lo[v];
            if (PAIRS && act && (fown || fcor)) {
                const int S = fm_mortar(fcode_f);
                double* R = A.slot + (size_t)(S * 3 * n + n + fm_half(fcode_f) * n + fk) * kSlotW;
#pragma unroll
                for (int v = 0; v < 4; ++v) R[4 + v] = ho[v] - lo[v];
            }
        }
    }
    if constexpr (MORT) {  // (every batch of the mortar launch holds a mortar element)
        __syncthreads();
        // ---- phase 3: high-order mortar fluxes of the large sides in place of this
        // lane's staged small traces (which every lane has read), then their
        // projection ----
        // (updated in place: lanes that repeat another's face node stay out)
        const bool large = PAIRS && tid < NT && (fown || fcor) && fcode_f >= 0 && !fm_small(fcode_f);
        if (large) {
            if constexpr (LATE) {
#pragma unroll 1
                for (int hh = 0; hh < 2; ++hh) {
                    double* const tr = &sPe[MB + (ff * 2 + hh) * n + fk];
                    double F[4];
#pragma unroll
                    for (int v = 0; v < 4; ++v) F[v] = tr[v * PP];
                    mortar_ho(hh, F);
#pragma unroll
                    for (int v = 0; v < 4; ++v) tr[v * PP] = F[v];
                }
            } else {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    sPe[v * PP + MB + (ff * 2 + 0) * n + fk] = onb[v];
                    sPe[v * PP + MB + (ff * 2 + 1) * n + fk] = us1[v];
                }
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
                            accf += tb.Pf[hh][fk][l] * (float)sPe[v * PP + MB + (ff * 2 + hh) * n + l];
                    acc = accf;
                } else {
#pragma unroll
                    for (int hh = 0; hh < 2; ++hh)
#pragma unroll
                        for (int l = 0; l < n; ++l)
                            acc += tb.P[hh][fk][l] * sPe[v * PP + MB + (ff * 2 + hh) * n + l];
                }
                ho[v] = sgf * sTw[0][fk] * hff * 0.5 * acc;
            }
            double* R = A.slot + (size_t)(S * 3 * n + fk) * kSlotW;
            if (act)
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
    //
    // The high-order flux through the subcell face after position pos of a line
    // is the sum of the line's pair fluxes (l, k) with l <= pos < k.  Each thread
    // holds pairs of its own node (the pair map), so it keeps its share of the
    // face it owns in registers (Hown) and only publishes what others need:
    //  N = 4, s1(a) = (a, a + 1) and s2(a) = (a, a + 2) modulo 5: the faces sum
    //    0: s1(0) + s2(0) + s2(3) + s1(4)
    //    1: s1(1) + s2(1) + s2(0) + s2(3) + s1(4) + s2(4)
    //    2: s1(2) + s2(2) + s2(1) + s2(3) + s1(4) + s2(4)
    //    3: s1(3) + s2(2) + s1(4) + s2(4)
    //    so entry a of the line takes s2(a), entry 4 s1(4) + s2(4), and s1(4) has
    //    one of its own;
    //  N = 3: 0: (01) + (03) + (02), 1: (12) + (03) + (02) + (13), 2: (23) + (03) + (13);
    //    (03), (02) and (13) are published.
    // The pair values carry Sbar only, the density's half of it (the line's
    // factor w h is applied to the faces' sums, twice for the density).
    // A node needs no logarithms: smooth pairs, and most pairs beside a shock, take
    // a series or polynomial of their own, and only a round with a pair of states
    // further apart than a factor of 1.41 the logarithms of its pairs' ratios.
    double Hown[2][4];
    const double last_a = a == N ? 1.0 : 0.0, last_b = b == N ? 1.0 : 0.0;  // (N = 4)
    const double in_a = a < 3 ? 1.0 : 0.0, in_b = b < 3 ? 1.0 : 0.0;
    {
#pragma unroll
        for (int i = 0; i < (PAIRS ? N : 0); ++i) {
            const unsigned c = pcode[i / 2] >> (16 * (i % 2));
            const int qo = (int)(c & 31);  // the partner's node
            const int d = N == 4 ? i / 2 : i < 2 ? i : (int)((c >> 10) & 1);
            const int rn = 1 + d, rt = 2 - d;
            const double hS = (&sS[0][0])[(c >> 5) & 31];  // Sbar / 2
            double f[4];  // density, normal and tangential momentum, energy
            const double Ln = sRe[(rn) * NN + q], Lt = sRe[(rt) * NN + q];
            const double Rn = sRe[(rn) * NN + qo], Rt = sRe[(rt) * NN + qo];
            if (!MIXED) {
                const double L0 = sRe[(0) * NN + q], L3 = sRe[(3) * NN + q], L6 = sRe[(6) * NN + q];
                const double R0 = sRe[(0) * NN + qo], R3 = sRe[(3) * NN + qo], R6 = sRe[(6) * NN + qo];
                const double s0 = L0 + R0, d0 = L0 - R0, s6 = L6 + R6, d6 = L6 - R6;
                // one reciprocal for both sums (rho^2 / p, their product's size, within the
                // range of Rcp3::rcp; NaN beyond); the round takes the shortest form that
                // serves all its lanes
                const double r = Rc::rcp(s0 * s6), r6 = s0 * r;
                const double f0 = d0 * (s6 * r), f6 = d6 * r6;
                const double z0 = f0 * f0, z6 = f6 * f6, zm = fmax(z0, z6);
                double hl, iz;  // rho^ln / 2 and 1 / z^ln
                if (__all(zm < kLnSeries)) {
                    hl = half_lnmean_series(s0, z0);
                    iz = inv_lnmean_series(r6, z6);
                } else {
                    hl = half_lnmean_poly(s0, z0);
                    iz = inv_lnmean_poly(r6, z6);
                    if (!__all(zm < kLnPoly)) {
                        double l0, l6;
                        flog2(L0 * Rc::rcp(R0), L6 * Rc::rcp(R6), l0, l6);
                        if (!(z0 < kLnPoly)) hl = 0.5 * d0 * Rc::rcp(l0);
                        if (!(z6 < kLnPoly)) iz = l6 * Rc::rcp(d6);
                        if (__any(zm != zm)) {  // a reciprocal for each sum
                            const double q6 = Rc::rcp(s6), g0 = d0 * Rc::rcp(s0), g6 = d6 * q6;
                            if (g0 * g0 < kLnPoly) hl = half_lnmean_poly(s0, g0 * g0);
                            if (g6 * g6 < kLnPoly) iz = inv_lnmean_poly(q6, g6 * g6);
                        }
                    }
                }
                const double sn = Ln + Rn, st = Lt + Rt;
                const double h = hS * (hl * sn);  // Sbar rho^ln {{vn}} / 2
                const double ig2 = 2.0 * ig1;
                if (A.vflux == DGIDP_FLUX_CHANDRASHEKAR) {
                    // Chandrashekar: beta = z / 2, so p~ = rho-bar / (2 beta-bar) =
                    // (rho_L + rho_R) / (z_L + z_R) and 1 / (2 beta^ln) = 1 / z^ln
                    const double fn = fma(h, sn, 2.0 * hS * (s0 * Rc::rcp(s6))), ft = h * st;
                    const double k2 = Ln * Ln + Lt * Lt + Rn * Rn + Rt * Rt;
                    f[1] = fn;
                    f[2] = ft;
                    f[3] = fma(h, fma(ig2, iz, -0.5 * k2), 0.5 * fma(sn, fn, st * ft));
                } else {
                    const double kin = fma(Lt, Rt, Ln * Rn);
                    f[1] = fma(h, sn, hS * (L3 + R3));
                    f[2] = h * st;
                    f[3] = fma(h, fma(ig2, iz, kin), hS * fma(R3, Ln, L3 * Rn));
                }
                f[0] = h;
            } else {
                const double scale = 2.0 * hS;
                const F2 L5 = unpack2(sRe[(5) * NN + q]), L6 = unpack2(sRe[(6) * NN + q]);
                const F2 R5 = unpack2(sRe[(5) * NN + qo]), R6 = unpack2(sRe[(6) * NN + qo]);
                const float L7 = unpack2(sRe[(7) * NN + q]).x, R7 = unpack2(sRe[(7) * NN + qo]).x;
                const float rL = L5.x, rR = R5.x, zL = L6.y, zR = R6.y;
                const float iz_ln = inv_lnmeanf(zL, zR, L7, R7);
                const float pL = L5.y, pR = R5.y;
                const float vnL = (float)Ln, vnR = (float)Rn, vtL = (float)Lt, vtR = (float)Rt;
                const float vna = 0.5f * (vnL + vnR), vta = 0.5f * (vtL + vtR);
                const float fr = lnmeanf(rL, rR, L6.x, R6.x) * vna;
                // (sums of products in the order of the positions along the line, so that
                // the single precision result does not depend on who holds the pair; the
                // other terms do not change with the order)
                const bool own = (c >> 11) & 1;
                const float vn0 = own ? vnR : vnL, vn1 = own ? vnL : vnR;
                float fn, ft, f3;
                if (A.vflux == DGIDP_FLUX_CHANDRASHEKAR) {
                    const float vt0 = own ? vtR : vtL, vt1 = own ? vtL : vtR;
                    const float pt = (rL + rR) / (zL + zR);
                    fn = fr * vna + pt;
                    ft = fr * vta;
                    f3 = fr * ((float)ig1 * iz_ln - 0.25f * (vn0 * vn0 + vt0 * vt0 + vn1 * vn1 + vt1 * vt1)) +
                         vna * fn + vta * ft;
                } else {
                    const float p0 = own ? pR : pL, p1 = own ? pL : pR;
                    fn = fr * vna + 0.5f * (pL + pR);
                    ft = fr * vta;
                    f3 = fr * (0.5f * (vnL * vnR + vtL * vtR) + (float)ig1 * iz_ln) + 0.5f * (p0 * vn1 + p1 * vn0);
                }
                f[0] = hS * fr;
                f[1] = scale * fn;
                f[2] = scale * ft;
                f[3] = scale * f3;
            }
            const int vi[4] = {0, rn, rt, 3};  // rows of the four components
            if constexpr (N == 4) {
                const int line = 2 * NN + d * n + (d == 0 ? b : a);
                const double last = d == 0 ? last_a : last_b, in = d == 0 ? in_a : in_b;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (i % 2 == 0) {
                        Hown[d][vi[j]] = f[j];
                        if (last != 0.0) sPe[vi[j] * PP + line] = f[j];
                    } else {
                        sPe[vi[j] * PP + d * NN + q] = fma(last, Hown[d][vi[j]], f[j]);
                        Hown[d][vi[j]] = fma(in, f[j], Hown[d][vi[j]]);
                    }
                }
            } else {
                // entries of a direction: (03), (02) and (13) of the four lines
                if (i < 2) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        Hown[i][vi[j]] = f[j];
                        if (i == 0 ? a == N : b == N) sPe[vi[j] * PP + 3 * n * i + (i == 0 ? b : a)] = f[j];
                    }
                } else {
                    const int at = d * 3 * n + n + n * ((d == 0 ? a : b) & 1) + (d == 0 ? b : a);
#pragma unroll
                    for (int j = 0; j < 4; ++j) sPe[vi[j] * PP + at] = f[j];
                }
            }
        }
    }
    if constexpr (PAIRS) __syncthreads();
    // ---- phase 5b: low-order subcell fluxes of the faces owned by this node,
    // x (a|a+1) and y (b|b+1), times the line's weight: w_b h_y / 2 and w_a h_x / 2.
    // With F = (f_L + f_R) / 2 - lambda (u_R - u_L) / 2 and f = u v_n + pressure terms,
    // four instructions per variable; equal states still leave the dissipation
    // exactly zero ----
    // (a node on the upper element boundary owns no face in that direction: it
    // takes itself as the neighbour with weight 0)
    const double whx = a < N ? 0.5 * hy * sTw[0][b] : 0.0, why = b < N ? 0.5 * hx * sTw[0][a] : 0.0;
    double FVo[2][4];
    {
        NodeP me;
        LDS_NODE(me, q);
#pragma unroll
        for (int d = 0; d < 2; ++d) {
            const int qo = d == 0 ? (a < N ? q + 1 : q) : (b < N ? q + n : q);
            NodeP o;
            LDS_NODE(o, qo);
            const double hw = 0.5 * (d == 0 ? whx : why);
            const double va = d == 0 ? me.v1 : me.v2, vb = d == 0 ? o.v1 : o.v2;
            const double hl = hw * fmax(fabs(va) + me.c, fabs(vb) + o.c);
            const double wa = hw * va, wb = hw * vb;
#pragma unroll
            for (int v = 0; v < 4; ++v)
                FVo[d][v] = fma(-hl, o.u[v] - me.u[v], fma(o.u[v], wb, me.u[v] * wa));
            FVo[d][1 + d] = fma(hw, me.p + o.p, FVo[d][1 + d]);
            FVo[d][3] += fma(o.p, wb, me.p * wa);
        }
    }
    // the node's low-order residual so far: its surface term and the faces it owns
    double RLO[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) RLO[v] = (fown ? fterm[v] : 0.0) - FVo[0][v] - FVo[1][v];
    // the owner of a subcell face forms its antidiffusive flux w (f^HO - f^FV),
    // keeps both fluxes (ADo, FVo) and leaves them for the face's other node:
    // the low-order one in the freed primitive rows, the antidiffusive one in
    // the pair buffer
    const double hasl = a > 0 ? 1.0 : 0.0, hasb = b > 0 ? 1.0 : 0.0;
    double ADo[2][4];
#pragma unroll
    for (int d = 0; d < (PAIRS ? 2 : 0); ++d) {
        const double wh = d == 0 ? whx : why;
        const int pos = d == 0 ? a : b, line = d == 0 ? b : a;
        const double has = d == 0 ? hasl : hasb;
        if constexpr (N == 4) {
            // s2 of the node before (from position 1 on), s2(3) (up to face 2), and
            // s1(4) + s2(4), at face 0 s1(4) alone
            const int e0i = d * NN + (d == 0 ? line * n : line), st = d == 0 ? 1 : n;
            const int i1 = d * NN + (pos > 0 ? q - st : q), i2 = e0i + 3 * st;
            const int i3 = pos > 0 ? e0i + N * st : 2 * NN + d * n + line;
            const double in = d == 0 ? in_a : in_b;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const double H = fma(has, sPe[v * PP + i1], fma(in, sPe[v * PP + i2], Hown[d][v] + sPe[v * PP + i3]));
                ADo[d][v] = fma(v == 0 ? 2.0 * wh : wh, H, -FVo[d][v]);
            }
        } else {
            const double low = pos < 2 ? 1.0 : 0.0;
            const int e0i = d * 3 * n + line;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const double H = fma(has, sPe[v * PP + e0i + 2 * n],
                                     fma(low, sPe[v * PP + e0i + n], Hown[d][v] + sPe[v * PP + e0i]));
                ADo[d][v] = fma(v == 0 ? 2.0 * wh : wh, H, -FVo[d][v]);
            }
        }
    }
    // every read of the primitives and of the pair fluxes is done
    __syncthreads();
#pragma unroll
    for (int d = 0; d < 2; ++d)
        if (d == 0 ? a < N : b < N) {
            const int fi = d == 0 ? q - b : q;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                if (PAIRS) sPe[v * PP + d * NN + q] = ADo[d][v];
                sRe[(d * 4 + v) * NFH + fi] = FVo[d][v];
            }
        }
    // the y faces' surface terms at the element's corners, in the x entries that
    // hold no face (a = N)
    if (fcor) {
        const int cs = N + n * ((fk ? 1 : 0) + (ff & 1 ? 2 : 0));
#pragma unroll
        for (int v = 0; v < 4; ++v) sPe[v * PP + cs] = fterm[v];
    }
    __syncthreads();

    // ---- phase 6: low-order residual, bounds, node factors ----
    // u^n of this node for the SSP combination, loaded where it is needed (so
    // that it occupies no registers through the flux phases)
    double un4[4] = {0, 0, 0, 0};
    if (MODE == MODE_STAGE && !LATE && A.a != 0.0) load_u<N>(A.un, e, q, un4);
    if (LATE) load_u<N>(A.uin, e, q, u0);
    const bool onf[4] = {a == 0, a == N, b == 0, b == N};
    // the subcell faces to the left of and below the node, read at a clamped
    // in-range position of its own line; a missing face (on the element
    // boundary) has weight 0 (hasl, hasb)
    double ADl[4], ADb[4], dS0[4], dS1[4];
    int slot0 = -1, slot1 = -1, nmf = 0;
    const double im = 4.0 * Rc::rcp(hx * hy) * sTw[1][a] * sTw[1][b];  // 1 / m_i
    {
        const int hl = a > 0 ? q - 1 : q, hb = NN + (b > 0 ? q - n : q);
        const int fl = a > 0 ? q - b - 1 : b * N, fb = b > 0 ? q - n : q;
        // at the corners the y face's surface term from its slot
        const double cor = (onf[0] || onf[1]) && (onf[2] || onf[3]) ? 1.0 : 0.0;
        const int cs = N + n * ((2 * a > N ? 1 : 0) + (2 * b > N ? 2 : 0));
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            if (PAIRS) {
                ADl[v] = sPe[v * PP + hl];
                ADb[v] = sPe[v * PP + hb];
            }
            const double Fl = sRe[v * NFH + fl], Fb = sRe[(4 + v) * NFH + fb];
            RLO[v] = fma(cor, sPe[v * PP + cs], fma(hasb, Fb, fma(hasl, Fl, RLO[v])));
        }
        if constexpr (MORT && PAIRS) {
            // a node lies on at most one x face (a = 0 or N) and one y face (b = 0 or
            // N): slot 0 takes the mortar of its x face, slot 1 that of its y face
            const int cx = onf[0] ? fcode[0] : (onf[1] ? fcode[1] : -1);
            const int cy = onf[2] ? fcode[2] : (onf[3] ? fcode[3] : -1);
            auto slot_of = [&](int code, int k) {
                const int S3 = fm_mortar(code) * 3 * n;
                return fm_small(code) ? S3 + n + fm_half(code) * n + k : S3 + k;
            };
            if (cx >= 0) slot0 = slot_of(cx, b);
            if (cy >= 0) slot1 = slot_of(cy, a);
            if (!LATE && slot0 >= 0)
#pragma unroll
                for (int v = 0; v < 4; ++v) dS0[v] = A.slot[(size_t)slot0 * kSlotW + 4 + v];
            if (!LATE && slot1 >= 0)
#pragma unroll
                for (int v = 0; v < 4; ++v) dS1[v] = A.slot[(size_t)slot1 * kSlotW + 4 + v];
            nmf = (cx >= 0) + (cy >= 0);
        }
    }
    if (MODE == MODE_RHS_LOW || MODE == MODE_RHS_HIGH) {
        if (act) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                double r = RLO[v];
                if (MODE == MODE_RHS_HIGH) {
                    r += fma(hasl, ADl[v], -ADo[0][v]) + fma(hasb, ADb[v], -ADo[1][v]);
                    const double* dS = A.slot + 4 + v;
                    r += (slot0 >= 0 ? dS[(size_t)slot0 * kSlotW] : 0.0) + (slot1 >= 0 ? dS[(size_t)slot1 * kSlotW] : 0.0);
                }
                A.uout[((unsigned)e * 4u + v) * NN + q] = r * im;
            }
        }
        return;
    }

    const double dtm = dt * im;
    double uFV[4], cf[4][4];
    double rmin = 0.0, pmin = 0.0, th = 1.0;
    unsigned long long inad = 0;
    {
#pragma unroll
        for (int v = 0; v < 4; ++v) uFV[v] = u0[v] + dtm * RLO[v];
        const double pFV = pressure<Rc>(uFV, g);
        if (act && (!(uFV[0] > 0.0) || !(pFV > 0.0))) inad = 1;
        rmin = A.beta * uFV[0];
        pmin = A.beta * pFV;
        // the faces' increments dt / m_i w (f^HO - f^FV) (left, right, below,
        // above), signed (zero for missing faces)
        const double dl = dtm * hasl, db = dtm * hasb;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            cf[0][v] = dl * ADl[v];
            cf[1][v] = -dtm * ADo[0][v];
            cf[2][v] = db * ADb[v];
            cf[3][v] = -dtm * ADo[1][v];
        }
        if (A.limiter != DGIDP_LIMIT_NONE) th = volume_factor(uFV, cf, rmin, pmin, ig1);
    }
    if (LATE && A.a != 0.0) load_u<N>(A.un, e, q, un4);
    sT[q] = th;
    __syncthreads();

    // ---- phase 7: limited volume update, SSP combination, mortar slots ----
    double asum = 0.0, thmin = 1.0;
    unsigned long long viol = 0;
    if (act) {
        double uvol[4];
        double tf[4];
        // face factor: the smaller of its two node factors
        // (a missing face reads the node itself; its increment is zero)
        const int qn4[4] = {a > 0 ? q - 1 : q, a < N ? q + 1 : q, b > 0 ? q - n : q, b < N ? q + n : q};
#pragma unroll
        for (int j = 0; j < 4; ++j) tf[j] = fmin(th, sT[qn4[j]]);
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
            if (A.limiter != DGIDP_LIMIT_NONE) {
                // p(uvol) >= pmin as 2 rho (E - pmin / (gamma - 1)) >= |m|^2 (rho >= rmin > 0)
                const double gp = 2.0 * uvol[0] * (uvol[3] - pmin * ig1) - (uvol[1] * uvol[1] + uvol[2] * uvol[2]);
                if (!(uvol[0] >= rmin) || !(gp >= 0.0)) viol = 1;
            }
        } else {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int slot = j == 0 ? slot0 : slot1;
                if (slot < 0) continue;
                double* S = A.slot + (size_t)slot * kSlotW;
                double c[4], dc[4];
                bool fin = true;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    c[v] = dtm * (LATE ? S[4 + v] : j == 0 ? dS0[v] : dS1[v]);  // (high-order minus low-order flux terms, phases 2 and 3)
                    dc[v] = nmf * c[v];
                    fin = fin && isfinite(dc[v]);
                }
                double ts = 1.0;
                // an undefined high-order mortar flux keeps the low-order flux
                if (A.limiter != DGIDP_LIMIT_NONE) ts = fin ? mortar_factor(uvol, dc, rmin, pmin, ig1) : 0.0;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    S[v] = uvol[v];
                    S[4 + v] = c[v];
                }
                S[8] = ts;
                S[9] = rmin;
                S[10] = pmin;
            }
        }
    }
    if (A.st) push_stats(A.st, inad, viol, thmin, asum, false);
}

// ---------------------------------------------------------------------------
// kernels of a row or column of nodes per lane (large meshes' time step, sensors): every
// wave works alone on 64 / (N+1) elements
// ---------------------------------------------------------------------------
template <int N>
struct RowGeo {
    static constexpr int n = N + 1, NN = n * n;
    static constexpr int WE = 64 / n;                     // elements per wave: 16 at N = 3, 12 at N = 4
    static constexpr int L = WE * n;                      // lanes with a row or column
    static constexpr int PER = (WE * NN + 63) / 64;       // nodes per lane when loading
    // LDS strides: rows 5 doubles apart and elements 20 (N = 3) or 25 apart: the 16
    // lanes of an access differ modulo 16 (but for two pairs at N = 4 by columns)
    static constexpr int RS = 5, ES = RS * n;
    static constexpr int kWaves = 4;                      // per block
};

// orders the LDS accesses of one wave (which the hardware keeps in order) for the
// compiler; no wave waits for another
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The same maximum on a large mesh, by waves of 64 / (N+1) elements: the nodes' wave
// speeds once per node, then one row of nodes per lane with the element's x faces at its
// ends, then one column with the y faces.  Bound: memory; besides the 32 B per node the
// face nodes' gathers, whose lines hold some five times the element's own bytes, so
// the wave speeds across a face of one of the block's 64 or 48 consecutive elements
// (of some 85% of the faces) come from LDS.  On 246,736 elements of N = 4 (198 MB) one
// thread per node takes 63.4 us, rows without the shared faces 59.9, this 44.8.
template <int N>
__global__ __launch_bounds__(256) void k_dt_rows(DtArgs A)
{
    using G = RowGeo<N>;
    constexpr int n = G::n, NN = G::NN;
    __shared__ double sL[G::kWaves][2][G::WE * G::ES];
    __shared__ double sM[G::kWaves][2][64];  // wave speeds across a mortar, by position
    __shared__ double sWt[n][2 * n];          // mortar weights, read per lane
    __shared__ double sRed[G::kWaves];
    const Tab<N>& tb = T<N>();
    const double g = A.gamma;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    // (contiguous element ranges per XCD from their ends, as in k_dt; elements past the
    // last repeat it)
    const int eb = xcd_batch_rev(blockIdx.x, gridDim.x) * (G::kWaves * G::WE), e0 = eb + wv * G::WE;
    const int t = min(lane, G::L - 1), el = t / n, k = t - el * n;
    const int e = min(e0 + el, A.E - 1);
    const bool idp = A.mode != DGIDP_DT_LOWORDER;
    double* const lx = sL[wv][0];
    double* const ly = sL[wv][1];
    if (threadIdx.x < 2 * NN) (&sWt[0][0])[threadIdx.x] = (&tb.Wt[0][0])[threadIdx.x];
    const double hx = A.h[2 * e], hy = A.h[2 * e + 1], wk = tb.w[k];
    int code[4] = {-1, -1, -1, -1}, nb[4] = {0, 0, 0, 0};
    double fu[4][4];  // the states across the faces at position k, or the boundary node's own
    if (idp) {
        __builtin_memcpy(code, __builtin_assume_aligned(A.fmort + 4 * (size_t)e, 16), 16);
        __builtin_memcpy(nb, __builtin_assume_aligned(A.fnbr + 4 * (size_t)e, 16), 16);
#pragma unroll
        for (int f = 0; f < 4; ++f) {
            nb[f] -= eb;
            if (code[f] != -1 || (unsigned)nb[f] >= (unsigned)(G::kWaves * G::WE))
                load_u<N>(A.u, code[f] < -1 ? e : nb[f] + eb, face_q<N>(code[f] < -1 ? f : f ^ 1, k), fu[f]);
        }
    }
#pragma unroll
    for (int i = 0; i < G::PER; ++i) {
        const int j = lane + 64 * i, ej = j / NN, q = j - ej * NN;
        NodeP o;
        load_node<N, Rc>(A.u, min(e0 + ej, A.E - 1), q, o, g);
        if (G::WE * NN % 64 == 0 || i + 1 < G::PER || ej < G::WE) {
            const int at = ej * G::ES + (q / n) * G::RS + q % n;
            lx[at] = wave_speed(o, 0);
            ly[at] = wave_speed(o, 1);
        }
    }
    // wave speeds across the faces at position k: of an element of another block from its
    // state, of one of this block from LDS
    // (lo2: of the second small element of a large side)
    double lo[4] = {0.0, 0.0, 0.0, 0.0}, lo2[4] = {0.0, 0.0, 0.0, 0.0};
    auto inside = [&](int f) { return code[f] == -1 && (unsigned)nb[f] < (unsigned)(G::kWaves * G::WE); };
    if (idp) {
#pragma unroll
        for (int f = 0; f < 4; ++f) {
            if (inside(f)) continue;
            NodeP o;
#pragma unroll
            for (int v = 0; v < 4; ++v) o.u[v] = fu[f][v];
            make_node<Rc>(o, g);
            if (code[f] < -1) {  // boundary: the ghost state of the face node
                const int j = (-2 - code[f]) * n + k;
                double x[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) x[v] = A.bext[(size_t)j * 4 + v];
                NodeP b;
                boundary_ghost(A.bkind[j], x, o, f, g, b.u);
                make_node<Rc>(b, g);
                o = b;
            }
            lo[f] = wave_speed(o, f >> 1);
        }
        auto large = [&](int f) { return code[f] >= 0 && !fm_small(code[f]); };
        if (large(0) || large(1) || large(2) || large(3)) {
            // (the state's registers are free again: all four faces' loads first)
#pragma unroll
            for (int f = 0; f < 4; ++f)
                if (large(f)) load_u<N>(A.u, A.fnbr2[e * 4 + f], face_q<N>(f ^ 1, k), fu[f]);
#pragma unroll
            for (int f = 0; f < 4; ++f) {
                if (!large(f)) continue;
                NodeP o;
#pragma unroll
                for (int v = 0; v < 4; ++v) o.u[v] = fu[f][v];
                make_node<Rc>(o, g);
                lo2[f] = wave_speed(o, f >> 1);
            }
        }
        __syncthreads();
#pragma unroll
        for (int f = 0; f < 4; ++f) {
            if (!inside(f)) continue;
            const int w = nb[f] / G::WE, q = face_q<N>(f ^ 1, k);
            lo[f] = sL[w][f >> 1][(nb[f] - w * G::WE) * G::ES + (q / n) * G::RS + q % n];
        }
    }
    __syncthreads();  // the rows are summed in place
    // edges across face f at position k: 2 |c_ij| lambda_ij, lm the wave speed of this side
    auto face = [&](int f, double lm) {
        const double hf = f < 2 ? hy : hx;
        double sum = 0.5 * wk * hf * fmax(lm, lo[f]);
        if (__any(code[f] >= 0)) {
            // mortar: the wave speeds of the other side by position (large side:
            // of both small elements; small side: of the large one)
            sM[wv][0][lane] = lo[f];
            sM[wv][1][lane] = lo2[f];
            wave_sync();
            if (code[f] >= 0) {
                const bool small = fm_small(code[f]);
                sum = 0.0;
#pragma unroll
                for (int hh = 0; hh < 2; ++hh) {
                    if (small && hh != fm_half(code[f])) continue;
#pragma unroll
                    for (int l = 0; l < n; ++l) {
                        const double wt = small ? 2.0 * sWt[l][hh * n + k] : sWt[k][hh * n + l];
                        if (wt == 0.0) continue;
                        sum += 2.0 * wt * hf * 0.25 * fmax(lm, sM[wv][small ? 0 : hh][el * n + l]);
                    }
                }
            }
            wave_sync();
        }
        return sum;
    };
    double y[n], s = 0.0;
    if (idp) {
        // edges along x carry 2 |c| = w_b h_y / 2, along y w_a h_x / 2
        double* row = lx + t * G::RS;
#pragma unroll
        for (int i = 0; i < n; ++i) y[i] = row[i];
        double prev = face(0, y[0]);
        const double last = face(1, y[N]), cx = 0.5 * wk * hy;
#pragma unroll
        for (int i = 0; i < n; ++i) {
            const double next = i < N ? cx * fmax(y[i], y[i + 1 < n ? i + 1 : N]) : last;
            row[i] = prev + next;
            prev = next;
        }
        wave_sync();
    }
    const double* colx = lx + el * G::ES + k;
    const double* coly = ly + el * G::ES + k;
#pragma unroll
    for (int j = 0; j < n; ++j) y[j] = coly[j * G::RS];
    if (idp) {
        double prev = face(2, y[0]);
        const double last = face(3, y[N]), cy = 0.5 * wk * hx;
#pragma unroll
        for (int j = 0; j < n; ++j) {
            const double next = j < N ? cy * fmax(y[j], y[j + 1 < n ? j + 1 : N]) : last;
            s = fmax(s, (colx[j * G::RS] + (prev + next)) * tb.winv[j]);
            prev = next;
        }
        s *= 4.0 * Rc::rcp(hx * hy) * tb.winv[k];
    } else {
#pragma unroll
        for (int j = 0; j < n; ++j)
            s = fmax(s, (N + 1) * (colx[j * G::RS] * Rc::rcp(hx) + y[j] * Rc::rcp(hy)));
    }
    s = wave_max(s);
    if (lane == 0) sRed[wv] = s;
    __syncthreads();
    dt_merge<G::kWaves>(A, sRed);
}

// ---------------------------------------------------------------------------
// modal sensors: the indicators (k_indicator), the features and the learned
// indicator (k_features).  All start from the squared orthonormal-Legendre
// coefficients of a nodal quantity q[b'][a'], in two sum-factorised passes:
//   r[b'][i] = sum_a' Vinv[i][a'] q[b'][a'],   m[j][i] = sum_b' Vinv[j][b'] r[b'][i]
//  Hennemann indicator: energy = max of the energy fractions of the highest and
//  the second-highest mode shells, alpha = logistic with threshold
//  T = 0.5 10^(-1.8 (N+1)^(1/4)) and sharpness ln(9999), zero below 1e-3, on rho p,
//  capped at 0.5 (FP32, external element order).
//  Features: x- and y-shell energy fractions of rho and of p for the shells
//  N-3 .. N (16 values; FP32, external order).
//
// Every wave works alone on 64 / (N+1) elements: it loads their nodes in order
// (all loads first), then takes one row of nodes per lane for the first pass and one
// column for the second, in place in LDS, so the matrix rows are scalar operands
// and a pass takes n reads and n^2 products for n modes; the reductions run
// over columns and rows in the same way, and no lane waits for another wave.
// Bound: memory (32 B per node read; what the last-level cache still holds of the state
// comes faster than the 5.2 TB/s of a large copy).  On 246,736 elements of N = 4 (198 MB),
// the form with one lane per mode, block barriers and one lane per element for the
// whole reduction against this one: modal indicator 51 -> 30 us, features 50 -> 33,
// learned indicator 62 -> 43.
// ---------------------------------------------------------------------------
// density and pressure of the wave's nodes lane + 64 i of elements e0 .. e0 + WE - 1
// (elements past the last repeat it)
template <int N>
__device__ __forceinline__ void modal_load(const double* __restrict__ u, int e0, int E, double gamma, int lane,
                                           double (&r)[RowGeo<N>::PER], double (&p)[RowGeo<N>::PER])
{
    using G = RowGeo<N>;
    double w[G::PER][4];
#pragma unroll
    for (int i = 0; i < G::PER; ++i) {
        const int k = lane + 64 * i, el = k / G::NN, q = k - el * G::NN;
        const double* pu = u + ((size_t)min(e0 + el, E - 1) * 4 * G::NN + q);
#pragma unroll
        for (int v = 0; v < 4; ++v) w[i][v] = pu[v * G::NN];
    }
#pragma unroll
    for (int i = 0; i < G::PER; ++i) {
        r[i] = w[i][0];
        p[i] = (gamma - 1.0) * (w[i][3] - 0.5 * (w[i][1] * w[i][1] + w[i][2] * w[i][2]) / w[i][0]);
    }
}

// Squared modes m[j] = m2[j][c] of column c of element t / n, where lane t < L is
// (element, c); x holds the nodal values in modal_load's order, Q is the wave's
// WE * ES doubles.  Q's column c of the element may be overwritten by its lane
// afterwards.
template <int N>
__device__ __forceinline__ void modal_modes(const Tab<N>& tb, double* Q, const double (&x)[RowGeo<N>::PER],
                                            int lane, int t, double (&m)[N + 1])
{
    using G = RowGeo<N>;
    constexpr int n = G::n;
#pragma unroll
    for (int i = 0; i < G::PER; ++i) {
        const int k = lane + 64 * i, el = k / G::NN, q = k - el * G::NN;
        if (G::WE * G::NN % 64 == 0 || i + 1 < G::PER || el < G::WE)
            Q[el * G::ES + (q / n) * G::RS + q % n] = x[i];
    }
    wave_sync();
    double y[n];
    double* row = Q + t * G::RS;  // (ES = RS n: the rows of all elements are RS apart)
#pragma unroll
    for (int k = 0; k < n; ++k) y[k] = row[k];
#pragma unroll
    for (int i = 0; i < n; ++i) {
        double s = 0.0;
#pragma unroll
        for (int k = 0; k < n; ++k) s += tb.Vinv[i][k] * y[k];
        row[i] = s;
    }
    wave_sync();
    const double* col = Q + (t / n) * G::ES + t % n;
#pragma unroll
    for (int k = 0; k < n; ++k) y[k] = col[k * G::RS];
#pragma unroll
    for (int j = 0; j < n; ++j) {
        double s = 0.0;
#pragma unroll
        for (int k = 0; k < n; ++k) s += tb.Vinv[j][k] * y[k];
        m[j] = s * s;
    }
}

template <int N>
__global__ __launch_bounds__(256) void k_indicator(const double* __restrict__ u, int E,
                                                   const int* __restrict__ perm, double gamma, double thresh,
                                                   double sharp, float* __restrict__ alpha)
{
    using G = RowGeo<N>;
    constexpr int n = G::n;
    __shared__ double sQ[G::kWaves][G::WE * G::ES];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int e0 = (blockIdx.x * G::kWaves + wv) * G::WE;
    if (e0 >= E) return;
    double* Q = sQ[wv];
    double r[G::PER], p[G::PER], m[n];
    modal_load<N>(u, e0, E, gamma, lane, r, p);
#pragma unroll
    for (int i = 0; i < G::PER; ++i) p[i] *= r[i];
    const int t = min(lane, G::L - 1), c = t % n;
    modal_modes<N>(T<N>(), Q, p, lane, t, m);
    // this column's part of the highest shell, the second-highest and the rest
    double s = 0.0;
#pragma unroll
    for (int j = 0; j < N - 1; ++j) s += m[j];
    double* col = Q + (t / n) * G::ES + c;
    col[0] = c == N ? s + m[N - 1] + m[N] : m[N];
    col[G::RS] = c == N ? 0.0 : c == N - 1 ? s + m[N - 1] : m[N - 1];
    col[2 * G::RS] = c < N - 1 ? s : 0.0;
    wave_sync();
    if (lane >= G::WE || e0 + lane >= E) return;
    double top1 = 0.0, top2 = 0.0, low2 = 0.0;
#pragma unroll
    for (int i = 0; i < n; ++i) {
        top1 += Q[lane * G::ES + i];
        top2 += Q[lane * G::ES + G::RS + i];
        low2 += Q[lane * G::ES + 2 * G::RS + i];
    }
    const double low1 = low2 + top2, en = fmax(top1 / (low1 + top1), top2 / low1);
    const double al = 1.0 / (1.0 + exp(-(sharp / thresh) * (en - thresh)));
    alpha[perm[e0 + lane]] = al < 1e-3 ? 0.0f : (float)fmin(al, 0.5);
}

template <int N>
static void launch_modal(int E, const double* u, const int* perm, double gamma, float* alpha, hipStream_t s)
{
    using G = RowGeo<N>;
    const double thresh = 0.5 * std::pow(10.0, -1.8 * std::pow((double)(N + 1), 0.25));
    const double sharp = std::log((1.0 - 1e-4) / 1e-4);
    hipLaunchKernelGGL(k_indicator<N>, dim3((E - 1) / (G::kWaves * G::WE) + 1), dim3(256), 0, s, u, E,
                       perm, gamma, thresh, sharp, alpha);
}

// NET = false writes the features, one group of elements per wave.  NET = true
// keeps those of NT groups (32 elements at N = 3, 24 at N = 4) in LDS and runs the
// network on them (the matrix-core pass of mlp::forward32: features rounded to FP32,
// then to BF16; the weights are staged in LDS once per block).
template <int N, bool NET>
__global__ __launch_bounds__(256) void k_features(const double* __restrict__ u, int E,
                                                  const int* __restrict__ perm, double gamma,
                                                  const uint16_t* __restrict__ wb, float* __restrict__ out)
{
    using G = RowGeo<N>;
    constexpr int n = G::n, NT = NET ? 2 : 1;
    static_assert(NT * G::WE <= 32 && N >= 3, "one network pass per wave; shells N-3 .. N");
    static_assert(G::WE * 16 % 64 == 0, "whole waves of features");
    __shared__ double sQ[G::kWaves][G::WE * G::ES];
    __shared__ double sS[G::kWaves][2][2][G::L];  // shell sums: quantity, direction
    __shared__ __align__(16) float sX[NET ? G::kWaves : 1][32][mlp::kNin + 4];
    __shared__ __align__(16) mlp::LdsWeights sW[1];  // not allocated when NET is false (unused)
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int tile0 = (blockIdx.x * G::kWaves + wv) * NT * G::WE;
    if (NET) {
        mlp::stage_weights(sW[0], wb, threadIdx.x, 256);
        __syncthreads();
    }
    double* Q = sQ[wv];
    const int t = min(lane, G::L - 1);
#pragma unroll 1
    for (int g = 0; g < NT; ++g) {
        const int e0 = tile0 + g * G::WE;
        if (e0 >= E) break;
        double x[2][G::PER];
        modal_load<N>(u, e0, E, gamma, lane, x[0], x[1]);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            double m[n], s = 0.0;
            modal_modes<N>(T<N>(), Q, x[k], lane, t, m);
            double* col = Q + (t / n) * G::ES + t % n;
#pragma unroll
            for (int j = 0; j < n; ++j) {
                s += m[j];
                col[j * G::RS] = m[j];
            }
            sS[wv][k][0][t] = s;
            wave_sync();
            s = 0.0;
#pragma unroll
            for (int i = 0; i < n; ++i) s += Q[t * G::RS + i];
            sS[wv][k][1][t] = s;
            wave_sync();
        }
        // feature f of an element: quantity f / 8 (rho, p), direction (f / 4) % 2
        // (x shells: sums over the y modes, y shells: over the x modes), shell N - 3 + f % 4
        const int f = lane & 15;
#pragma unroll
        for (int i = 0; i < G::WE / 4; ++i) {
            const int el = (lane >> 4) + 4 * i;
            const double* S = &sS[wv][f >> 3][0][el * n];
            double all = 0.0;
#pragma unroll
            for (int j = 0; j < n; ++j) all += S[j];
            const float v = (float)(sS[wv][f >> 3][(f >> 2) & 1][el * n + N - 3 + (f & 3)] / all);
            if (NET) sX[wv][g * G::WE + el][f] = v;
            else if (e0 + el < E) out[(size_t)perm[e0 + el] * 16 + f] = v;
        }
        wave_sync();
    }
    if (!NET || tile0 >= E) return;
    const int c = lane & 31, hf = lane >> 5;
    const bool ok = c < NT * G::WE && tile0 + c < E;
    float xv[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) xv[j] = ok ? sX[wv][c][hf * 8 + j] : 0.0f;
    const float y = mlp::forward32(sW[0], mlp::pack_bf16x8(xv), lane);
    if (hf == 0 && ok) out[perm[tile0 + c]] = y;
}

template <int N, bool NET>
static void launch_features(int E, const double* u, const int* perm, double gamma, const uint16_t* wb, float* out,
                            hipStream_t s)
{
    constexpr int per = RowGeo<N>::kWaves * RowGeo<N>::WE * (NET ? 2 : 1);
    hipLaunchKernelGGL((k_features<N, NET>), dim3((E - 1) / per + 1), dim3(256), 0, s, u, E, perm, gamma, wb, out);
}

int launch_indicator(int N, int E, const double* u, const int* perm, double gamma, float* alpha,
                     float* feat, hipStream_t s)
{
    if (E <= 0) return 0;
    if (N != 3 && N != 4) return -1;
    if (alpha) {
        if (N == 3) launch_modal<3>(E, u, perm, gamma, alpha, s);
        else launch_modal<4>(E, u, perm, gamma, alpha, s);
    }
    if (feat) {
        if (N == 3) launch_features<3, false>(E, u, perm, gamma, nullptr, feat, s);
        else launch_features<4, false>(E, u, perm, gamma, nullptr, feat, s);
    }
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_learned_indicator(int N, int E, const double* u, const int* perm, double gamma, const uint16_t* wb,
                             float* alpha, hipStream_t s)
{
    if (E <= 0) return 0;
    if (N == 3) launch_features<3, true>(E, u, perm, gamma, wb, alpha, s);
    else if (N == 4) launch_features<4, true>(E, u, perm, gamma, wb, alpha, s);
    else return -1;
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// ---------------------------------------------------------------------------
// solution transfer between meshes (Sec. 2.4): one thread per new node.
// Children take the parent polynomial at their nodes (tensor product of the
// mortar interpolation matrices); a new parent takes the exact L2 projection
// of its four children (tensor product of the mortar projections, summed).
// ---------------------------------------------------------------------------
template <int N>
__global__ __launch_bounds__(256) void k_transfer(int E, const int* __restrict__ tkind,
                                                  const int* __restrict__ tsrc,
                                                  const double* __restrict__ uold,
                                                  double* __restrict__ unew)
{
    constexpr int n = N + 1, NN = n * n;
    const Tab<N>& tb = T<N>();
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= E * NN) return;
    const int e = i / NN, q = i - e * NN, a = q % n, b = q / n;
    const int kind = tkind[e];
    double out[4] = {0, 0, 0, 0};
    if (kind == 0) {
#pragma unroll
        for (int v = 0; v < 4; ++v) out[v] = uold[((size_t)tsrc[4 * e] * 4 + v) * NN + q];
    } else if (kind == 1) {
        const int p = tsrc[4 * e], c = tsrc[4 * e + 1], cx = c & 1, cy = c >> 1;
        const double* up = uold + (size_t)p * 4 * NN;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            double acc = 0.0;
#pragma unroll
            for (int l = 0; l < n; ++l) {
                double row = 0.0;
#pragma unroll
                for (int k = 0; k < n; ++k) row += tb.I[cx][a][k] * up[(v * n + l) * n + k];
                acc += tb.I[cy][b][l] * row;
            }
            out[v] = acc;
        }
    } else {
        for (int c = 0; c < 4; ++c) {
            const int cx = c & 1, cy = c >> 1;
            const double* uc = uold + (size_t)tsrc[4 * e + c] * 4 * NN;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                double acc = 0.0;
#pragma unroll
                for (int l = 0; l < n; ++l) {
                    double row = 0.0;
#pragma unroll
                    for (int k = 0; k < n; ++k) row += tb.P[cx][a][k] * uc[(v * n + l) * n + k];
                    acc += tb.P[cy][b][l] * row;
                }
                out[v] += acc;
            }
        }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) unew[((size_t)e * 4 + v) * NN + q] = out[v];
}

// Zhang-Shu scaling toward the reference mean (Sec. 2.4): one wave per group
// (the four children of a refined element, or one new parent).  A troubled
// group (a node with rho < eps or p < eps) is scaled by the largest theta that
// lifts every node to rho, p >= eps (aimed at eps (1 + 2^-40)); one theta per
// group keeps the group's mass.  counts[0] limited groups, counts[1] groups
// whose mean is itself below the thresholds (theta = 0).
// every node of the group scaled by t toward ub has rho >= eps and p >= eps
// (a wave-wide answer; every lane of the wave calls it)
template <int N>
__device__ bool zs_group_ok(const double* __restrict__ unew, const int* R, int cnt, int lane,
                            const double* ub, double t, double eps, double gamma)
{
    constexpr int NN = (N + 1) * (N + 1);
    int bad = 0;
    for (int j = lane; j < cnt * NN; j += 64) {
        const double* ue = unew + (size_t)R[2 + j / NN] * 4 * NN;
        const int q = j % NN;
        double w[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) w[v] = ub[v] + t * (ue[v * NN + q] - ub[v]);
        const double p = (gamma - 1.0) * (w[3] - 0.5 * (w[1] * w[1] + w[2] * w[2]) / w[0]);
        if (!(w[0] >= eps) || !(p >= eps)) bad = 1;
    }
    return !__any(bad);
}

template <int N>
__global__ __launch_bounds__(256) void k_zhang_shu(int G, const int* __restrict__ grp,
                                                   const double* __restrict__ uold,
                                                   double* __restrict__ unew, double eps,
                                                   double gamma, unsigned long long* counts)
{
    constexpr int n = N + 1, NN = n * n;
    const Tab<N>& tb = T<N>();
    const int lane = threadIdx.x & 63;
    const int g = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (g >= G) return;  // whole waves leave together
    const int* R = grp + 6 * g;
    const int kind = R[0];
    const int cnt = kind == 1 ? 4 : 1;
    const double ig1 = 1.0 / (gamma - 1.0);
    // reference mean: the old parent (refinement) or the projected parent
    const double* ref = kind == 1 ? uold + (size_t)R[1] * 4 * NN : unew + (size_t)R[2] * 4 * NN;
    double ub[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        double s = 0.0;
        for (int q = lane; q < NN; q += 64) s += tb.w[q % n] * tb.w[q / n] * ref[v * NN + q];
        ub[v] = wave_sum(s) * 0.25;
    }
    int trouble = 0;
    double em = 0.0;  // largest |E| of the group: the rounding scale of its pressures
    for (int j = lane; j < cnt * NN; j += 64) {
        const double* ue = unew + (size_t)R[2 + j / NN] * 4 * NN;
        const int q = j % NN;
        double w[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) w[v] = ue[v * NN + q];
        const double p = (gamma - 1.0) * (w[3] - 0.5 * (w[1] * w[1] + w[2] * w[2]) / w[0]);
        if (!(w[0] >= eps) || !(p >= eps)) trouble = 1;
        em = fmax(em, fabs(w[3]));
    }
    const double emax = wave_max(em);
    if (!__any(trouble)) return;
    // density aimed at eps (1 + 2^-40); pressure in addition 2^-40 max|E| above,
    // since p = (gamma-1)(E - |m|^2/(2 rho)) is known only to a few ulps of E
    const double et = eps * kMargin;
    const double pt = et + 0x1p-40 * emax;
    const double pb = (gamma - 1.0) * (ub[3] - 0.5 * (ub[1] * ub[1] + ub[2] * ub[2]) / ub[0]);
    const bool fixable = ub[0] > et && pb > pt;
    double theta = 0.0;
    if (fixable) {
        double t = 1.0;
        for (int j = lane; j < cnt * NN; j += 64) {
            const double* ue = unew + (size_t)R[2 + j / NN] * 4 * NN;
            const int q = j % NN;
            double d[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) d[v] = ue[v * NN + q] - ub[v];
            double ti = 1.0;
            if (ub[0] + d[0] < et) ti = (ub[0] - et) / (-d[0]);
            ti = fmin(ti, theta_p(ub, d, pt, ig1));
            t = fmin(t, ti);
        }
        theta = wave_min(t);
        // the quadratic's coefficients cancel at the scale rho_bar E_bar and p
        // divides that rounding by rho: where a node's density gets small the
        // factor can miss, so the scaled states are checked directly and, if
        // one fails, the factor is bisected between 0 (the mean) and theta
        if (!zs_group_ok<N>(unew, R, cnt, lane, ub, theta, eps, gamma)) {
            double lo = 0.0, hi = theta;
#pragma unroll 1
            for (int it = 0; it < 60; ++it) {
                const double mid = 0.5 * (lo + hi);
                if (zs_group_ok<N>(unew, R, cnt, lane, ub, mid, eps, gamma)) lo = mid;
                else hi = mid;
            }
            theta = lo;
        }
    }
    for (int j = lane; j < cnt * NN; j += 64) {
        double* ue = unew + (size_t)R[2 + j / NN] * 4 * NN;
        const int q = j % NN;
#pragma unroll
        for (int v = 0; v < 4; ++v) ue[v * NN + q] = ub[v] + theta * (ue[v * NN + q] - ub[v]);
    }
    if (lane == 0) {
        atomicAdd(&counts[0], 1ull);
        if (!fixable) atomicAdd(&counts[1], 1ull);
    }
}

int launch_transfer(int N, int E_new, const int* tkind, const int* tsrc, const double* uold,
                    double* unew, hipStream_t s)
{
    const int NN = (N + 1) * (N + 1);
    const int grid = (E_new * NN + 255) / 256;
    if (E_new <= 0) return 0;
    if (N == 3) hipLaunchKernelGGL(k_transfer<3>, dim3(grid), dim3(256), 0, s, E_new, tkind, tsrc, uold, unew);
    else if (N == 4) hipLaunchKernelGGL(k_transfer<4>, dim3(grid), dim3(256), 0, s, E_new, tkind, tsrc, uold, unew);
    else return -1;
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_zhang_shu(int N, int G, const int* zgrp, const double* uold, double* unew, double eps,
                     double gamma, unsigned long long* counts, hipStream_t s)
{
    if (G <= 0) return 0;
    const int grid = (G + 3) / 4;  // four waves (groups) per block
    if (N == 3)
        hipLaunchKernelGGL(k_zhang_shu<3>, dim3(grid), dim3(256), 0, s, G, zgrp, uold, unew, eps, gamma, counts);
    else if (N == 4)
        hipLaunchKernelGGL(k_zhang_shu<4>, dim3(grid), dim3(256), 0, s, G, zgrp, uold, unew, eps, gamma, counts);
    else
        return -1;
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// ---------------------------------------------------------------------------
// small utility kernels
// ---------------------------------------------------------------------------
// Elements between the external and the internal order, kPermVec values of type V per
// thread, a block's stride apart, all loads first; V is 16 bytes wide where src and
// dst are 16-byte aligned (an element's values are a multiple of that).  Bound: HBM; with
// one double per thread and 64-bit divisions 395 MB took 95 us (4.2 TB/s), now 60.
constexpr int kPermVec = 4;
template <int N, typename V>
__global__ __launch_bounds__(256) void k_permute(unsigned total, const int* __restrict__ perm,
                                                 const V* __restrict__ src, V* __restrict__ dst, int to_int)
{
    constexpr unsigned per = 4 * (N + 1) * (N + 1) * sizeof(double) / sizeof(V);
    const unsigned i0 = blockIdx.x * (256 * kPermVec) + threadIdx.x;
    V x[kPermVec];
    unsigned to[kPermVec];
#pragma unroll
    for (int k = 0; k < kPermVec; ++k) {
        const unsigned i = min(i0 + 256 * k, total - 1), e = i / per;
        const unsigned j = (unsigned)perm[e] * per + (i - e * per);
        to[k] = to_int ? i : j;
        x[k] = src[to_int ? j : i];
    }
#pragma unroll
    for (int k = 0; k < kPermVec; ++k)
        if (i0 + 256 * k < total) dst[to[k]] = x[k];
}

__global__ void k_set_double(double* p, double v) { *p = v; }

int launch_set_double(double* p, double v, hipStream_t s)
{
    hipLaunchKernelGGL(k_set_double, dim3(1), dim3(1), 0, s, p, v);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

__global__ __launch_bounds__(kStatSpread) void k_stats_reset(DevStats* st)
{
    st += threadIdx.x;
    st->fv_inadmissible = 0;
    st->violations = 0;
    st->theta_vol_min_bits = __double_as_longlong(1.0);
    st->theta_mort_min_bits = __double_as_longlong(1.0);
    st->alpha_vol_sum = 0.0;
    st->alpha_mort_sum = 0.0;
}

__global__ void k_check_state(int total_nodes, int NN, double g, const double* u, unsigned long long* bad)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= total_nodes) return;
    const int e = i / NN, q = i - e * NN;
    double w[4];
    for (int v = 0; v < 4; ++v) w[v] = u[((size_t)e * 4 + v) * NN + q];
    const double p = (g - 1.0) * (w[3] - 0.5 * (w[1] * w[1] + w[2] * w[2]) / w[0]);
    const bool ok = isfinite(w[0]) && isfinite(w[1]) && isfinite(w[2]) && isfinite(w[3]) &&
                    w[0] > 0.0 && p > 0.0;
    if (!ok) atomicMin(bad, (unsigned long long)i);
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
template <int N>
static int stage_N(const DevMesh& m, const KernelParams& kp, const double* uin, const double* un,
                   double* uout, double a, double b, const DtSource& dt, DevStats* st, int mode,
                   hipStream_t s, bool rev = false, bool mortars = false)
{
    using G = Geo<N>;
    StageArgs A;
    set_stage(A, m, kp, uin, un, uout, a, b, dt, st);
    A.blist = m.blist;
    const int nb = (m.E + G::EPB - 1) / G::EPB;
    const bool mixed = kp.precision == DGIDP_MIXED;
    // A large mesh: the batches with a mortar element
    // (the first m.nbm entries of the batch list) in one launch, the others in
    // a second one without mortar code, in which the first launch's mortars are
    // corrected.  The first ends with a partly idle GPU, so a mesh of fewer than
    // kSplitMin batches, or with a larger mortar share, runs as one launch of the
    // mortar variant: five steps of the 22,156-leaf blast (5,539 batches, N = 3) take
    // 348 us in one launch and 478 in two, of the 246,736-leaf quadrants (49,348,
    // N = 4) 3,851 and 3,748.  A mesh without mortars runs the conforming variant alone.
    constexpr int kSplitMin = 16384;
    const bool split = m.nbm == 0 || (nb >= kSplitMin && 8LL * m.nbm <= nb);
    const bool two = split && m.nbm > 0;
    // dt from the accumulators: in a stage of two launches the first reduces them
    // per wave, stores dt, and the second reads it.  In one launch over a large mesh
    // k_dt_final reduces them once.
    if (dt.dtmax && dt.dt_out && !two && nb >= kFinalMin) {
        hipLaunchKernelGGL(k_dt_final, dim3(1), dim3(64), 0, s, dt.dtmax, dt.cfl, dt.dt_out, st);
        A.dt = dt.dt_out;
        A.dtmax = nullptr;
    }
    // the mortar corrections of this stage
    A.mo = {m.slot, m.slot_node, m.slot_partner, mortars ? m.M : 0, uout, b, kp.gamma, kp.limiter, st};
    A.mblocks = 0;
    auto go = [&](auto modec, auto mixc) {
        constexpr int MD = decltype(modec)::value;
        constexpr bool MX = decltype(mixc)::value;
        if (!split) {
            A.blist = nullptr;  // element batches in mesh order
            A.boff = 0;
            hipLaunchKernelGGL((k_stage<N, MD, MX, true>), dim3(nb), dim3(G::BS), 0, s, A);
            return;
        }
        A.blist = m.nbm > 0 ? m.blist : nullptr;
        if (m.nbm > 0) {
            A.boff = 0;
            hipLaunchKernelGGL((k_stage<N, MD, MX, true>), dim3(m.nbm), dim3(G::BS), 0, s, A);
            if (A.dtmax) {
                A.dt = dt.dt_out;
                A.dtmax = nullptr;
            }
            // whole rounds over the XCDs, so that the batch ranges keep their XCD
            A.mblocks = ((A.mo.M * 3 * (N + 1) + G::BS - 1) / G::BS + 7) / 8 * 8;
        }
        if (nb > m.nbm) {
            // (only this launch may walk its ranges backwards: its blocks cost
            // alike, where the mortar launch and an unsplit stage start the
            // costlier mortar batches first on purpose)
            A.boff = m.nbm;
            A.rev = rev ? 1 : 0;
            hipLaunchKernelGGL((k_stage<N, MD, MX, false>), dim3(A.mblocks + nb - m.nbm), dim3(G::BS), 0, s, A);
        }
    };
    using BT = std::true_type;
    using BF = std::false_type;
    if (mode == MODE_STAGE) {
        using MS = std::integral_constant<int, MODE_STAGE>;
        if (mixed) go(MS(), BT());
        else go(MS(), BF());
    } else if (mode == MODE_RHS_HIGH) {
        using MH = std::integral_constant<int, MODE_RHS_HIGH>;
        if (mixed) go(MH(), BT());
        else go(MH(), BF());
    } else {
        go(std::integral_constant<int, MODE_RHS_LOW>(), BF());
    }
    if (hipGetLastError() != hipSuccess) return -1;
    return A.mo.M > 0 && !two ? run_mortar<Rc, false>(N, A.mo, s) : 0;
}

int launch_stage(int N, const DevMesh& m, const KernelParams& kp, const double* uin,
                 const double* un, double* uout, double a, double b, const DtSource& dt,
                 DevStats* st, hipStream_t s, bool rev, bool mortars)
{
    if (m.E == 0) return 0;
    if (local_bounds(kp)) {
        if (local::launch_stage(N, m, kp, uin, un, uout, a, b, dt, st, s, rev)) return -1;
        return mortars ? launch_mortar(N, m, kp, uout, b, st, s) : 0;
    }
    if (N == 3) return stage_N<3>(m, kp, uin, un, uout, a, b, dt, st, MODE_STAGE, s, rev, mortars);
    if (N == 4) return stage_N<4>(m, kp, uin, un, uout, a, b, dt, st, MODE_STAGE, s, rev, mortars);
    return -1;
}

int launch_rhs(int N, const DevMesh& m, const KernelParams& kp, const double* u, int which,
               double* du, hipStream_t s)
{
    if (m.E == 0) return 0;
    const int mode = which == DGIDP_RHS_HIGH ? MODE_RHS_HIGH : MODE_RHS_LOW;
    const DtSource none;
    if (N == 3) return stage_N<3>(m, kp, u, nullptr, du, 0.0, 1.0, none, nullptr, mode, s);
    if (N == 4) return stage_N<4>(m, kp, u, nullptr, du, 0.0, 1.0, none, nullptr, mode, s);
    return -1;
}

int launch_mortar(int N, const DevMesh& m, const KernelParams& kp, double* uout, double b, DevStats* st, hipStream_t s)
{
    if (m.M == 0) return 0;
    if (local_bounds(kp)) return local::launch_mortar(N, m, kp, uout, b, st, s);
    return run_mortar<Rc, false>(N, {m.slot, m.slot_node, m.slot_partner, m.M, uout, b, kp.gamma, kp.limiter, st}, s);
}

int launch_dt(int N, const DevMesh& m, const KernelParams& kp, const double* u, int mode,
              unsigned long long* acc, unsigned long long* other, hipStream_t s)
{
    if (local_bounds(kp)) return local::launch_dt(N, m, kp, u, mode, acc, other, s);
    const DtArgs A = dt_args(m, kp, u, mode, acc, other);
    // rows and columns per lane from kRowsMin elements on: its chain is longer, and
    // below, fewer waves than fill the chip are left.  Of a blast with one refined
    // level, one thread per node against rows: N = 3, 19,864 elements 6.9 and 8.6 us,
    // 31,012 8.2 and 8.8, 44,688 9.8 and 9.7, 60,856 12.8 and 11.6; N = 4, 31,012 11.2 and
    // 11.7, 44,688 14.9 and 13.5, 79,420 21.6 and 18.9.
    constexpr int kRowsMin = 40960;
    if (m.E < kRowsMin) return run_dt<Rc>(N, A, s);
    if (N == 3) hipLaunchKernelGGL(k_dt_rows<3>, dim3((m.E - 1) / (4 * RowGeo<3>::WE) + 1), dim3(256), 0, s, A);
    else if (N == 4) hipLaunchKernelGGL(k_dt_rows<4>, dim3((m.E - 1) / (4 * RowGeo<4>::WE) + 1), dim3(256), 0, s, A);
    else return -1;
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_permute(int N, int E, const int* perm, const double* src, double* dst, int to_internal,
                   hipStream_t s)
{
    if (E <= 0) return 0;
    if (N != 3 && N != 4) return -1;
    const bool wide = ((uintptr_t)src | (uintptr_t)dst) % sizeof(double2) == 0;
    // (below 2^30 values, the mesh limit)
    const unsigned total = (unsigned)E * 4u * (unsigned)((N + 1) * (N + 1)) / (wide ? 2 : 1);
    const dim3 grid((total - 1) / (256 * kPermVec) + 1);
    auto go = [&](auto n, auto v) {
        using V = decltype(v);
        hipLaunchKernelGGL((k_permute<decltype(n)::value, V>), grid, dim3(256), 0, s, total, perm, (const V*)src,
                           (V*)dst, to_internal);
    };
    using N3 = std::integral_constant<int, 3>;
    using N4 = std::integral_constant<int, 4>;
    if (N == 3) wide ? go(N3(), double2()) : go(N3(), double());
    else wide ? go(N4(), double2()) : go(N4(), double());
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_stats_reset(DevStats* st, hipStream_t s)
{
    hipLaunchKernelGGL(k_stats_reset, dim3(1), dim3(kStatSpread), 0, s, st);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_check_state(int N, int E, double gamma, const double* u, unsigned long long* bad,
                       hipStream_t s)
{
    const int NN = (N + 1) * (N + 1);
    const int total = E * NN;
    hipLaunchKernelGGL(k_check_state, dim3((total + 255) / 256), dim3(256), 0, s, total, NN, gamma,
                       u, bad);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace dgidp
