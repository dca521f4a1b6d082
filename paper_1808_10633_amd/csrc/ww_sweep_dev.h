// ww_sweep_dev.h -- device code of the characteristic WENO5 sweep, shared by
// the single-box kernels and the batched persistent kernel.
//
// One thread computes the flux at one interface i+1/2 of the sweep axis
// (arXiv:1808.10633, Sec. 2.1, eq. 1 per characteristic field).  A block
// first stages the cells of its tile (plus the 3-cell halo on each side of
// the sweep axis) in LDS together with the per-cell quantities every
// interface needs (pressure, 1/rho, fast/slow/Alfven speeds), so each cell's
// equation of state and wave speeds are evaluated once per block.
//
// Per interface:
//   1. the six stencil cells i-2..i+3 are read from LDS; their physical
//      fluxes are formed; the mean flux of cells i and i+1 and the five
//      cell-to-cell differences of F and U are taken (eq. 1 is linear in
//      these; the projection rows carry the 1/2 of the Lax-Friedrichs split, a
//      power-of-two scaling), and the largest |lambda^s| per field over the
//      stencil gives the local Lax-Friedrichs speed.  The central term of eq.
//      (1) is (-F_{i-1} + 7F_i + 7F_{i+1} - F_{i+2})/12 = (F_i + F_{i+1})/2
//      + (DF_{i-1/2} - DF_{i+3/2})/12: its first part sums over the fields to
//      itself (R L = I) and is added to the back-projected rest unprojected,
//      its second uses the differences projected for the weights;
//   2. the mean state of cells i and i+1 (arithmetic mean of the primitive
//      variables) gives the seven-wave eigen-system with the Roe-Balsara
//      normalisation; the left eigenvectors are applied as
//      L_U X = L_W (dW/dU) X: the Jacobian dW/dU once per vector, then the
//      sparse primitive rows, after rotating the transverse components onto
//      the (B_t, perpendicular) basis, in which every row has at most four
//      entries and the +- members of a wave pair share their terms;
//   3. per field: split F^{s+-} differences, WENO5 weights (eqs. 3-7, with the
//      three weights put over one common denominator), phi_N (eq. 2), eq. (1);
//   4. back-projection R_U F^s = (dU/dW) R_W F^s, again through the sparse
//      primitive columns; the flux is stored in grid components.
// The sweep axis is a template parameter: no data is transposed.
#pragma once
#include "ww_index.h"
#include "ww_internal.h"
#include "ww_update_dev.h"

#include <math.h>

#include <type_traits>

namespace ww {
namespace sw {

constexpr int NQ = 13;      // staged quantities per cell
// LDS slots: 0 rho, 1 mn, 2 mt1, 3 mt2, 4 Bn, 5 Bt1, 6 Bt2, 7 E,
//            8 p, 9 1/rho, 10 c_f, 11 c_s, 12 c_A   (sweep frame)
// Tiles staged with the cell fluxes (PRE: the FP32 x sweeps) add 13 v_n and
// 14..19 the sweep-frame flux components 1..6 (the mass flux is m_n): every
// cell serves six interfaces, and its flux is then formed once per tile
// instead of once per interface, for 20 quantities of LDS.
constexpr int NQ_PRE = 20;
template <bool PRE> constexpr int nq() { return PRE ? NQ_PRE : NQ; }
constexpr int TILE = 64;    // lanes per row
constexpr int ROWS = 4;     // waves per block
constexpr int NCX = TILE + 5;

// Reciprocal: hardware estimate refined by Newton steps (two in FP64, one in
// FP32), to within rounding of the correctly rounded quotient.
__device__ __forceinline__ double frcp(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    double e = fma(-x, r, 1.0);
    r = fma(r, e, r);
    e = fma(-x, r, 1.0);
    return fma(r, e, r);
}
__device__ __forceinline__ float frcp(float x)
{
    float r = __builtin_amdgcn_rcpf(x);
    float e = fmaf(-x, r, 1.0f);
    return fmaf(r, e, r);
}
// Reciprocal of the nonlinear weights' common denominator.  FP64: one Newton
// step on the estimate, which is good to about 2^-23, leaving a relative error
// near 2^-46 in the weights (about 1e-14), far below the scheme's truncation
// error and the weights' own sensitivity to rounding in the smoothness
// indicators.  FP32: the estimate itself (within 1 ulp).
__device__ __forceinline__ double frcp_w(double x)
{
    const double r = __builtin_amdgcn_rcp(x);
    return fma(r, fma(-x, r, 1.0), r);
}
__device__ __forceinline__ float frcp_w(float x) { return __builtin_amdgcn_rcpf(x); }

// Square root in FP64 for finite x >= 0: the hardware reciprocal-square-root
// estimate, one Goldschmidt step towards g = sqrt(x), h = 1/(2 sqrt(x)), then
// a Newton correction g += (x - g^2) h with the residual formed by a fused
// multiply-add (Markstein's formulation).  With exactly rounded FMAs the
// result is the correctly rounded root for estimate errors up to 2^-22 and
// within 1 ulp up to 2^-14.  The estimate is taken at x + 2^-1022, so x = 0
// gives 0 and x < 0 gives NaN; the wave speeds and normalisations passed here
// are never subnormal or infinite, so the range scaling and special-case
// selects of the general routine are left out.
__device__ __forceinline__ double fsqrt(double x)
{
    const double y = __builtin_amdgcn_rsq(x + 0x1p-1022);
    double g = x * y, h = 0.5 * y;
    const double r = fma(-g, h, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    const double d = fma(-g, g, x);
    return fma(d, h, g);
}
__device__ __forceinline__ float fsqrt(float x) { return sqrtf(x); }

// 1/sqrt(x) in FP64 for finite x > 0: the estimate refined by two Newton
// steps y += y (1 - x y^2) / 2.
__device__ __forceinline__ double frsq(double x)
{
    double y = __builtin_amdgcn_rsq(x);
#pragma unroll
    for (int i = 0; i < 2; ++i) y = fma(0.5 * y, fma(-x * y, y, 1.0), y);
    return y;
}

// Staging runs at a raised wave priority.  Two blocks share a CU, so while
// one block stages its tile (global loads, equation of state, LDS writes) the
// other is usually deep in its interface arithmetic; without the raise the
// older waves of that block win the issue arbitration and the staging block's
// loads and barrier are delayed.  The raise ends after the staging barrier.
constexpr int STAGE_PRIO = 2;
__device__ __forceinline__ void stage_begin() { __builtin_amdgcn_s_setprio(STAGE_PRIO); }
__device__ __forceinline__ void stage_end() { __builtin_amdgcn_s_setprio(0); }

// Square roots of the scales 18 and 12 that fold the linear weights
// d = (1, 6, 3)/10 and the 1/3, 1/6 of eq. (2) into the (epsilon + IS_k).
constexpr double SQ18 = 4.2426406871192851464, SQ12 = 3.4641016151377545870;

// The nonlinear part of phi_N of eq. (2) with the weights of eqs. (3)-(7),
// phi_N + (b - 2c + d)/12 = omega_0 (a-2b+c)/3 + omega_2 (b-2c+d)/6.
// ee = (epsilon/4, sqrt(18) epsilon/4, sqrt(12) epsilon/4).
// With r_0 = sqrt(18) q_0, r_1 = q_1, r_2 = sqrt(12) q_2 (q_k = (epsilon +
// IS_k)/4, as in phi_n) and R_k = r_k^2: A = R_1 R_2, B = R_0 R_1, C = R_0 R_2
// are 12, 6 and 36 times the common-denominator numerators of alpha_0,
// alpha_2, alpha_1, so omega_0 = 3A / S and omega_2 = 6B / S with
// S = 3A + 6B + C, and the result is (A (a-2b+c) + B (b-2c+d)) / S (one
// reciprocal, no separate scaling of the differences), returned as num / S.
template <typename T>
__device__ __forceinline__ void phi_fold(T a, T b, T c, T d, const T (&ee)[3], T &num, T &inv)
{
#pragma clang fp contract(off)
    const T b2 = b * b, c2 = c * c;
    T r0 = fma(a, fma(T(4 * SQ18), a, T(-11 * SQ18) * b), fma(T(10 * SQ18), b2, ee[1]));
    T r1 = fma(T(4), b2 + c2, fma(T(-5), b * c, ee[0]));
    T r2 = fma(d, fma(T(4 * SQ12), d, T(-11 * SQ12) * c), fma(T(10 * SQ12), c2, ee[2]));
    if constexpr (sizeof(T) == 4) {
        // FP32: keep the products of the squares in range (see phi_n)
        const T s = __builtin_amdgcn_rcpf(fmax(r0, fmax(r1, r2)));
        r0 *= s; r1 *= s; r2 *= s;
    }
    r0 *= r0; r1 *= r1; r2 *= r2;
    const T A = r1 * r2, B = r0 * r1;
    inv = frcp_w(fma(T(3), A, fma(T(6), B, r0 * r2)));
    const T y = fma(T(-2), c, b) + d;
    num = fma(A, fma(T(-2), b, a) + c, B * y);
}

// phi_N of eq. (2) for the variants:
// WZ: the WENO-Z weights of Borges et al. (2008) instead (exponent 1, an
// ablation): alpha_k = d_k (1 + tau5 / (eps + IS_k)), tau5 = |IS_0 - IS_2|.
// LBL: also the largest deviation of a weight from the linear weights.
template <typename T, bool LBL, bool WZ>
__device__ __forceinline__ T phi_n(T a, T b, T c, T d, const T (&ee)[3], T *dev)
{
    const T e4 = ee[0];
    // Smoothness indicators of eqs. (5)-(7), expanded into the quadratic forms
    // IS_0 = 16a^2 - 44ab + 40b^2, IS_1 = 16b^2 - 20bc + 16c^2,
    // IS_2 = 40c^2 - 44cd + 16d^2 (all positive definite), and divided by 4
    // together with epsilon: the weights depend only on ratios of the
    // (epsilon + IS_k), so they are unchanged (an exact power-of-two scale).
    T b2 = b * b, c2 = c * c;
    T q0 = fma(a, fma(T(4), a, T(-11) * b), fma(T(10), b2, e4));
    T q1 = fma(T(4), b2 + c2, fma(T(-5), b * c, e4));
    T q2 = fma(d, fma(T(4), d, T(-11) * c), fma(T(10), c2, e4));
    if constexpr (sizeof(T) == 4) {
        // FP32: the products of four (epsilon + IS)/4 below overflow once IS
        // passes ~5e9 (strong blasts); scaled by (about) their largest they
        // stay in (0, 1], and the weights, which depend only on ratios, are
        // unchanged, so the hardware reciprocal estimate serves as the scale
        const T s = __builtin_amdgcn_rcpf(fmax(q0, fmax(q1, q2)));
        q0 *= s; q1 *= s; q2 *= s;
    }
    T n0, n1, n2;
    if constexpr (WZ) {
        // alpha_k = d_k (q_k + t) / q_k with t = |q_0 - q_2| (= tau5 / 4),
        // over the common denominator q0 q1 q2
        const T t = fabs(q0 - q2);
        n0 = (q0 + t) * q1 * q2;
        n1 = T(6) * (q1 + t) * q0 * q2;
        n2 = T(3) * (q2 + t) * q0 * q1;
    } else {
        q0 *= q0; q1 *= q1; q2 *= q2;
        // alpha_k = d_k / q_k with d = (1, 6, 3); omega_k = alpha_k / sum alpha,
        // written over the common denominator q0 q1 q2 (one reciprocal).
        n0 = q1 * q2; n1 = T(6) * q0 * q2; n2 = T(3) * q0 * q1;
    }
    T inv = frcp(n0 + n1 + n2);
    if constexpr (LBL) {
        // largest deviation of (omega_0, omega_1, omega_2) from (0.1, 0.6, 0.3)
        T w0 = n0 * inv, w1 = n1 * inv, w2 = n2 * inv;
        T dv = fmax(fmax(fabs(w0 - T(0.1)), fabs(w1 - T(0.6))), fabs(w2 - T(0.3)));
        *dev = fmax(*dev, dv);
    }
    // eq. (2): omega_0 (a-2b+c)/3 + (omega_2 - 1/2)(b-2c+d)/6
    T x3 = (a - T(2) * b + c) * T(1.0 / 3.0);
    T y6 = (b - T(2) * c + d) * T(1.0 / 6.0);
    return fma(inv, fma(n0, x3, n2 * y6), T(-0.5) * y6);
}

// eq. (1) for one field, less the projected mean flux l (F_i + F_{i+1})/2.
// df, du: projected flux and state differences (k = 0..4 at i-3/2 .. i+5/2),
// both already carrying the 1/2 of the Lax-Friedrichs split; al: LF speed.
// The remaining central part (df_1 - df_3)/6 and the linear parts of the two
// phi_N, (dp_1 - 2dp_2 + dp_3)/12 and -(dm_1 - 2dm_2 + dm_3)/12, add up to
// (dp_1 - dp_2 + dm_2 - dm_3)/6.
template <typename T, bool LBL = false, bool WZ = false>
__device__ __forceinline__ T weno_field(const T (&df)[5], const T (&du)[5], T al, const T (&ee)[3], T *dev = nullptr)
{
#pragma clang fp contract(off)
    T dp[5], dm[5];
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        dp[k] = fma(al, du[k], df[k]);
        dm[k] = fma(-al, du[k], df[k]);
    }
    if constexpr (LBL || WZ) {
        return T(1.0 / 6.0) * (df[1] - df[3]) - phi_n<T, LBL, WZ>(dp[0], dp[1], dp[2], dp[3], ee, dev)
                                              + phi_n<T, LBL, WZ>(dm[4], dm[3], dm[2], dm[1], ee, dev);
    } else {
        T np, ip, nm, im;
        phi_fold<T>(dp[0], dp[1], dp[2], dp[3], ee, np, ip);
        phi_fold<T>(dm[4], dm[3], dm[2], dm[1], ee, nm, im);
        const T lin = T(1.0 / 6.0) * ((dp[1] - dp[2]) + (dm[2] - dm[3]));
        return fma(nm, im, fma(-np, ip, lin));
    }
}

// Sweep-frame physical flux of one cell (rho, mn, mt1, mt2, Bt1, Bt2, E
// components) from its conserved variables w, pressure p and 1/rho; returns
// the normal velocity.  The fused operations are written out and nothing else
// is contracted, here and where the fluxes are differenced: the values then
// do not depend on what else a kernel does with them, and kernels that compute
// one flux two ways (fused and separate update) agree bit for bit.
template <typename T>
__device__ __forceinline__ T cell_flux(const T (&w)[8], T p, T ir, T (&F)[7])
{
#pragma clang fp contract(off)
    const T mn = w[1], m1 = w[2], m2 = w[3], bn = w[4], b1 = w[5], b2 = w[6], e = w[7];
    const T vn = mn * ir, v1 = m1 * ir, v2 = m2 * ir;
    const T pt = fma(T(0.5), fma(b2, b2, fma(b1, b1, bn * bn)), p);
    F[0] = mn;
    F[1] = fma(-bn, bn, fma(mn, vn, pt));
    F[2] = fma(m1, vn, -(bn * b1));
    F[3] = fma(m2, vn, -(bn * b2));
    F[4] = fma(vn, b1, -(v1 * bn));
    F[5] = fma(vn, b2, -(v2 * bn));
    F[6] = fma(e + pt, vn, -(bn * fma(v2, b2, fma(v1, b1, vn * bn))));
    return vn;
}

// Stage one cell from its sweep-frame conserved variables w (rho, mn, mt1,
// mt2, Bn, Bt1, Bt2, E): the variables and the derived quantities.  LIN:
// slots 0..10 only (the learned router's routed sweeps: linear fluxes and
// features need no c_s, c_A).
template <typename T, bool PRE = false, bool LIN = false>
__device__ __forceinline__ void stage_values(const T (&w)[8], double gamma, T *q, int qs)
{
#pragma clang fp contract(off)
    const T r = w[0], mn = w[1], m1 = w[2], m2 = w[3], bn = w[4], b1 = w[5], b2 = w[6], e = w[7];
    // pressure recovery (kept in FP64 for every storage type)
    const double ird = frcp((double)r);
    const double mm = fma((double)m2, (double)m2, fma((double)m1, (double)m1, (double)mn * mn));
    const double bb = fma((double)b2, (double)b2, fma((double)b1, (double)b1, (double)bn * bn));
    const double pd = (gamma - 1.0) * fma(-0.5, bb, fma(-0.5 * mm, ird, (double)e));
    T p = (T)pd;
    T ir = (T)ird;
    T a2 = T(gamma) * p * ir;
    T bn2 = bn * bn * ir;
    T bt2 = fma(b1, b1, b2 * b2) * ir;
    T dd = a2 - bn2;
    T disc = fma(dd, dd, bt2 * fma(T(2), a2, fma(T(2), bn2, bt2)));
    T cf2 = T(0.5) * (a2 + bn2 + bt2 + fsqrt(disc));
    T cs2 = a2 * bn2 * frcp(cf2);       // (unused, and not computed, with LIN)
    q[0 * qs] = r;  q[1 * qs] = mn; q[2 * qs] = m1; q[3 * qs] = m2;
    q[4 * qs] = bn; q[5 * qs] = b1; q[6 * qs] = b2; q[7 * qs] = e;
    q[8 * qs] = p;
    q[9 * qs] = ir;
    q[10 * qs] = fsqrt(cf2);
    if constexpr (!LIN) {
        q[11 * qs] = fsqrt(cs2);
        q[12 * qs] = fsqrt(bn2);
    }
    if constexpr (PRE) {
        T F[7];
        const T vn = cell_flux(w, p, ir, F);
        q[13 * qs] = vn;
#pragma unroll
        for (int c = 1; c < 7; ++c) q[(13 + c) * qs] = F[c];
    }
}

// A wave-uniform pointer to device memory, kept in scalar registers: without
// this the compiler reassociates (base + v sv) + lane offset into per-lane
// 64-bit multiplies, two quarter-rate instructions per address.
template <typename T>
using GlobalPtr = T __attribute__((address_space(1))) *;
template <typename T>
__device__ __forceinline__ GlobalPtr<T> uniform(T *p)
{
    GlobalPtr<T> g = (GlobalPtr<T>)p;
    asm volatile("" : "+s"(g));
    return g;
}
// Load, store of the element at a 32-bit byte offset (per lane) from a uniform
// base: the offset is relative to a tile or to an array under 2^32 bytes (2^30
// FP32 elements; a variable of a 1024^3 box is larger).
template <typename T>
__device__ __forceinline__ T ld32(const T *base, uint32_t elem)
{
    return *(GlobalPtr<const T>)((GlobalPtr<const char>)uniform(base) + (uint32_t)(elem * (uint32_t)sizeof(T)));
}
template <typename T>
__device__ __forceinline__ void st32(T *base, uint32_t elem, T x)
{
    *(GlobalPtr<T>)((GlobalPtr<char>)uniform(base) + (uint32_t)(elem * (uint32_t)sizeof(T))) = x;
}
// The same, or (FAR) at a 64-bit offset, for elements anywhere in an array.
template <bool FAR>
using ElemOff = typename std::conditional<FAR, uint64_t, uint32_t>::type;
template <bool FAR, typename T>
__device__ __forceinline__ T ld_off(const T *base, ElemOff<FAR> elem)
{
    if constexpr (FAR) return uniform(base)[elem];
    else return ld32(base, elem);
}
template <bool FAR, typename T>
__device__ __forceinline__ void st_off(T *base, ElemOff<FAR> elem, T x)
{
    if constexpr (FAR) uniform(base)[elem] = x;
    else st32<T>(base, elem, x);
}

// Stage one cell: its variables read from the state (cm: sweep-frame order).
template <typename T, bool PRE = false, bool LIN = false>
__device__ __forceinline__ void stage_cell(const T *__restrict__ u, long id, long sv,
                                           const int (&cm)[8], double gamma, T *q, int qs)
{
    T w[8];
#pragma unroll
    for (int v = 0; v < 8; ++v) w[v] = u[id + cm[v] * sv];
    stage_values<T, PRE, LIN>(w, gamma, q, qs);
}

// Stage cells c = tid, tid + 256, ... (< ncell, at most IT per thread) of a
// tile: every global load of the thread's cells first, then the equation of
// state and LDS stores of each.  A thread's loads are then in flight
// together rather than one cell's latency after another's, which matters at
// two waves per SIMD.  cell_id(c, id) gives the state index of tile cell c,
// false if the cell is not staged; c's LDS slot is sq + c.
template <int IT, bool PRE = false, bool LIN = false, typename T, typename CellId>
__device__ __forceinline__ void stage_tile(const T *__restrict__ u, long sv, const int (&cm)[8], double gamma,
                                           T *sq, int qs, int ncell, CellId cell_id)
{
    const int tid = threadIdx.x + TILE * threadIdx.y;
    T w[IT][8];
    bool ok[IT];
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        const int c = tid + it * TILE * ROWS;
        long id = 0;
        ok[it] = c < ncell && cell_id(c, id);
        if (ok[it]) {
#pragma unroll
            for (int v = 0; v < 8; ++v) w[it][v] = u[id + cm[v] * sv];
        }
    }
#pragma unroll
    for (int it = 0; it < IT; ++it)
        if (ok[it]) stage_values<T, PRE, LIN>(w[it], gamma, sq + tid + it * TILE * ROWS, qs);
}

// Interface flux from six staged cells.  sq: LDS base, qs: stride between
// quantities, off: offset of cell i-2, cstr: stride between cells.
// out: sweep-frame flux (rho, mn, mt1, mt2, Bt1, Bt2, E).
// LBL: also return in *dev the largest deviation of any weight of any field
// from the linear weights (the label of a troubled interface).
// GLF: the LF speed of field s is ag[s] (global speeds of the sweep, an
// ablation) instead of the largest |lambda^s| over the six cells.
// PRE: the cells were staged with their fluxes and v_n (NQ_PRE quantities).
// REREAD: the mean mass flux is read from the tile again at the end instead of
// waiting in registers: with it the FP64 fused x sweep fits 256 VGPRs (without,
// it spills 4; the FP64 y/z tiles fit without and spill 7 with it).
template <typename T, bool LBL = false, bool WZ = false, bool GLF = false, bool PRE = false, bool REREAD = false>
__device__ __forceinline__ void face_flux(const T *__restrict__ sq, int qs, int off, int cstr,
                                          double gamma, double igm1, T eps, T (&out)[7],
                                          T *dev = nullptr, const double *ag = nullptr)
{
    // every fused operation is written out (see cell_flux)
#pragma clang fp contract(off)
#define QQ(q, j) sq[(q) * qs + off + (j) * cstr]
    T Fs[7], dY[5][7], dZ[5][7], am[7];
    T Fp[7], Up[7];
#pragma unroll
    for (int j = 0; j < 6; ++j) {
        T vn, Fj[7];
        const T w[8] = { QQ(0, j), QQ(1, j), QQ(2, j), QQ(3, j), QQ(4, j), QQ(5, j), QQ(6, j), QQ(7, j) };
        if constexpr (PRE) {
            vn = QQ(13, j);
            Fj[0] = w[1];
#pragma unroll
            for (int c = 1; c < 7; ++c) Fj[c] = QQ(13 + c, j);
        } else {
            vn = cell_flux(w, QQ(8, j), QQ(9, j), Fj);
        }
        const T cf = QQ(10, j), cs = QQ(11, j), ca = QQ(12, j);
        const T Uj[7] = { w[0], w[1], w[2], w[3], w[5], w[6], w[7] };
        T lam[7] = { fabs(vn - cf), fabs(vn - ca), fabs(vn - cs), fabs(vn),
                     fabs(vn + cs), fabs(vn + ca), fabs(vn + cf) };
#pragma unroll
        for (int c = 0; c < 7; ++c) {
            am[c] = (j == 0) ? lam[c] : fmax(am[c], lam[c]);
            if (j == 3) Fs[c] = Fp[c] + Fj[c];             // twice the mean flux
            if (j > 0) { dY[j - 1][c] = Fj[c] - Fp[c]; dZ[j - 1][c] = Uj[c] - Up[c]; }
            Fp[c] = Fj[c];
            Up[c] = Uj[c];
        }
    }
    if constexpr (GLF) {
#pragma unroll
        for (int c = 0; c < 7; ++c) am[c] = T(ag[c]);
    }

    // Interface state: mean of the primitive variables of cells i and i+1.
    // Eigen-system normalisation in FP64 for every storage type.
    const double r2 = QQ(0, 2), r3 = QQ(0, 3), i2 = QQ(9, 2), i3 = QQ(9, 3);
    const double rb = 0.5 * (r2 + r3);
    const double vnb = 0.5 * fma((double)QQ(1, 3), i3, (double)QQ(1, 2) * i2);
    const double v1b = 0.5 * fma((double)QQ(2, 3), i3, (double)QQ(2, 2) * i2);
    const double v2b = 0.5 * fma((double)QQ(3, 3), i3, (double)QQ(3, 2) * i2);
    const double bnb = 0.5 * ((double)QQ(4, 2) + (double)QQ(4, 3));
    const double b1b = 0.5 * ((double)QQ(5, 2) + (double)QQ(5, 3));
    const double b2b = 0.5 * ((double)QQ(6, 2) + (double)QQ(6, 3));
    const double pb = 0.5 * ((double)QQ(8, 2) + (double)QQ(8, 3));
    // 1/rho, a and 1/a^2, c_f and 1/c_f^2 from one reciprocal square root
    // each, and c_s = a c_A / c_f with c_A = |B_n| rho^-1/2 (four fewer roots
    // and reciprocals, 1 % of the FP64 y sweep).  The FP64 WENO-Z kernels have
    // no registers left for the longer live ranges of that form; they take
    // each quantity separately.
    constexpr bool LEAN = sizeof(T) == 4 || !WZ;
    double irb, isr = 0.0;
    if constexpr (LEAN) { isr = frsq(rb); irb = isr * isr; }
    else irb = frcp(rb);
    const double a2 = gamma * pb * irb;
    const double bn2 = bnb * bnb * irb;
    const double btt = fma(b1b, b1b, b2b * b2b);
    const double bt2 = btt * irb;
    const double dd = a2 - bn2;
    const double sqD = fsqrt(fma(dd, dd, bt2 * fma(2.0, a2, fma(2.0, bn2, bt2))));
    const double cf2 = 0.5 * (a2 + bn2 + bt2 + sqD);
    double icf2, rcf = 0.0, cs2 = 0.0;
    if constexpr (LEAN) { rcf = frsq(cf2); icf2 = rcf * rcf; }
    else { icf2 = frcp(cf2); cs2 = a2 * bn2 * icf2; }
    double af, as;
    if (sqD <= 1e-12 * (a2 + bn2 + bt2)) {
        af = 1.0; as = 0.0;
    } else {
        // (cf^2 - a^2)(cf^2 - bn^2) = bt^2 cf^2 avoids the cancellation
        double P, Q;
        if (dd >= 0.0) { P = 0.5 * (dd + bt2 + sqD); Q = bt2 * cf2 * frcp(P); }
        else           { Q = 0.5 * (-dd + bt2 + sqD); P = bt2 * cf2 * frcp(Q); }
        const double isq = frcp(sqD);
        const double af2 = fmin(fmax(a2 * P * icf2 * isq, 0.0), 1.0);
        const double as2 = fmin(fmax(Q * isq, 0.0), 1.0);
        af = fsqrt(af2); as = fsqrt(as2);
    }
    double be1, be2;
    if (bt2 > 1e-24 * (a2 + bn2)) {
        const double ibt = frsq(btt);
        be1 = b1b * ibt; be2 = b2b * ibt;
    } else {
        // B_t ~ 0: any unit vector spans the degenerate wave pairs; the first
        // transverse axis keeps the two transverse momenta in separate
        // characteristic fields, so a planar flow (no component or gradient
        // along one transverse axis) stays planar
        be1 = 1.0; be2 = 0.0;
    }
    const double sg = (bnb >= 0.0) ? 1.0 : -1.0;
    double cfm, csm, am_, ia2;
    if constexpr (LEAN) {
        const double ra = frsq(a2);
        am_ = a2 * ra; ia2 = ra * ra;
        cfm = cf2 * rcf; csm = am_ * fabs(bnb) * isr * rcf;
    } else {
        cfm = fsqrt(cf2); csm = fsqrt(cs2); am_ = fsqrt(a2);
        isr = frsq(rb); ia2 = frcp(a2);
    }
    const double sr = rb * isr;
    const double gm1 = gamma - 1.0;
    const double hv2 = 0.5 * fma(v2b, v2b, fma(v1b, v1b, vnb * vnb));

    // rows of L_W, per wave pair: odd (sign-flipping) and even parts, with
    // the 1/2 of the Lax-Friedrichs split folded in (exact power-of-two scale)
    // and the 1/rho and (gamma - 1) of dW/dU: xf below leaves the velocity
    // components rho times and the pressure 1/(gamma - 1) times too large, and
    // every row entry that multiplies them carries the inverse factor
    const double i2a2 = 0.25 * ia2, ir2 = i2a2 * irb, ig2 = i2a2 * gm1 * irb;
    const T kf1 = T(af * cfm * ir2), kf2 = T(as * csm * sg * ir2);
    const T kf4 = T(as * am_ * isr * i2a2), kf6 = T(af * ig2);
    const T ks1 = T(as * csm * ir2), ks2 = T(af * cfm * sg * ir2);
    const T ks4 = T(af * am_ * isr * i2a2), ks6 = T(as * ig2);
    const T ka3 = T(0.25 * sg * irb), ka5 = T(0.25 * isr), ke6 = T(ia2 * gm1), kh = T(0.5);

    // dW/dU at the interface state (without the two scales above) followed by
    // the rotation of the transverse components onto (beta, perpendicular).
    const T tv = T(vnb), t1 = T(v1b), t2 = T(v2b), th = T(hv2);
    const T tb1 = T(b1b), tb2 = T(b2b), e1 = T(be1), e2 = T(be2);
    auto xf = [&](T (&X)[7]) {
        const T w1 = fma(-tv, X[0], X[1]);
        const T w2 = fma(-t1, X[0], X[2]);
        const T w3 = fma(-t2, X[0], X[3]);
        const T w6 = fma(-tb2, X[5], fma(-tb1, X[4], fma(-t2, X[3], fma(-t1, X[2], fma(-tv, X[1], fma(th, X[0], X[6]))))));
        const T pv = fma(e1, w2, e2 * w3), qv = fma(e2, w2, -(e1 * w3));
        const T pB = fma(e1, X[4], e2 * X[5]), qB = fma(e1, X[5], -(e2 * X[4]));
        X[1] = w1; X[2] = pv; X[3] = qv; X[4] = pB; X[5] = qB; X[6] = w6;
    };
#pragma unroll
    for (int k = 0; k < 5; ++k) { xf(dY[k]); xf(dZ[k]); }

    T G[7];
    const T teps = T(0.25) * eps;     // epsilon / 4 for the weights
    const T ee[3] = { teps, teps * T(SQ18), teps * T(SQ12) };

    // One wave pair (sigma = -1 field index lo, sigma = +1 field index hi).
    // proj(X, odd, even) gives the odd and even parts of the row applied to X.
    auto pair = [&](auto proj, int lo, int hi, T &S, T &D) {
        T odf[5], edf[5], odu[5], edu[5];
#pragma unroll
        for (int k = 0; k < 5; ++k) { proj(dY[k], odf[k], edf[k]); proj(dZ[k], odu[k], edu[k]); }
        T df[5], du[5];
#pragma unroll
        for (int k = 0; k < 5; ++k) { df[k] = edf[k] + odf[k]; du[k] = edu[k] + odu[k]; }
        T fplus = weno_field<T, LBL, WZ>(df, du, am[hi], ee, dev);
#pragma unroll
        for (int k = 0; k < 5; ++k) { df[k] = edf[k] - odf[k]; du[k] = edu[k] - odu[k]; }
        T fminus = weno_field<T, LBL, WZ>(df, du, am[lo], ee, dev);
        S = fplus + fminus;
        D = fplus - fminus;
    };

    T S, D;
    // fast pair (fields 0 and 6)
    pair([&](const T (&X)[7], T &o, T &e) { o = fma(kf1, X[1], -(kf2 * X[2])); e = fma(kf4, X[4], kf6 * X[6]); },
         0, 6, S, D);
    {
        const T c0 = T(rb * af), c1 = T(af * cfm), c2 = T(-as * csm * sg), c4 = T(as * sr * am_),
                c6 = T(rb * af * a2);
        G[0] = c0 * S; G[1] = c1 * D; G[2] = c2 * D; G[4] = c4 * S; G[6] = c6 * S;
    }
    // slow pair (fields 2 and 4)
    pair([&](const T (&X)[7], T &o, T &e) { o = fma(ks1, X[1], ks2 * X[2]); e = fma(ks6, X[6], -(ks4 * X[4])); },
         2, 4, S, D);
    {
        const T c0 = T(rb * as), c1 = T(as * csm), c2 = T(af * cfm * sg), c4 = T(-af * sr * am_),
                c6 = T(rb * as * a2);
        G[0] = fma(c0, S, G[0]); G[1] = fma(c1, D, G[1]); G[2] = fma(c2, D, G[2]); G[4] = fma(c4, S, G[4]);
        G[6] = fma(c6, S, G[6]);
    }
    // Alfven pair (fields 1 and 5)
    pair([&](const T (&X)[7], T &o, T &e) { o = ka3 * X[3]; e = ka5 * X[5]; }, 1, 5, S, D);
    G[3] = T(sg) * D;
    G[5] = T(sr) * S;
    // entropy (field 3)
    {
        T df[5], du[5];
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            df[k] = kh * fma(-ke6, dY[k][6], dY[k][0]);
            du[k] = kh * fma(-ke6, dZ[k][6], dZ[k][0]);
        }
        G[0] += weno_field<T, LBL, WZ>(df, du, am[3], ee, dev);
    }

    // back to (vt1, vt2), (Bt1, Bt2) and through dU/dW, onto the mean flux
    const T gv1 = fma(e1, G[2], e2 * G[3]), gv2 = fma(e2, G[2], -(e1 * G[3]));
    const T gb1 = fma(e1, G[4], -(e2 * G[5])), gb2 = fma(e2, G[4], e1 * G[5]);
    const T trb = T(rb);
    if constexpr (REREAD) {
        Fs[0] = *(const volatile T *)&QQ(1, 2) + *(const volatile T *)&QQ(1, 3);
    }
#undef QQ
    out[0] = fma(T(0.5), Fs[0], G[0]);
    out[1] = fma(T(0.5), Fs[1], fma(trb, G[1], tv * G[0]));
    out[2] = fma(T(0.5), Fs[2], fma(trb, gv1, t1 * G[0]));
    out[3] = fma(T(0.5), Fs[3], fma(trb, gv2, t2 * G[0]));
    out[4] = fma(T(0.5), Fs[4], gb1);
    out[5] = fma(T(0.5), Fs[5], gb2);
    const T kin = fma(t2, gv2, fma(t1, gv1, tv * G[1]));
    out[6] = fma(T(0.5), Fs[6], fma(G[6], T(igm1), fma(tb2, gb2, fma(tb1, gb1, fma(trb, kin, th * G[0])))));
}

// Linear fifth-order component-wise flux of the six staged cells (the cheap
// flux of interfaces the learned router calls smooth): one Lax-Friedrichs
// speed alpha = max(|v_n| + c_f) over the stencil for every component and
// the linear-weight form of eq. (1), (2,-13,47,27,-3)/60 on F^+ and the
// mirror (-3,27,47,-13,2)/60 on F^-.  With F^+- = (F +- alpha U)/2 the two
// stencils add up to the sixth-order central combination of F,
// (1,-8,37,37,-8,1)/60, plus alpha times the fifth difference of U,
// (1,-5,10,-10,5,-1)/60: the same flux in 12 operations per component.
template <typename T>
__device__ __forceinline__ void linear_flux(const T *__restrict__ sq, int qs, int off, int cstr,
                                            T (&out)[7])
{
#define QL(q, j) sq[(q) * qs + off + (j) * cstr]
    T F[6][7], U[6][7], al = T(0);
#pragma unroll
    for (int j = 0; j < 6; ++j) {
        T r = QL(0, j), mn = QL(1, j), m1 = QL(2, j), m2 = QL(3, j);
        T bn = QL(4, j), b1 = QL(5, j), b2 = QL(6, j), e = QL(7, j);
        T p = QL(8, j), ir = QL(9, j), cf = QL(10, j);
        T vn = mn * ir, v1 = m1 * ir, v2 = m2 * ir;
        T pt = p + T(0.5) * (bn * bn + b1 * b1 + b2 * b2);
        F[j][0] = mn; F[j][1] = mn * vn + pt - bn * bn; F[j][2] = m1 * vn - bn * b1;
        F[j][3] = m2 * vn - bn * b2; F[j][4] = vn * b1 - v1 * bn; F[j][5] = vn * b2 - v2 * bn;
        F[j][6] = (e + pt) * vn - bn * (vn * bn + v1 * b1 + v2 * b2);
        U[j][0] = r; U[j][1] = mn; U[j][2] = m1; U[j][3] = m2; U[j][4] = b1; U[j][5] = b2; U[j][6] = e;
        al = fmax(al, fabs(vn) + cf);
    }
#undef QL
#pragma unroll
    for (int c = 0; c < 7; ++c) {
        const T cen = fma(T(37), F[2][c] + F[3][c], fma(T(-8), F[1][c] + F[4][c], F[0][c] + F[5][c]));
        const T dis = fma(T(10), U[2][c] - U[3][c], fma(T(-5), U[1][c] - U[4][c], U[0][c] - U[5][c]));
        out[c] = fma(al, dis, cen) * T(1.0 / 60.0);
    }
}

// Store a sweep-frame interface flux in grid components:
// rho, mx, my, mz, B_(N+1), B_(N+2), E.
template <int N, typename T>
__device__ __forceinline__ void store_face(T *__restrict__ flux, const FaceBox &F, const int (&pos)[3],
                                           const T (&out)[7])
{
    constexpr int T1 = (N + 1) % 3, T2 = (N + 2) % 3;
    const long fi = F.idx(pos[0], pos[1], pos[2]);
    flux[0 * F.sc + fi] = out[0];
    flux[(1 + N) * F.sc + fi] = out[1];
    flux[(1 + T1) * F.sc + fi] = out[2];
    flux[(1 + T2) * F.sc + fi] = out[3];
    flux[4 * F.sc + fi] = out[4];
    flux[5 * F.sc + fi] = out[5];
    flux[6 * F.sc + fi] = out[6];
}

// Periodic image of cell index x (-n <= x < 2n) in 0..n-1.  WRAP tiles (the
// batched form's periodic patches) stage each ghost cell from its image
// directly, so the patch needs no ghost fill.
__device__ __forceinline__ int pwrap(int x, int n) { return x < 0 ? x + n : (x >= n ? x - n : x); }

// Cells of an x tile of ROWS rows x TILE faces.
constexpr int XROWS_CELLS = ROWS * NCX;

// One x tile of ROWS rows (transverse (j,k) pairs, tile index ta) x TILE
// consecutive faces (tile index tb), one face per thread.  sq: LDS of
// NQ * XROWS_CELLS elements.  Ends with a block barrier, so consecutive tiles
// may reuse sq.  WRAP: ghost cells from their periodic images, staged with a
// thread's loads first (the batched kernel).
template <typename T, bool WZ = false, bool GLF = false, bool WRAP = false>
__device__ __forceinline__ void sweep_tile_xrows(const T *__restrict__ u, T *__restrict__ flux,
                                                 const Geom &G, const FaceBox &F, const Phys &P,
                                                 int ta, int tb, T *sq)
{
    const int cm[8] = { 0, 1, 2, 3, 4, 5, 6, 7 };
    constexpr int NC = XROWS_CELLS;
    const int lane = threadIdx.x, w = threadIdx.y, tid = lane + TILE * w;
    const int nlast = G.n[0] + 2;   // last cell index along the sweep axis
    const int nrows = F.cnt[1] * F.cnt[2];
    const int r0 = ta * ROWS, f0 = tb * TILE;
    stage_begin();
    auto cell_id = [&](int c, long &id) {
        const int rr = c / NCX, xi = c - rr * NCX;
        const int row = r0 + rr;
        int x = f0 - 3 + xi;
        if (row >= nrows || x > nlast) return false;
        int j = F.lo[1] + row % F.cnt[1], k = F.lo[2] + row / F.cnt[1];
        if (WRAP) { x = pwrap(x, G.n[0]); j = pwrap(j, G.n[1]); k = pwrap(k, G.n[2]); }
        id = G.base + x * G.s[0] + j * G.s[1] + k * G.s[2];
        return true;
    };
    if constexpr (WRAP) {
        stage_tile<(NC + 255) / 256>(u, G.sv, cm, P.gamma, sq, NC, NC, cell_id);
    } else {
        for (int c = tid; c < NC; c += TILE * ROWS) {
            long id;
            if (cell_id(c, id)) stage_cell(u, id, G.sv, cm, P.gamma, sq + c, NC);
        }
    }
    __syncthreads();
    stage_end();
    const int row = r0 + w;
    int pos[3];
    pos[0] = f0 + lane;
    pos[1] = F.lo[1] + row % F.cnt[1];
    pos[2] = F.lo[2] + row / F.cnt[1];
    if (row < nrows && pos[0] < F.cnt[0]) {
        T out[7];
        face_flux<T, false, WZ, GLF>(sq, NC, w * NCX + lane, 1, P.gamma, P.igm1, (T)P.eps, out, nullptr, P.ag);
        store_face<0, T>(flux, F, pos, out);
    }
    __syncthreads();
}

// Values of one cell of the fused x sweeps: its y and z faces' fluxes and the
// RK arrays the stage form reads.
template <typename T>
struct FusedCell {
    T fyl[5], fyr[5], fzl[5], fzr[5], w0[5], w1[5];
};

// x sweep over the flattened (row, face) space, for rows of at least
// XSEG_MIN faces: tile t takes the TILE*ROWS consecutive faces t*256 ..
// of the row-major face sequence, which touch at most 4 rows (XTile); it
// stages the cells of its row segments with their 3 + 2 halo (256 + 5*4
// cells at most, the size of the regular x tile) and each thread takes one
// face.  Only the last tile of the sweep is ragged.
constexpr int XSEG_MIN = 86;
constexpr int XSEG_CELLS = ROWS * NCX;

// Scalar constants of an x sweep's tiles (launch constants).
struct XSegArgs {
    FastDiv nf, n1;            // faces per row, rows per plane of the face box
    uint32_t total;            // faces of the sweep
};
__host__ inline XSegArgs xseg_args(const FaceBox &F)
{
    XSegArgs A;
    A.nf = FastDiv((uint32_t)F.cnt[0]);
    A.n1 = FastDiv((uint32_t)F.cnt[1]);
    A.total = (uint32_t)F.sc;
    return A;
}

// State index of the tile's first staged cell, and the jump of state_rel.
__device__ __forceinline__ long xseg_base(const Geom &G, const FaceBox &F, const XTile &X)
{
    return G.base + (X.fa0 - 3) + (long)(F.lo[1] + X.jj0) * G.s[1] + (long)(F.lo[2] + X.kk0) * G.s[2];
}
__device__ __forceinline__ uint32_t xseg_jump(const Geom &G, const FaceBox &F)
{
    return (uint32_t)(G.s[2] - (long)F.cnt[1] * G.s[1]);
}


// Stage the tile's cells (x sweep frame), sq with stride XSEG_CELLS; ub: the
// state at the tile's first cell.  A thread's loads first (stage_tile's
// order), at 32-bit offsets: a tile spans at most nine state rows of at most
// 2^20 + 6 cells.
template <typename T, bool PRE = false, bool LIN = false>
__device__ __forceinline__ void xseg_stage(const T *__restrict__ ub, long sv, uint32_t jump, double gamma,
                                           const XTile &X, int tid, T *sq)
{
    constexpr int IT = (XSEG_CELLS + 255) / 256;
    T w[IT][8];
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        const int c = tid + it * TILE * ROWS;
        if (c < X.ncell) {
            const uint32_t r = X.state_rel(c, jump);
#pragma unroll
            for (int v = 0; v < 8; ++v) w[it][v] = ld32(ub + v * sv, r);
        }
    }
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        const int c = tid + it * TILE * ROWS;
        if (c < X.ncell) stage_values<T, PRE, LIN>(w[it], gamma, sq + c, XSEG_CELLS);
    }
}

template <typename T, bool WZ = false, bool GLF = false, bool PRE = false>
__device__ __forceinline__ void sweep_tile_xseg(const T *__restrict__ u, T *__restrict__ flux,
                                                const Geom &G, const FaceBox &F, const Phys &P,
                                                const XSegArgs &A, uint32_t tile, T *sq)
{
    stage_begin();
    const int tid = threadIdx.x + TILE * threadIdx.y;
    const XTile X = xtile(tile * (TILE * ROWS), A.total, A.nf, A.n1);
    xseg_stage<T, PRE>(u + xseg_base(G, F, X), G.sv, xseg_jump(G, F), P.gamma, X, tid, sq);
    __syncthreads();
    stage_end();
    if (tid < X.nface) {
        T out[7];
        face_flux<T, false, WZ, GLF, PRE>(sq, XSEG_CELLS, X.cell_of(tid, X.row_of(tid)), 1, P.gamma, P.igm1,
                                                (T)P.eps, out, nullptr, P.ag);
        // faces are stored in the order of their numbers; the x frame is the grid's
        T *const fb = flux + X.g0;
#pragma unroll
        for (int c = 0; c < 7; ++c) st32<T>(fb + c * F.sc, tid, out[c]);
    }
}

// The cell between tile faces t and t + 1 of row s (face x index f): its y
// and z faces' fluxes (offsets ry, rz) and RK arrays (offset rel), read at
// 32-bit offsets from the tile's scalar bases (64-bit products and the row
// divisions were a fifth of the fused sweep's VALU time).  A row of the x faces advances both face
// boxes by a row of n0 + 2 faces; passing to the next plane, the y faces' rows
// (one fewer per plane) lag by one.
template <typename T>
struct FusedTile {
    const T *fy, *fz;          // y, z face fluxes at row 0 of the tile, x face 0's cell
    const T *u0, *acc_in;      // RK arrays at the tile's first staged cell
                               // (the batched form: at the patch's cell (0, 0, 0);
                               // FAR: at the box's)
    T *acc_out, *out;
    int nx2;                   // n0 + 2
};
template <typename T>
__device__ __forceinline__ FusedTile<T> fused_tile(const XFuse<T> &xf, long ubase, const XTile &X)
{
    FusedTile<T> B;
    B.nx2 = X.nf + 1;
    B.fy = xf.fy + 1 + (long)(X.jj0 - 1) * B.nx2 + (long)X.kk0 * xf.by.s[2];
    B.fz = xf.fz + 1 + (long)X.jj0 * B.nx2 + (long)(X.kk0 - 1) * xf.bz.s[2];
    B.u0 = xf.u0 + ubase;
    B.acc_in = xf.acc_in + ubase;
    B.acc_out = xf.acc_out + ubase;
    B.out = xf.out + ubase;
    return B;
}

template <bool FAR = false, typename T>
__device__ __forceinline__ void fused_tile_load(const XFuse<T> &xf, const FusedTile<T> &B, long sv, ElemOff<FAR> ry,
                                                ElemOff<FAR> rz, ElemOff<FAR> rel, FusedCell<T> &c)
{
    const int hs[5] = { 0, 1, 2, 3, 6 }, hv[5] = { 0, 1, 2, 3, 7 };
    const StageCoef &q = xf.c;
    const bool u0 = (q.mode == 1 && q.s < 3) || q.mode == 2;
    const bool ac = (q.mode == 1 && q.s > 0) || (q.mode == 2 && q.a1 != 0.0);
#pragma unroll
    for (int h = 0; h < 5; ++h) {
        c.fyl[h] = ld_off<FAR>(B.fy + hs[h] * xf.by.sc, ry);
        c.fyr[h] = ld_off<FAR>(B.fy + hs[h] * xf.by.sc + B.nx2, ry);
        c.fzl[h] = ld_off<FAR>(B.fz + hs[h] * xf.bz.sc, rz);
        c.fzr[h] = ld_off<FAR>(B.fz + hs[h] * xf.bz.sc + xf.bz.s[2], rz);
        c.w0[h] = u0 ? ld_off<FAR>(B.u0 + hv[h] * sv, rel) : T(0);
        c.w1[h] = ac ? ld_off<FAR>(B.acc_in + hv[h] * sv, rel) : T(0);
    }
}

// The RK combination of that cell from its x fluxes and the loaded values (the
// update kernel's expressions and order, x, y, z: identical results).
template <bool FAR = false, typename T>
__device__ __forceinline__ void fused_tile_store(const XFuse<T> &xf, const FusedTile<T> &B, const Geom &G,
                                                 const T *hx, int nh, int t, ElemOff<FAR> rel, const FusedCell<T> &c)
{
    const int hv[5] = { 0, 1, 2, 3, 7 };
    const T idx = T(G.idl[0]), idy = T(G.idl[1]), idz = T(G.idl[2]);
    const StageCoef &q = xf.c;
    const T bdt = T(q.bdt), cdt = T(q.cdt), a0 = T(q.a0), a1 = T(q.a1);
#pragma unroll
    for (int h = 0; h < 5; ++h) {
        T L = T(0);
        L -= (hx[h * nh + t + 1] - hx[h * nh + t]) * idx;
        L -= (c.fyr[h] - c.fyl[h]) * idy;
        L -= (c.fzr[h] - c.fzl[h]) * idz;
        T *const out = B.out + hv[h] * G.sv, *const acc = B.acc_out + hv[h] * G.sv;
        if (q.mode == 0) {
            st_off<FAR, T>(out, rel, L);
        } else if (q.mode == 2) {
            st_off<FAR, T>(out, rel, q.a1 != 0.0 ? a0 * c.w0[h] + a1 * c.w1[h] + cdt * L : a0 * c.w0[h] + cdt * L);
        } else if (q.s == 0) {
            st_off<FAR, T>(acc, rel, c.w0[h] + bdt * L);
            st_off<FAR, T>(out, rel, c.w0[h] + cdt * L);
        } else if (q.s < 3) {
            st_off<FAR, T>(acc, rel, c.w1[h] + bdt * L);
            st_off<FAR, T>(out, rel, c.w0[h] + cdt * L);
        } else {
            st_off<FAR, T>(out, rel, c.w1[h] + cdt * L);
        }
    }
}

// The x sweep with the hydro part of the update fused in.  Tiles of 256
// faces overlap by one (tile t starts at face 255 t of the row-major face
// sequence), so both faces of every cell of a row meet in one tile.  After
// the fluxes, each thread puts its face's rho, m, E fluxes in LDS (hx, 5 x
// 256), and thread tid takes the cell between faces tid and tid+1 when both
// lie in one row and the row is interior: its x difference from LDS, its y
// and z differences from the other sweeps' face fluxes (same expressions
// and order as the update kernel: the results are identical), then the RK
// combination of rho, m, E.  Only the transverse-B fluxes (slots 4, 5) are
// stored, once per face (the overlapping face by the next tile).
constexpr int XFUSE_STRIDE = TILE * ROWS - 1;

template <typename T, bool WZ = false, bool GLF = false, bool PRE = false>
__device__ __forceinline__ void sweep_tile_xseg_fused(const T *__restrict__ u, T *__restrict__ flux,
                                                      const Geom &G, const FaceBox &F, const Phys &P,
                                                      const XSegArgs &A, uint32_t tile, T *sq, T *hx,
                                                      const XFuse<T> &xf)
{
    constexpr int NH = TILE * ROWS;
    stage_begin();
    {
        const int tid = threadIdx.x + TILE * threadIdx.y;
        const XTile X = xtile(tile * XFUSE_STRIDE, A.total, A.nf, A.n1);
        xseg_stage<T, PRE>(u + xseg_base(G, F, X), G.sv, xseg_jump(G, F), P.gamma, X, tid, sq);
        __syncthreads();
        stage_end();
        if (tid < X.nface) {
            T out[7];
            face_flux<T, false, WZ, GLF, PRE, sizeof(T) == 8>(sq, XSEG_CELLS, X.cell_of(tid, X.row_of(tid)), 1,
                                                              P.gamma, P.igm1, (T)P.eps, out, nullptr, P.ag);
            hx[0 * NH + tid] = out[0];
            hx[1 * NH + tid] = out[1];
            hx[2 * NH + tid] = out[2];
            hx[3 * NH + tid] = out[3];
            hx[4 * NH + tid] = out[6];
            if (tid < XFUSE_STRIDE || X.g0 + tid == A.total - 1) {
                st32<T>(flux + 4 * F.sc + X.g0, tid, out[4]);
                st32<T>(flux + 5 * F.sc + X.g0, tid, out[5]);
            }
        }
    }
    // The cell between faces t and t + 1 of one row (face f sits at f - 1/2);
    // interior rows are 1..n of the face box's transverse numbering.  Tile
    // and thread numbers are opaque to the compiler here: the tile's rows and
    // bases are formed again instead of staying in registers through the
    // flux, where the FP64 form has none left.
    int t = threadIdx.x + TILE * threadIdx.y;
    asm volatile("" : "+v"(t), "+s"(tile));
    const XTile X = xtile(tile * XFUSE_STRIDE, A.total, A.nf, A.n1);
    const long ubase = xseg_base(G, F, X);
    const int s = X.row_of(t), f = X.face_x(t, s), jj = X.jj(s), kk = X.kk(s);
    const bool cell = t + 1 < X.nface && t < XFUSE_STRIDE && f + 1 < X.nf && jj >= 1 && jj <= G.n[1] && kk >= 1 &&
                      kk <= G.n[2];
    const uint32_t rel = X.state_rel(X.cell_of(t, s) + 3, xseg_jump(G, F));
    const FusedTile<T> B = fused_tile(xf, ubase, X);
    FusedCell<T> fc;
    if (cell)
        fused_tile_load(xf, B, G.sv, f + __umul24(s - (s >= X.sw ? 1 : 0), B.nx2), f + __umul24(s, B.nx2), rel, fc);
    __syncthreads();
    if (cell) fused_tile_store(xf, B, G, hx, NH, t, rel, fc);
}

// y or z sweep with PW positions of the transverse plane (x fastest) per
// tile and FT faces along the sweep: fewer positions per tile stage fewer
// halo cells per face ((FT+5)/FT) in the same LDS.
template <int PW, int FT>
__host__ __device__ constexpr int yz_cells() { return PW * (FT + 5); }

// Scalar constants of a y/z sweep's tiles (launch constants).
struct YZArgs {
    FastDiv na, nb;            // positions along x, tiles along the sweep axis
    uint32_t npos, ntile, per_xcd;
};

// Hardware block b runs on XCD b % 8 (blocks are dealt round-robin to the
// eight XCDs, each with its own L2).
constexpr int NXCD = 8;

// y/z sweeps: tiles (ta: positions of the transverse plane, tb: faces along
// the sweep axis) are renumbered so that each XCD walks whole columns of
// tiles, tb fastest.  A tile's 5 halo rows along the sweep axis were staged
// by the tile before it on the same XCD and come from that XCD's L2.
__device__ __forceinline__ bool column_tile(const YZArgs &Y, uint32_t &ta, uint32_t &tb, uint32_t &lb)
{
    lb = (blockIdx.x % NXCD) * Y.per_xcd + blockIdx.x / NXCD;
    if (lb >= Y.ntile) return false;
    ta = Y.nb.div(lb);
    tb = lb - ta * Y.nb.d;
    return true;
}

// Tile (ta, tb) of a y/z sweep, one thread's place in it.  Element offsets
// within a tile are 32-bit: they stay within one variable (or face
// component), and a context keeps at least three states of eight variables,
// so that one variable holds at most 288 GB / 96 B = 3.0e9 < 2^32 elements.
// (Their byte offsets can pass 2^32: they index by element, not by ld32, st32.)
template <int DIR, int PW, int FT>
struct YZTile {
    static constexpr int N = DIR, A = 0, B = DIR == 1 ? 2 : 1;
    uint32_t a0, b0;           // first position
    int np, f0;                // positions of the tile, first face
    int pl, fr;                // the thread's position and row within the tile
    int q;                     // rows its position lies beyond (a0, b0)'s
    __device__ __forceinline__ YZTile(const YZArgs &Y, uint32_t ta, uint32_t tb, int tid)
    {
        const uint32_t p0 = ta * PW;
        b0 = Y.na.div(p0);
        a0 = p0 - b0 * Y.na.d;
        np = (int)(Y.npos - p0 < (uint32_t)PW ? Y.npos - p0 : (uint32_t)PW);
        f0 = (int)tb * FT;
        pl = tid % PW;
        fr = PW == TILE ? __builtin_amdgcn_readfirstlane(tid / PW) : tid / PW;
        q = yz_rows_on(a0, pl, Y.na, PW);
    }
    __device__ __forceinline__ int pos_a(const FaceBox &F, const YZArgs &Y) const
    {
        return F.lo[A] + (int)(a0 + pl - q * Y.na.d);
    }
    __device__ __forceinline__ int pos_b(const FaceBox &F) const { return F.lo[B] + (int)b0 + q; }
    // offset of the thread's face row fr from the tile's first face in the flux box
    __device__ __forceinline__ uint32_t face_rel(const FaceBox &F, const YZArgs &Y, int row) const
    {
        return (uint32_t)pl + (uint32_t)q * (uint32_t)(F.s[B] - Y.na.d) + (uint32_t)row * (uint32_t)F.s[N];
    }
    __device__ __forceinline__ long face_base(const FaceBox &F) const
    {
        return (long)a0 + (long)b0 * F.s[B] + (long)f0 * F.s[N];
    }
};

template <int DIR, int PW, int FT, typename T, bool LIN = false>
__device__ __forceinline__ void yz_stage(const T *__restrict__ u, const Geom &G, const FaceBox &F, double gamma,
                                         const YZArgs &Y, const YZTile<DIR, PW, FT> &t, T *sq)
{
    constexpr int N = DIR, T1 = (DIR + 1) % 3, T2 = (DIR + 2) % 3, B = DIR == 1 ? 2 : 1;
    constexpr int NC = yz_cells<PW, FT>(), RP = 256 / PW;
    const int cm[8] = { 0, 1 + N, 1 + T1, 1 + T2, 4 + N, 4 + T1, 4 + T2, 7 };
    const T *const ub = u + (G.base + F.lo[0] + (long)t.a0 + (long)(F.lo[B] + (int)t.b0) * G.s[B] +
                             (long)(t.f0 - 3) * G.s[N]);
    const int rows = min(FT + 5, G.n[N] + 6 - t.f0);     // the state's rows end at n + 2
    if (t.pl >= t.np) return;
    const uint32_t rel = (uint32_t)t.pl + (uint32_t)t.q * (uint32_t)(G.s[B] - Y.na.d);
    // one cell after another (a thread's loads first, as stage_tile does,
    // measured 2 % slower here)
    for (int r = t.fr; r < rows; r += RP) {
        const uint32_t e = rel + (uint32_t)r * (uint32_t)G.s[N];
        T w[8];
#pragma unroll
        for (int v = 0; v < 8; ++v) w[v] = uniform(ub + cm[v] * G.sv)[e];
        stage_values<T, false, LIN>(w, gamma, sq + (r * PW + t.pl), NC);
    }
}

template <int DIR, int PW, int FT, typename T, bool WZ = false, bool GLF = false>
__device__ __forceinline__ void sweep_tile_yz(const T *__restrict__ u, T *__restrict__ flux,
                                              const Geom &G, const FaceBox &F, const Phys &P, const YZArgs &Y,
                                              uint32_t ta, uint32_t tb, T *sq)
{
    constexpr int T1 = (DIR + 1) % 3, T2 = (DIR + 2) % 3;
    stage_begin();
    const YZTile<DIR, PW, FT> t(Y, ta, tb, threadIdx.x + TILE * threadIdx.y);
    yz_stage<DIR, PW, FT, T>(u, G, F, P.gamma, Y, t, sq);
    __syncthreads();
    stage_end();
    T *const fb = flux + t.face_base(F);
    for (int r = t.fr; r < FT; r += 256 / PW) {
        if (t.pl < t.np && t.f0 + r < F.cnt[DIR]) {
            T out[7];
            face_flux<T, false, WZ, GLF>(sq, yz_cells<PW, FT>(), r * PW + t.pl, PW, P.gamma, P.igm1, (T)P.eps, out,
                                         nullptr, P.ag);
            const uint32_t rel = t.face_rel(F, Y, r);
            const int gc[7] = { 0, 1 + DIR, 1 + T1, 1 + T2, 4, 5, 6 };   // sweep frame -> grid component
#pragma unroll
            for (int c = 0; c < 7; ++c) uniform(fb + gc[c] * F.sc)[rel] = out[c];
        }
    }
}

template <int DIR, int PW, int FT>
__host__ inline YZArgs yz_args(const FaceBox &F, uint32_t nxcd)
{
    constexpr int B = DIR == 1 ? 2 : 1;
    YZArgs Y;
    Y.npos = (uint32_t)F.cnt[0] * (uint32_t)F.cnt[B];
    Y.na = FastDiv((uint32_t)F.cnt[0]);
    const uint32_t na = (Y.npos + PW - 1) / PW, nb = (uint32_t)(F.cnt[DIR] + FT - 1) / FT;
    Y.nb = FastDiv(nb);
    Y.ntile = na * nb;
    Y.per_xcd = (Y.ntile + nxcd - 1) / nxcd;
    return Y;
}

// Number of tiles (ta, tb) of sweep_tile_xrows.
__host__ __device__ inline void xrows_tiles(const FaceBox &F, long &na, long &nb)
{
    na = ((long)F.cnt[1] * F.cnt[2] + ROWS - 1) / ROWS;
    nb = (F.cnt[0] + TILE - 1) / TILE;
}

}  // namespace sw
}  // namespace ww
