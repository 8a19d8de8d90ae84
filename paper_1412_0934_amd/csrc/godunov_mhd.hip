// gfx950 kernels of one unsplit MUSCL-Hancock step of ideal MHD with
// hyperbolic-parabolic divergence cleaning (GLM), on a periodic box.
//
// The Euler step's method family (Sec. 2) carried to the MHD equations of the
// paper's Enzo solver (Sec. 4): conserved U = (rho, rho v, E, B, psi) with
// E = p/(gamma-1) + rho|v|^2/2 + |B|^2/2; limited primitive slopes; the
// conservative MUSCL-Hancock half step, in which the upper- and lower-face
// values of a cell along each axis move by the same increment
//   dU = -dt/(2dx) sum_d [F_d(W + S_d/2) - F_d(W - S_d/2)];
// at every face the GLM 2x2 problem for (B_n, psi) fixes the normal field
//   B_n* = (B_nL + B_nR)/2 - (psi_R - psi_L)/(2 ch),
//   psi* = (psi_L + psi_R)/2 - ch (B_nR - B_nL)/2,
// whose fluxes are psi* and ch^2 B_n*, and the HLLD solver of Miyoshi and
// Kusano (2005) with that normal field gives the other seven fluxes; then
// U' = U - dt/dx ((dF_x + dF_y) + dF_z) and psi' <- psi' exp(-alpha ch dt/dx).
//
// Double precision takes one launch per step (and a one-thread launch for the
// next dt and ch): the tile march of the Euler step (godunov_tile.h) with nine
// variables; the predicted face states never leave the chip.
// Single precision takes two launches over a library-owned scratch: predict
// (one thread per cell: 7-point stencil, slopes, half step, six predicted face
// states) and a flux sweep (z-marching column tiles: x and y faces through LDS,
// z faces in registers, the update, and optionally the signal speeds of the
// new state): its results are kept bit for bit.
// Every value is written by one thread and the reductions are maxima:
// deterministic.
#include "godunov_internal.h"
#include "godunov_math.h"
#include "godunov_tile.h"

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

namespace gd {

namespace mhd {

enum { LIM_MINMOD = 0, LIM_MC = 1, LIM_NONE = 2 };
constexpr int NV = 9;

template <typename T>
struct Par {
    int nx, ny, nz, n;        // box and its cell count
    T gamma, gm1, inv_gm1, rho_floor, p_floor;
    T h;                      // dt / (2 dx)
    T c;                      // dt / dx
    T ch, ch2;                // cleaning speed and its square
    T ich2;                   // 1 / (2 ch)
    T damp;                   // exp(-alpha ch dt / dx)
};

// The step's time-dependent parameters (h, c, ch, ch^2, damp) when dt or ch
// come from device scalars: computed on the device by k_params, read by every
// kernel of the step.
template <typename T>
__device__ __forceinline__ void take_dynamic(Par<T> &P, const T *__restrict__ dyn)
{
    if (!dyn) return;
    P.h = dyn[0]; P.c = dyn[1]; P.ch = dyn[2]; P.ch2 = dyn[3]; P.damp = dyn[4];
}

template <typename T>
__device__ __forceinline__ T limited(int lim, T a, T b)
{
    if (lim == LIM_NONE) return T(0.5) * (a + b);
    if (!((a > T(0) && b > T(0)) || (a < T(0) && b < T(0)))) return T(0);
    if (lim == LIM_MINMOD) return fabs(a) <= fabs(b) ? a : b;
    T m = fmin(fmin(T(2) * fabs(a), T(2) * fabs(b)), T(0.5) * fabs(a + b));
    return a > T(0) ? m : -m;
}

// sqrt(x), x >= 0, from the hardware reciprocal square root refined by one
// Newton step (relative error within about 4e-15 in FP64)
template <typename T>
__device__ __forceinline__ T hw_sqrt(T x)
{
    return x > T(0) ? x * fast_rsqrt(x) : T(0);
}

// The helpers below are inlined in several places whose results have to agree:
// the tile's columns and the ring's predict the same cells, the step and
// cfl_dt_mhd reduce the same speeds. In double precision their products and sums
// are therefore fused as written, by fma() and not by the compiler's choice,
// which shared a product among six face states in one loop and fused it into each
// in the other. In single precision, whose step has one copy of each, the
// expressions are left to the compiler.

// sum of three products
__device__ __forceinline__ double dot3(const double *x, const double *y)
{
#pragma clang fp contract(off)
    return fma(x[2], y[2], fma(x[1], y[1], x[0] * y[0]));
}

// Divisions and square roots: EXACT = IEEE-rounded (the signal speeds behind
// dt and ch), else the refined hardware estimates (the step's arithmetic).
template <bool EXACT, typename T>
__device__ __forceinline__ void to_prim(const Par<T> &P, const T U[NV], T W[NV])
{
    if constexpr (sizeof(T) == 8) {
#pragma clang fp contract(off)
        const T rho = U[0] < P.rho_floor ? P.rho_floor : U[0];
        if constexpr (EXACT) {
            W[1] = U[1] / rho; W[2] = U[2] / rho; W[3] = U[3] / rho;
        } else {
            const T ir = fast_rcp(rho);
            W[1] = U[1] * ir; W[2] = U[2] * ir; W[3] = U[3] * ir;
        }
        const T p = P.gm1 * fma(T(-0.5), dot3(U + 5, U + 5), fma(T(-0.5), dot3(U + 1, W + 1), U[4]));
        W[0] = rho;
        W[4] = p < P.p_floor ? P.p_floor : p;
    } else {
        T rho = U[0] < P.rho_floor ? P.rho_floor : U[0];
        T u, v, w;
        if constexpr (EXACT) {
            u = U[1] / rho; v = U[2] / rho; w = U[3] / rho;
        } else {
            const T ir = fast_rcp(rho);
            u = U[1] * ir; v = U[2] * ir; w = U[3] * ir;
        }
        T kin = T(0.5) * (U[1] * u + U[2] * v + U[3] * w);
        T mag = T(0.5) * (U[5] * U[5] + U[6] * U[6] + U[7] * U[7]);
        T p = P.gm1 * (U[4] - kin - mag);
        if (p < P.p_floor) p = P.p_floor;
        W[0] = rho; W[1] = u; W[2] = v; W[3] = w; W[4] = p;
    }
    W[5] = U[5]; W[6] = U[6]; W[7] = U[7]; W[8] = U[8];
}

// total energy of a primitive state in double precision
__device__ __forceinline__ double energy(const Par<double> &P, const double W[NV])
{
#pragma clang fp contract(off)
    return fma(0.5, dot3(W + 5, W + 5), fma(0.5 * W[0], dot3(W + 1, W + 1), W[4] * P.inv_gm1));
}

template <typename T>
__device__ __forceinline__ void to_cons(const Par<T> &P, const T W[NV], T U[NV])
{
    const T rho = W[0];
    U[0] = rho;
    if constexpr (sizeof(T) == 8) {
#pragma clang fp contract(off)
        U[1] = rho * W[1]; U[2] = rho * W[2]; U[3] = rho * W[3];
        U[4] = energy(P, W);
    } else {
        U[1] = rho * W[1]; U[2] = rho * W[2]; U[3] = rho * W[3];
        U[4] = W[4] * P.inv_gm1 + T(0.5) * rho * (W[1] * W[1] + W[2] * W[2] + W[3] * W[3]) +
               T(0.5) * (W[5] * W[5] + W[6] * W[6] + W[7] * W[7]);
    }
    U[5] = W[5]; U[6] = W[6]; U[7] = W[7]; U[8] = W[8];
}

// fast magnetosonic speed of the primitive state along the axis whose field
// component is bn
template <bool EXACT, typename T>
__device__ __forceinline__ T fast_speed(const Par<T> &P, const T W[NV], T bn)
{
    const T ir = EXACT ? T(1) / W[0] : fast_rcp(W[0]);
    if constexpr (sizeof(T) == 8) {
#pragma clang fp contract(off)
        const T a2 = P.gamma * W[4] * ir;
        const T s = fma(dot3(W + 5, W + 5), ir, a2);
        const T disc = fma(s, s, T(-4) * a2 * (bn * bn * ir));
        const T r = disc < T(0) ? T(0) : disc;
        if constexpr (EXACT) return sqrt(T(0.5) * (s + sqrt(r)));
        else return hw_sqrt(T(0.5) * (s + hw_sqrt(r)));
    }
    const T a2 = P.gamma * W[4] * ir;
    const T b2 = (W[5] * W[5] + W[6] * W[6] + W[7] * W[7]) * ir;
    const T s = a2 + b2;
    T disc = s * s - T(4) * a2 * (bn * bn * ir);
    disc = disc < T(0) ? T(0) : disc;
    if constexpr (EXACT) return sqrt(T(0.5) * (s + sqrt(disc)));
    else return hw_sqrt(T(0.5) * (s + hw_sqrt(disc)));
}

// physical GLM-MHD flux along axis D
template <int D, typename T>
__device__ __forceinline__ void phys_flux(const Par<T> &P, const T W[NV], T F[NV])
{
    const T rho = W[0], p = W[4];
    const T un = W[1 + D], Bn = W[5 + D];
    if constexpr (sizeof(T) == 8) {
#pragma clang fp contract(off)
        const T pT = fma(T(0.5), dot3(W + 5, W + 5), p), m = rho * un;
        F[0] = m;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            F[1 + k] = fma(m, W[1 + k], k == D ? fma(-Bn, Bn, pT) : -(Bn * W[5 + k]));
            F[5 + k] = k == D ? W[8] : fma(un, W[5 + k], -(W[1 + k] * Bn));
        }
        F[4] = fma(energy(P, W) + pT, un, -(Bn * dot3(W + 1, W + 5)));
        F[8] = P.ch2 * Bn;
        return;
    }
    const T B2 = W[5] * W[5] + W[6] * W[6] + W[7] * W[7];
    const T pT = p + T(0.5) * B2;
    const T uB = W[1] * W[5] + W[2] * W[6] + W[3] * W[7];
    const T E = p * P.inv_gm1 + T(0.5) * rho * (W[1] * W[1] + W[2] * W[2] + W[3] * W[3]) +
                T(0.5) * B2;
    F[0] = rho * un;
#pragma unroll
    for (int k = 0; k < 3; ++k) F[1 + k] = rho * un * W[1 + k] - Bn * W[5 + k] + (k == D ? pT : T(0));
    F[4] = (E + pT) * un - Bn * uB;
#pragma unroll
    for (int k = 0; k < 3; ++k) F[5 + k] = k == D ? W[8] : un * W[5 + k] - W[1 + k] * Bn;
    F[8] = P.ch2 * Bn;
}

// HLLD in the frame of the face: L, R = (rho, u_n, u_t1, u_t2, p, Bn, B_t1,
// B_t2) with the same Bn; fluxes of (rho, m_n, m_t1, m_t2, E, B_t1, B_t2).
template <typename T>
__device__ __forceinline__ void hlld(const Par<T> &P, const T L[8], const T R[8], T F[7])
{
    const T Bn = L[5];
    const T sgn = Bn > T(0) ? T(1) : (Bn < T(0) ? T(-1) : T(0));
    T Uc[2][8], Fc[2][7], pT[2], cf[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const T *W = s ? R : L;
        const T rho = W[0], u = W[1], v = W[2], w = W[3], p = W[4], By = W[6], Bz = W[7];
        const T B2 = Bn * Bn + By * By + Bz * Bz;
        pT[s] = p + T(0.5) * B2;
        const T E = p * P.inv_gm1 + T(0.5) * rho * (u * u + v * v + w * w) + T(0.5) * B2;
        const T uB = u * Bn + v * By + w * Bz;
        Uc[s][0] = rho; Uc[s][1] = rho * u; Uc[s][2] = rho * v; Uc[s][3] = rho * w;
        Uc[s][4] = E; Uc[s][5] = Bn; Uc[s][6] = By; Uc[s][7] = Bz;
        Fc[s][0] = rho * u;
        Fc[s][1] = rho * u * u + pT[s] - Bn * Bn;
        Fc[s][2] = rho * u * v - Bn * By;
        Fc[s][3] = rho * u * w - Bn * Bz;
        Fc[s][4] = (E + pT[s]) * u - Bn * uB;
        Fc[s][5] = u * By - v * Bn;
        Fc[s][6] = u * Bz - w * Bn;
        const T Wf[NV] = { rho, u, v, w, p, Bn, By, Bz, T(0) };
        cf[s] = fast_speed<false>(P, Wf, Bn);
    }
    const T SL = fmin(L[1] - cf[0], R[1] - cf[1]);
    const T SR = fmax(L[1] + cf[0], R[1] + cf[1]);
    if (SL >= T(0)) {
        for (int q = 0; q < 7; ++q) F[q] = Fc[0][q];
        return;
    }
    if (SR <= T(0)) {
        for (int q = 0; q < 7; ++q) F[q] = Fc[1][q];
        return;
    }
    const T dL = (SL - L[1]) * L[0], dR = (SR - R[1]) * R[0];
    const T idd = fast_rcp(dR - dL);
    const T SM = (dR * R[1] - dL * L[1] - pT[1] + pT[0]) * idd;
    const T pTs = (dR * pT[0] - dL * pT[1] + dL * dR * (R[1] - L[1])) * idd;

    // single-star states
    T Us[2][8], sq[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const T *W = s ? R : L;
        const T S = s ? SR : SL;
        const T rho = W[0], u = W[1], v = W[2], w = W[3], By = W[6], Bz = W[7];
        const T isd = fast_rcp(S - SM);
        const T rs = rho * (S - u) * isd;
        const T den = rho * (S - u) * (S - SM) - Bn * Bn;
        T vs = v, ws = w, Bys = By, Bzs = Bz;
        if (!(fabs(den) <= T(1e-12) * (rho * (S - u) * (S - u) + Bn * Bn))) {
            const T iden = fast_rcp(den);
            const T t = Bn * (SM - u) * iden;
            vs = v - By * t;
            ws = w - Bz * t;
            const T q = (rho * (S - u) * (S - u) - Bn * Bn) * iden;
            Bys = By * q;
            Bzs = Bz * q;
        }
        const T uB = u * Bn + v * By + w * Bz;
        const T uBs = SM * Bn + vs * Bys + ws * Bzs;
        const T Es = ((S - u) * Uc[s][4] - pT[s] * u + pTs * SM + Bn * (uB - uBs)) * isd;
        Us[s][0] = rs; Us[s][1] = rs * SM; Us[s][2] = rs * vs; Us[s][3] = rs * ws;
        Us[s][4] = Es; Us[s][5] = Bn; Us[s][6] = Bys; Us[s][7] = Bzs;
        sq[s] = hw_sqrt(rs);
    }
    const T SLs = SM - fabs(Bn) * fast_rcp(sq[0]);
    const T SRs = SM + fabs(Bn) * fast_rcp(sq[1]);
    // the side of the contact the face lies on: left when SM >= 0 (values are
    // selected, not indexed, so that everything stays in registers)
    const bool left = SM >= T(0);
    const T SK = left ? SL : SR;
    T UcK[8], UsK[8], Fs[7];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        UcK[q] = left ? Uc[0][q] : Uc[1][q];
        UsK[q] = left ? Us[0][q] : Us[1][q];
    }
#pragma unroll
    for (int q = 0; q < 7; ++q) {
        const int c = q < 5 ? q : q + 1;
        Fs[q] = (left ? Fc[0][q] : Fc[1][q]) + SK * (UsK[c] - UcK[c]);
    }
    // outside the Alfven waves: the single-star flux of that side
    if ((left && SLs >= T(0)) || (!left && SRs <= T(0))) {
        for (int q = 0; q < 7; ++q) F[q] = Fs[q];
        return;
    }
    // between the Alfven waves: the double-star states
    const T irL = fast_rcp(Us[0][0]), irR = fast_rcp(Us[1][0]);
    const T vL = Us[0][2] * irL, wL = Us[0][3] * irL;
    const T vR = Us[1][2] * irR, wR = Us[1][3] * irR;
    const T ByL = Us[0][6], BzL = Us[0][7], ByR = Us[1][6], BzR = Us[1][7];
    const T iss = fast_rcp(sq[0] + sq[1]);
    const T vss = (sq[0] * vL + sq[1] * vR + (ByR - ByL) * sgn) * iss;
    const T wss = (sq[0] * wL + sq[1] * wR + (BzR - BzL) * sgn) * iss;
    const T Byss = (sq[0] * ByR + sq[1] * ByL + sq[0] * sq[1] * (vR - vL) * sgn) * iss;
    const T Bzss = (sq[0] * BzR + sq[1] * BzL + sq[0] * sq[1] * (wR - wL) * sgn) * iss;
    const T uBss = SM * Bn + vss * Byss + wss * Bzss;
    const T vK = left ? vL : vR, wK = left ? wL : wR;
    const T ByK = left ? ByL : ByR, BzK = left ? BzL : BzR;
    const T uBs = SM * Bn + vK * ByK + wK * BzK;
    const T rK = UsK[0], sqK = left ? sq[0] : sq[1];
    const T sgnK = left ? T(-1) : T(1);
    const T Uss[8] = { rK, rK * SM, rK * vss, rK * wss, UsK[4] + sgnK * sqK * (uBs - uBss) * sgn,
                       Bn, Byss, Bzss };
    const T SKs = left ? SLs : SRs;
#pragma unroll
    for (int q = 0; q < 7; ++q) {
        const int c = q < 5 ? q : q + 1;
        F[q] = Fs[q] + SKs * (Uss[c] - UsK[c]);
    }
}

// GLM + HLLD flux through a face normal to D from unrotated primitive states
template <int D, typename T>
__device__ __forceinline__ void face_flux(const Par<T> &P, const T WL[NV], const T WR[NV], T F[NV])
{
    constexpr int t1 = (D + 1) % 3, t2 = (D + 2) % 3;
    const T Bns = T(0.5) * (WL[5 + D] + WR[5 + D]) - (WR[8] - WL[8]) * fast_rcp(T(2) * P.ch);
    const T psis = T(0.5) * (WL[8] + WR[8]) - T(0.5) * P.ch * (WR[5 + D] - WL[5 + D]);
    const T L[8] = { WL[0], WL[1 + D], WL[1 + t1], WL[1 + t2], WL[4], Bns, WL[5 + t1], WL[5 + t2] };
    const T R[8] = { WR[0], WR[1 + D], WR[1 + t1], WR[1 + t2], WR[4], Bns, WR[5 + t1], WR[5 + t2] };
    T Fr[7];
    hlld(P, L, R, Fr);
    F[0] = Fr[0];
    F[1 + D] = Fr[1]; F[1 + t1] = Fr[2]; F[1 + t2] = Fr[3];
    F[4] = Fr[4];
    F[5 + D] = psis; F[5 + t1] = Fr[5]; F[5 + t2] = Fr[6];
    F[8] = P.ch2 * Bns;
}

__device__ __forceinline__ int wrap(int i, int n)
{
    if (i < 0) i += n;
    else if (i >= n) i -= n;
    if ((unsigned)i >= (unsigned)n) { i %= n; if (i < 0) i += n; }
    return i;
}

__device__ __forceinline__ int cell(int nx, int ny, int nz, int i, int j, int k)
{
    return (wrap(k, nz) * ny + wrap(j, ny)) * nx + wrap(i, nx);
}

template <bool EXACT, typename T>
__device__ __forceinline__ void load_prim(const Par<T> &P, const T *__restrict__ u, int c, T W[NV])
{
    T U[NV];
#pragma unroll
    for (int q = 0; q < NV; ++q) U[q] = u[q * P.n + c];
    to_prim<EXACT>(P, U, W);
}

// face-state scratch: fs[(d*2 + side)*9 + q][cell], side 0 the upper-face
// state W*+ and side 1 the lower-face state W*-; flux scratch: fl[d*9 + q][cell]
// holds the flux through the lower face of the cell along d.

// The upper- and lower-face values W +- S/2 of a cell along d, with the
// density and pressure floors.
template <typename T>
__device__ __forceinline__ void face_values(const Par<T> &P, const T W[NV], const T S[NV], T up[NV],
                                            T dn[NV])
{
#pragma unroll
    for (int q = 0; q < NV; ++q) {
        up[q] = W[q] + T(0.5) * S[q];
        dn[q] = W[q] - T(0.5) * S[q];
    }
    up[0] = fmax(up[0], P.rho_floor); dn[0] = fmax(dn[0], P.rho_floor);
    up[4] = fmax(up[4], P.p_floor); dn[4] = fmax(dn[4], P.p_floor);
}

template <typename T, int LIM>
__global__ __launch_bounds__(256) void k_predict(Par<T> P, const T *__restrict__ dyn,
                                                 const T *__restrict__ u, T *__restrict__ fs)
{
    take_dynamic(P, dyn);
    const int i = blockIdx.x * 64 + threadIdx.x % 64;
    const int j = blockIdx.y * 4 + threadIdx.x / 64;
    const int k = blockIdx.z;
    if (i >= P.nx || j >= P.ny) return;
    const int c = (k * P.ny + j) * P.nx + i;
    T W[NV], dU[NV], S[3][NV];
    load_prim<false>(P, u, c, W);
#pragma unroll
    for (int q = 0; q < NV; ++q) dU[q] = T(0);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        {
            T Wm[NV], Wp[NV];
            load_prim<false>(P, u, cell(P.nx, P.ny, P.nz, i - (d == 0), j - (d == 1), k - (d == 2)), Wm);
            load_prim<false>(P, u, cell(P.nx, P.ny, P.nz, i + (d == 0), j + (d == 1), k + (d == 2)), Wp);
#pragma unroll
            for (int q = 0; q < NV; ++q) S[d][q] = limited<T>(LIM, W[q] - Wm[q], Wp[q] - W[q]);
        }
        T up[NV], dn[NV], Fu[NV], Fd[NV];
        face_values(P, W, S[d], up, dn);
        if (d == 0) { phys_flux<0>(P, up, Fu); phys_flux<0>(P, dn, Fd); }
        else if (d == 1) { phys_flux<1>(P, up, Fu); phys_flux<1>(P, dn, Fd); }
        else { phys_flux<2>(P, up, Fu); phys_flux<2>(P, dn, Fd); }
#pragma unroll
        for (int q = 0; q < NV; ++q) dU[q] -= Fu[q] - Fd[q];
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        T up[NV], dn[NV], Uu[NV], Ud[NV], Wu[NV], Wd[NV];
        face_values(P, W, S[d], up, dn);
        to_cons(P, up, Uu);
        to_cons(P, dn, Ud);
#pragma unroll
        for (int q = 0; q < NV; ++q) { Uu[q] += P.h * dU[q]; Ud[q] += P.h * dU[q]; }
        to_prim<false>(P, Uu, Wu);
        to_prim<false>(P, Ud, Wd);
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            // streamed out: the sweep reads each value back once, long after
            __builtin_nontemporal_store(Wu[q], &fs[(size_t)((d * 2 + 0) * NV + q) * P.n + c]);
            __builtin_nontemporal_store(Wd[q], &fs[(size_t)((d * 2 + 1) * NV + q) * P.n + c]);
        }
    }
}

// ------------------------------------------------------------ flux sweep (FP32)

// A workgroup owns a 16 x 16 column tile and marches up a z-range. Per plane,
// the predicted x-face states of the tile (and of one halo cell at each end
// of a row) are staged in LDS, every x face of the tile is evaluated once
// (faces on a tile border by both tiles) and its flux overwrites the left
// state it read; each cell takes its x flux difference; the same for y; the
// z face above a cell is evaluated in registers and serves the plane above
// as its lower face; then the update, and optionally the signal speeds of
// the new state for the next step's dt and cleaning speed.
constexpr int MTX = 16, MTY = 16, MT = MTX * MTY;
constexpr int MSLOT = (MTX + 1) * (MTY + 1);

template <typename T>
struct SweepSmem {
    T st[2][NV][MSLOT];      // [0] left state, then the flux; [1] right state
    double red[2][MT / 64];  // wave maxima of the speed reduction
};

template <typename T>
__device__ __forceinline__ void load_state(const Par<T> &P, const T *__restrict__ fs, int d,
                                           int side, int c, T W[NV])
{
#pragma unroll
    for (int q = 0; q < NV; ++q)
        W[q] = __builtin_nontemporal_load(&fs[(size_t)((d * 2 + side) * NV + q) * P.n + c]);
}

// Faces of one direction: slot s of the x pass is row s / (MTX+1), face
// s % (MTX+1) of that row (its right cell is tile column s % (MTX+1)); slot s
// of the y pass is column s % MTX, face s / MTX of that column.
template <int D, typename T>
__device__ __forceinline__ void sweep_pass(const Par<T> &P, const T *__restrict__ fs, int i, int j,
                                           int k, int tx, int ty, SweepSmem<T> &sm, T dF[NV])
{
    constexpr int NS = D == 0 ? (MTX + 1) * MTY : MTX * (MTY + 1);
    const int lo = D == 0 ? ty * (MTX + 1) + tx : ty * MTX + tx;        // the cell's lower face
    const int hi = D == 0 ? lo + 1 : lo + MTX;                         // its upper face
    const int c = cell(P.nx, P.ny, P.nz, i, j, k);
    {
        T W[NV];
        load_state(P, fs, D, 1, c, W);              // right state of the lower face
#pragma unroll
        for (int q = 0; q < NV; ++q) sm.st[1][q][lo] = W[q];
        load_state(P, fs, D, 0, c, W);              // left state of the upper face
#pragma unroll
        for (int q = 0; q < NV; ++q) sm.st[0][q][hi] = W[q];
        // the halo cells below the first and above the last cell of the row
        const int edge = D == 0 ? tx : ty;
        if (edge == 0) {
            load_state(P, fs, D, 0, cell(P.nx, P.ny, P.nz, i - (D == 0), j - (D == 1), k), W);
#pragma unroll
            for (int q = 0; q < NV; ++q) sm.st[0][q][lo] = W[q];
        }
        if (edge == (D == 0 ? MTX : MTY) - 1) {
            load_state(P, fs, D, 1, cell(P.nx, P.ny, P.nz, i + (D == 0), j + (D == 1), k), W);
#pragma unroll
            for (int q = 0; q < NV; ++q) sm.st[1][q][hi] = W[q];
        }
    }
    __syncthreads();
    for (int t = threadIdx.x; t < NS; t += MT) {
        T WL[NV], WR[NV], F[NV];
#pragma unroll
        for (int q = 0; q < NV; ++q) { WL[q] = sm.st[0][q][t]; WR[q] = sm.st[1][q][t]; }
        face_flux<D>(P, WL, WR, F);
#pragma unroll
        for (int q = 0; q < NV; ++q) sm.st[0][q][t] = F[q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NV; ++q) dF[q] = sm.st[0][q][hi] - sm.st[0][q][lo];
    __syncthreads();
}

// two waves per SIMD: the FP64 sweep sits at the 256-register limit
template <typename T>
__global__ __launch_bounds__(MT) __attribute__((amdgpu_waves_per_eu(2)))
void k_sweep(Par<T> P, const T *__restrict__ dyn,
                                              const T *__restrict__ u, const T *__restrict__ fs,
                                              T *__restrict__ out, int ntx, int nty, int zlen,
                                              int nitem, int per_xcd,
                                              unsigned long long *__restrict__ acc)
{
    __shared__ SweepSmem<T> sm;
    take_dynamic(P, dyn);
    // workgroups are dealt to the eight XCDs in turn: give each XCD a
    // contiguous range of work items, so that neighbouring tiles share its L2
    const int b = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (b >= nitem) return;
    const int bx = b % ntx, br = b / ntx;
    const int by = br % nty, bz = br / nty;
    const int tx = threadIdx.x % MTX, ty = threadIdx.x / MTX;
    const int i = bx * MTX + tx, j = by * MTY + ty;
    const bool own = i < P.nx && j < P.ny;
    const int k0 = bz * zlen, k1 = min(k0 + zlen, P.nz);

    // flux through the z face below the first plane
    T Flo[NV];
    {
        T WL[NV], WR[NV];
        load_state(P, fs, 2, 0, cell(P.nx, P.ny, P.nz, i, j, k0 - 1), WL);
        load_state(P, fs, 2, 1, cell(P.nx, P.ny, P.nz, i, j, k0), WR);
        face_flux<2>(P, WL, WR, Flo);
    }
    double smax = 0.0, dmax = 0.0;
    for (int k = k0; k < k1; ++k) {
        T dFx[NV], dFy[NV];
        sweep_pass<0>(P, fs, i, j, k, tx, ty, sm, dFx);
        sweep_pass<1>(P, fs, i, j, k, tx, ty, sm, dFy);
        T Fhi[NV];
        {
            T WL[NV], WR[NV];
            load_state(P, fs, 2, 0, cell(P.nx, P.ny, P.nz, i, j, k), WL);
            load_state(P, fs, 2, 1, cell(P.nx, P.ny, P.nz, i, j, k + 1), WR);
            face_flux<2>(P, WL, WR, Fhi);
        }
        if (own) {
            const int c = (k * P.ny + j) * P.nx + i;
            T U[NV];
#pragma unroll
            for (int q = 0; q < NV; ++q) {
                const T dFz = Fhi[q] - Flo[q];
                T v = u[(size_t)q * P.n + c] - P.c * ((dFx[q] + dFy[q]) + dFz);
                if (q == 8) v *= P.damp;
                __builtin_nontemporal_store(v, &out[(size_t)q * P.n + c]);
                U[q] = v;
            }
            if (acc) {
                T W[NV];
                to_prim<true>(P, U, W);
                double sum = 0.0;
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    const double v = (double)fabs(W[1 + d]) + (double)fast_speed<true>(P, W, W[5 + d]);
                    sum += v;
                    dmax = fmax(dmax, v);
                }
                smax = fmax(smax, sum);
            }
        }
#pragma unroll
        for (int q = 0; q < NV; ++q) Flo[q] = Fhi[q];
    }
    if (!acc) return;
    // block maxima: wave maxima by shuffles, then the first wave over the waves
    for (int o = 32; o > 0; o >>= 1) {
        smax = fmax(smax, __shfl_xor(smax, o));
        dmax = fmax(dmax, __shfl_xor(dmax, o));
    }
    const int w = threadIdx.x / 64;
    if ((threadIdx.x & 63) == 0) { sm.red[0][w] = smax; sm.red[1][w] = dmax; }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int q = 1; q < MT / 64; ++q) {
            smax = fmax(smax, sm.red[0][q]);
            dmax = fmax(dmax, sm.red[1][q]);
        }
        atomicMax(&acc[0], (unsigned long long)__double_as_longlong(smax));
        atomicMax(&acc[1], (unsigned long long)__double_as_longlong(dmax));
    }
}

// ------------------------------------------------------------ one launch (FP64)

// dt and ch of a step: the host's values, or device scalars where they are
// given.
struct Dynamic {
    const double *dt_dev, *ch_dev;
    double dx, alpha;
};

// A value that every lane holds, moved to scalar registers.
__device__ __forceinline__ double uniform(double v)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const unsigned lo = __builtin_amdgcn_readfirstlane((int)(unsigned)b);
    const unsigned hi = __builtin_amdgcn_readfirstlane((int)(unsigned)(b >> 32));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// The time-dependent parameters of a step whose dt or ch come from the device.
template <typename T>
__device__ __forceinline__ void take_scalars(Par<T> &P, const Dynamic &D, double dt, double ch)
{
    if (!D.dt_dev && !D.ch_dev) return;
    if (D.dt_dev) dt = *D.dt_dev;
    if (D.ch_dev) ch = *D.ch_dev;
    P.h = uniform(T(dt / (2.0 * D.dx)));
    P.c = uniform(T(dt / D.dx));
    P.ch = uniform(T(ch));
    P.ch2 = uniform(T(ch * ch));
    P.ich2 = uniform(T(1.0 / (2.0 * ch)));
    P.damp = uniform(T(exp(-D.alpha * ch * dt / D.dx)));
}

// GLM + HLLD flux through a face, states and flux rotated to its frame:
// (rho, u_n, u_t1, u_t2, p, B_n, B_t1, B_t2, psi) and the fluxes of
// (rho, m_n, m_t1, m_t2, E, B_n, B_t1, B_t2, psi).
// The flux of every region is the physical flux of the state the face lies in
// -- K itself, K* or K** on the side K of the contact -- with the normal
// velocity S_M and total pressure p_T* of the fan (u_K and p_TK outside it):
// F_K + S_K (U*_K - U_K) + S*_K (U**_K - U*_K) collapses to it by the jump
// conditions, so neither side's conserved vector nor flux is formed. In the
// degenerate case, whose star field keeps the side's tangential values, the
// induction flux keeps u_K instead of S_M on them, as the sum above does.
// Products and sums are fused as written, so that all inlined copies give the
// same bits.
template <typename T>
__device__ __forceinline__ void glm_hlld(const Par<T> &P, const T L[NV], const T R[NV], T F[NV])
{
#pragma clang fp contract(off)
    const T half = T(0.5);
    const T Bn = fma(-(R[8] - L[8]), P.ich2, half * (L[5] + R[5]));
    F[5] = fma(-half * P.ch, R[5] - L[5], half * (L[8] + R[8]));
    F[8] = P.ch2 * Bn;
    const T Bn2 = Bn * Bn;
    // total pressure and fast speed of both sides
    T pT[2], cf[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const T *W = s ? R : L;
        const T B2 = fma(W[7], W[7], fma(W[6], W[6], Bn2));
        pT[s] = fma(half, B2, W[4]);
        const T ir = fast_rcp(W[0]);
        const T a2 = P.gamma * W[4] * ir;
        const T q = fma(B2, ir, a2);
        const T disc = fma(q, q, T(-4) * a2 * (Bn2 * ir));
        cf[s] = hw_sqrt(half * (q + hw_sqrt(disc < T(0) ? T(0) : disc)));
    }
    const T SL = fmin(L[1] - cf[0], R[1] - cf[1]);
    const T SR = fmax(L[1] + cf[0], R[1] + cf[1]);
    const T dL = (SL - L[1]) * L[0], dR = (SR - R[1]) * R[0];
    const T idd = fast_rcp(dR - dL);
    T SM = fma(dR, R[1], fma(-dL, L[1], pT[0] - pT[1])) * idd;
    T pS = fma(dL * dR, R[1] - L[1], fma(dR, pT[0], -(dL * pT[1]))) * idd;

    // K, the side of the contact the face lies on, and O, the other one
    const bool supL = SL >= T(0), supR = SR <= T(0);
    const bool left = supL || (!supR && SM >= T(0));
    const bool sup = supL || supR;
    const T rK = left ? L[0] : R[0], uK = left ? L[1] : R[1];
    const T vK = left ? L[2] : R[2], wK = left ? L[3] : R[3];
    const T pK = left ? L[4] : R[4], pTK = left ? pT[0] : pT[1];
    const T yK = left ? L[6] : R[6], zK = left ? L[7] : R[7];
    const T SK = left ? SL : SR, dK = left ? dL : dR;
    const T uO = left ? R[1] : L[1], vO = left ? R[2] : L[2], wO = left ? R[3] : L[3];
    const T yO = left ? R[6] : L[6], zO = left ? R[7] : L[7];
    const T SO = left ? SR : SL, dO = left ? dR : dL;

    // single-star states of both sides; outside the fan K* is K, selected value by
    // value: the quotients by S_K - u_K give it in exact arithmetic only, and are
    // 0/0 where the fast speed is lost in u_K
    const T SMK = sup ? uK : SM;
    pS = sup ? pTK : pS;
    const T isd = fast_rcp(SK - SMK);
    const T rs = sup ? rK : dK * isd;
    const T ddK = dK * (SK - uK);
    const T denK = fma(dK, SK - SMK, -Bn2);
    const bool badK = sup || fabs(denK) <= T(1e-12) * (ddK + Bn2);
    const T idK = fast_rcp(denK);
    const T tK = badK ? T(0) : Bn * (SMK - uK) * idK;
    const T fK = badK ? T(1) : (ddK - Bn2) * idK;
    const T vs = fma(-yK, tK, vK), ws = fma(-zK, tK, wK), ys = yK * fK, zs = zK * fK;
    const T rO = dO * fast_rcp(SO - SM);
    const T ddO = dO * (SO - uO);
    const T denO = fma(dO, SO - SM, -Bn2);
    const bool badO = fabs(denO) <= T(1e-12) * (ddO + Bn2);
    const T idO = fast_rcp(denO);
    const T tO = badO ? T(0) : Bn * (SM - uO) * idO;
    const T fO = badO ? T(1) : (ddO - Bn2) * idO;
    const T vo = fma(-yO, tO, vO), wo = fma(-zO, tO, wO), yo = yO * fO, zo = zO * fO;

    const T B2K = fma(zK, zK, fma(yK, yK, Bn2));
    const T EK = fma(half, fma(rK, fma(wK, wK, fma(vK, vK, uK * uK)), B2K), pK * P.inv_gm1);
    const T uB = fma(wK, zK, fma(vK, yK, uK * Bn));
    const T uBs = fma(ws, zs, fma(vs, ys, SMK * Bn));
    T E = sup ? EK : isd * fma(Bn, uB - uBs, fma(pS, SMK, fma(SK - uK, EK, -(pTK * uK))));

    // between the Alfven waves: the double-star state
    const T iq = fast_rsqrt(rs), sqK = rs * iq, sqO = hw_sqrt(rO);
    const T sg = left ? T(1) : T(-1);
    // S*_K = S_M -+ |B_n| / sqrt(rho*): the face lies inside it when S*_K has
    // passed it
    const bool dbl = !sup && sg * SM - fabs(Bn) * iq < T(0);
    const T sgn = Bn > T(0) ? sg : (Bn < T(0) ? -sg : T(0));
    const T iss = fast_rcp(sqK + sqO);
    const T sK = sqK * iss, sO = sqO * iss, si = sgn * iss, sp = sgn * (sqK * sO);
    const T vd = fma(si, yo - ys, fma(sO, vo, sK * vs));
    const T wd = fma(si, zo - zs, fma(sO, wo, sK * ws));
    const T yd = fma(sp, vo - vs, fma(sO, ys, sK * yo));
    const T zd = fma(sp, wo - ws, fma(sO, zs, sK * zo));
    const T uBd = fma(wd, zd, fma(vd, yd, SMK * Bn));
    const T v = dbl ? vd : vs, w = dbl ? wd : ws, y = dbl ? yd : ys, z = dbl ? zd : zs;
    const T uBf = dbl ? uBd : uBs;
    E = fma(-(sgn * sqK), uBs - uBf, E);

    const T mass = rs * SMK;
    F[0] = mass;
    F[1] = fma(mass, SMK, pS - Bn2);
    F[2] = fma(mass, v, -(Bn * y));
    F[3] = fma(mass, w, -(Bn * z));
    F[4] = fma(SMK, E + pS, -(Bn * uBf));
    const T du = badK ? uK - SMK : T(0);
    F[6] = fma(du, yK, fma(SMK, y, -(Bn * v)));
    F[7] = fma(du, zK, fma(SMK, z, -(Bn * w)));
}

// Position of natural component q in the frame of a face normal to D
template <int D>
__host__ __device__ constexpr int slot(int q)
{
    return q == 0 || q == 4 || q == 8 ? q : (q < 4 ? 1 + (q - 1 - D + 3) % 3 : 5 + (q - 5 - D + 3) % 3);
}

// A face state after the half step: the conserved values of W +- S/2 plus the
// increment h dU common to the cell's six faces.
template <typename T>
__device__ __forceinline__ void half_step(const Par<T> &P, const T W[NV], const T dU[NV], T Wn[NV])
{
    T U[NV], V[NV];
    to_cons(P, W, U);
#pragma unroll
    for (int q = 0; q < NV; ++q) U[q] = fma(P.h, dU[q], U[q]);
    to_prim<false>(P, U, V);
#pragma unroll
    for (int q = 0; q < NV; ++q) Wn[q] = V[q];
}

template <typename T, int TX, int TY>
struct MhdSmem {
    T w[NV][TY + 4][TX + 4];                 // plane k with its two-deep x-y halo
    T f[NV][TileGeom<TX, TY>::NF];           // a face's right state, then its flux
    double red[2][TileGeom<TX, TY>::NT / 64];
};

// The loads and stores of one cell, plane base and variable stride scalar
template <typename T>
__device__ __forceinline__ void load9(const T *__restrict__ p, int n, uint32_t at, T U[NV])
{
#pragma unroll
    for (int q = 0; q < NV; ++q)
        U[q] = *reinterpret_cast<const T *>(reinterpret_cast<const char *>(p + (size_t)q * n) + at);
}

// One workgroup: a TX x TY column tile and planes [z0, z1), marched as in
// godunov_tile: a ring of columns around the tile holds the predicted states
// its outer faces need; every face is solved once, by the owner of its lower
// cell, which keeps the upper-face states in registers; lower-face states and
// fluxes pass through LDS. Per plane, between three barriers:
//   slopes, half step | face states, z face, update of plane k-1 | x and y
//   faces, plane k+1 staged | (x-y flux divergence, then the next plane)
// Bound by registers: nine FP64 variables leave no room for a second buffer of
// faces or for the column's own plane (it is read back from LDS); two
// workgroups of four waves per CU at 256 registers. With one loop for all
// waves, halo loads held by every thread and the slopes kept from the half step
// to the face states, 70 registers spilled, the prefetched plane among them
// (its whole latency then stood between two barriers), and a step took
// 0.635 ms; with the interior lanes masked one by one, 16 spilled and 0.332 ms.
// 128^3 box, dt and ch on the device: 0.305 ms a step against 0.591 ms for the
// two launches over 54 staged values per cell.
template <typename T, int LIM, int TX, int TY>
__global__ __launch_bounds__(tile_threads(TX, TY))
__attribute__((amdgpu_waves_per_eu(2))) void k_step(
    Par<T> P, Dynamic D, double dt_host, double ch_host, const T *__restrict__ u,
    T *__restrict__ out, int ntx, int nty, int zlen, int nitem, int per_xcd,
    unsigned long long *__restrict__ speed_acc)
{
    using Geo = TileGeom<TX, TY>;
    __shared__ MhdSmem<T, TX, TY> sm;
    // workgroups are dealt to the eight XCDs in turn: give each XCD a
    // contiguous range of work items, so that neighbouring tiles share its L2
    const int item = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (item >= nitem) return;
    take_scalars(P, D, dt_host, ch_host);
    const int bx = item % ntx, br = item / ntx;
    const int x0 = bx * TX, y0 = (br % nty) * TY, z0 = (br / nty) * zlen;
    const int z1 = min(z0 + zlen, P.nz);
    const int tid = threadIdx.x;
    const int ax = min(TX, P.nx - x0), ay = min(TY, P.ny - y0);

    // byte offset in a plane; two wraps cover the stencil's reach of two cells
    // for every extent
    auto place = [&](int i, int j) {
        i = wrap_once(wrap_once(x0 + i, P.nx), P.nx);
        j = wrap_once(wrap_once(y0 + j, P.ny), P.ny);
        return (uint32_t)(j * P.nx + i) * (uint32_t)sizeof(T);
    };
    auto plane = [&](int k) {
        return u + (size_t)wrap_once(wrap_once(k, P.nz), P.nz) * (P.nx * P.ny);
    };
    double smax = 0.0, dmax = 0.0;
    // The tile's waves and the ring's run loops of their own (the branch is the
    // same for a whole wave, and both loops pass the same barriers): the ring
    // has no z face, no update and no second face, and stages the halo instead,
    // so neither side pays registers for what the other one holds.
    if (uniform(tid >> 6) < Geo::NINT / 64) {
        // lanes outside a clipped tile compute on its first column, and neither
        // write nor reduce: what a masked branch may or may not set would keep
        // its registers throughout the branch
        const bool own = tid % TX < ax && tid / TX < ay;
        const bool live = uniform(tid) / TX < ay;
        const int ci = own ? tid % TX : 0, cj = own ? tid / TX : 0;
        const int lx = ci + 2, ly = cj + 2;
        const uint32_t col = place(ci, cj);
        const int xlo = Geo::xface(ci, cj), xhi = Geo::xface(ci + 1, cj);
        const int ylo = Geo::yface(ci, cj), yhi = Geo::yface(ci, cj + 1);
        // planes k-1 and k+1 of the column (plane k is in LDS); zprev the upper
        // z state of plane k-1; up1, up2 the upper x and y states, then fluxes
        T Wm[NV], Wp[NV], zprev[NV], acc[NV], up1[NV], up2[NV];
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            Wm[q] = Wp[q] = zprev[q] = acc[q] = up1[q] = T(0);
            up2[q] = T(0);
        }
        {
            T Ua[NV], Ub[NV], Uc[NV];
            load9(plane(z0 - 2), P.n, col, Ua);
            load9(plane(z0 - 1), P.n, col, Ub);
            load9(plane(z0), P.n, col, Uc);
            to_prim<false>(P, Ua, Wm);
            to_prim<false>(P, Uc, Wp);
            to_prim<false>(P, Ub, Uc);
            if (own) {
#pragma unroll
                for (int q = 0; q < NV; ++q) sm.w[q][ly][lx] = Uc[q];
            }
        }
        __syncthreads();
        for (int k = z0 - 1;; ++k) {
            const bool pre = k < z0, post = k == z1;
            // the column's cell of plane k and its limited slopes along axis d;
            // formed twice, for the half step and for the face states, rather
            // than held (54 registers) in between
            T W0[NV], S[NV], dU[NV];
            auto slopes = [&](int d) {
#pragma unroll
                for (int q = 0; q < NV; ++q) {
                    const T c = W0[q] = sm.w[q][ly][lx];
                    if (d == 0) S[q] = limited_slope<LIM>(c - sm.w[q][ly][lx - 1], sm.w[q][ly][lx + 1] - c);
                    else if (d == 1) S[q] = limited_slope<LIM>(c - sm.w[q][ly - 1][lx], sm.w[q][ly + 1][lx] - c);
                    else S[q] = limited_slope<LIM>(c - Wm[q], Wp[q] - c);
                }
            };
            // ---- the x-y flux divergence of plane k-1; the half step of plane k
            if (live) {
                if (k > z0) {
#pragma unroll
                    for (int q = 0; q < NV; ++q)
                        acc[q] = ((up1[q] - sm.f[q][xlo]) +
                                  (up2[slot<1>(q)] - sm.f[slot<1>(q)][ylo])) + acc[q];
                }
#pragma unroll
                for (int q = 0; q < NV; ++q) dU[q] = T(0);
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    // axis after axis: interleaved they would hold three times
                    // the registers
                    __builtin_amdgcn_sched_barrier(0);
                    slopes(d);
                    T up[NV], dn[NV], Fu[NV], Fd[NV];
                    face_values(P, W0, S, up, dn);
                    if (d == 0) { phys_flux<0>(P, up, Fu); phys_flux<0>(P, dn, Fd); }
                    else if (d == 1) { phys_flux<1>(P, up, Fu); phys_flux<1>(P, dn, Fd); }
                    else { phys_flux<2>(P, up, Fu); phys_flux<2>(P, dn, Fd); }
#pragma unroll
                    for (int q = 0; q < NV; ++q) dU[q] -= Fu[q] - Fd[q];
                }
            }
            __syncthreads();
            if (live) {
                T up[NV], dn[NV];
                slopes(2);
                face_values(P, W0, S, up, dn);
                half_step(P, dn, dU, dn);
                half_step(P, up, dU, up);
                __builtin_amdgcn_sched_barrier(0);
                if (!pre) {
                    // the z face below the plane; completes plane k-1
                    T L[NV], R[NV], F[NV];
#pragma unroll
                    for (int q = 0; q < NV; ++q) {
                        L[slot<2>(q)] = zprev[q];
                        R[slot<2>(q)] = dn[q];
                    }
                    glm_hlld(P, L, R, F);
                    if (k > z0) {
                        T U[NV];
                        load9(plane(k - 1), P.n, col, U);
                        T *o = out + (size_t)(k - 1) * (P.nx * P.ny);
#pragma unroll
                        for (int q = 0; q < NV; ++q) {
                            U[q] = fma(-P.c, acc[q] + F[slot<2>(q)], U[q]);
                            if (q == 8) U[q] *= P.damp;
                        }
                        if (own) {
#pragma unroll
                            for (int q = 0; q < NV; ++q)
                                __builtin_nontemporal_store(
                                    U[q], reinterpret_cast<T *>(
                                              reinterpret_cast<char *>(o + (size_t)q * P.n) + col));
                        }
                        if (speed_acc && own) {
                            T W[NV];
                            to_prim<true>(P, U, W);
                            double sum = 0.0;
#pragma unroll
                            for (int d = 0; d < 3; ++d) {
                                const double v = (double)fabs(W[1 + d]) +
                                                 (double)fast_speed<true>(P, W, W[5 + d]);
                                sum += v;
                                dmax = fmax(dmax, v);
                            }
                            smax = fmax(smax, sum);
                        }
                    }
#pragma unroll
                    for (int q = 0; q < NV; ++q) acc[q] = -F[slot<2>(q)];
                }
#pragma unroll
                for (int q = 0; q < NV; ++q) zprev[q] = up[q];
                __builtin_amdgcn_sched_barrier(0);
                slopes(0);
                face_values(P, W0, S, up1, dn);
                half_step(P, dn, dU, dn);
                if (own) {
#pragma unroll
                    for (int q = 0; q < NV; ++q) sm.f[q][xlo] = dn[q];
                }
                half_step(P, up1, dU, up1);
                __builtin_amdgcn_sched_barrier(0);
                slopes(1);
                face_values(P, W0, S, up, dn);
                half_step(P, dn, dU, dn);
                if (own) {
#pragma unroll
                    for (int q = 0; q < NV; ++q) sm.f[slot<1>(q)][ylo] = dn[q];
                }
                half_step(P, up, dU, up);
#pragma unroll
                for (int q = 0; q < NV; ++q) up2[slot<1>(q)] = up[q];
            }
            if (post) break;
            __syncthreads();

            // ---- the load of plane k+2, in flight through the solves of the
            // cell's upper x and y faces; the column moves up
            T Un[NV], R[NV];
            load9(plane(k + 2), P.n, col, Un);
            if (live && !pre) {
#pragma unroll
                for (int q = 0; q < NV; ++q) R[q] = sm.f[q][xhi];
                glm_hlld(P, up1, R, up1);
                if (own) {
#pragma unroll
                    for (int q = 0; q < NV; ++q) sm.f[q][xhi] = up1[q];
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int q = 0; q < NV; ++q) R[q] = sm.f[q][yhi];
                glm_hlld(P, up2, R, up2);
                if (own) {
#pragma unroll
                    for (int q = 0; q < NV; ++q) sm.f[q][yhi] = up2[q];
                }
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = 0; q < NV; ++q) Wm[q] = sm.w[q][ly][lx];
            if (own) {
#pragma unroll
                for (int q = 0; q < NV; ++q) sm.w[q][ly][lx] = Wp[q];
            }
            to_prim<false>(P, Un, Wp);
            __syncthreads();
        }
    } else {
        // ---- a ring column: its one face with the tile (an x face for the
        // left and right columns, a y face for the bottom and top rows), whose
        // left (lower) state the left and bottom columns hold and solve; and
        // the halo cell behind it, the first four lanes a corner cell too
        const int r = tid - Geo::NINT;
        const bool own = r < 2 * (ax + ay);
        const bool ring_x = r >= 2 * ax;
        const int e = ring_x ? r - 2 * ax : r;
        const bool far = e >= (ring_x ? ay : ax);             // right or top
        const int at = far ? e - (ring_x ? ay : ax) : e;
        const int ci = ring_x ? (far ? ax : -1) : at, cj = ring_x ? at : (far ? ay : -1);
        const int hi = ring_x ? (far ? ax + 1 : -2) : at, hj = ring_x ? at : (far ? ay + 1 : -2);
        const int ki = (r & 1) ? ax : -1, kj = (r & 2) ? ay : -1;
        const bool corner = r < 4;
        const int lx = ci + 2, ly = cj + 2;
        const int dx = ring_x, dy = !ring_x;
        const uint32_t col = own ? place(ci, cj) : 0, hcol = own ? place(hi, hj) : 0;
        const uint32_t kcol = place(ki, kj);
        const int face = ring_x ? Geo::xface(ci + !far, cj) : Geo::yface(ci, cj + !far);
        T Wm[NV], Wp[NV], up1[NV];
#pragma unroll
        for (int q = 0; q < NV; ++q) Wm[q] = Wp[q] = up1[q] = T(0);
        if (own) {
            T Ub[NV], Uc[NV];
            load9(plane(z0 - 1), P.n, col, Ub);
            load9(plane(z0), P.n, col, Uc);
            to_prim<false>(P, Uc, Wp);
            to_prim<false>(P, Ub, Uc);
#pragma unroll
            for (int q = 0; q < NV; ++q) sm.w[q][ly][lx] = Uc[q];
        }
        __syncthreads();
        for (int k = z0 - 1;; ++k) {
            const bool pre = k < z0, post = k == z1;
            const bool active = own && !pre && !post;
            T W0[NV], S[NV], dU[NV];
            if (active) {
#pragma unroll
                for (int q = 0; q < NV; ++q) dU[q] = T(0);
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int q = 0; q < NV; ++q) {
                        const T c = W0[q] = sm.w[q][ly][lx];
                        if (d == 0) S[q] = limited_slope<LIM>(c - sm.w[q][ly][lx - 1], sm.w[q][ly][lx + 1] - c);
                        else if (d == 1) S[q] = limited_slope<LIM>(c - sm.w[q][ly - 1][lx], sm.w[q][ly + 1][lx] - c);
                        else S[q] = limited_slope<LIM>(c - Wm[q], Wp[q] - c);
                    }
                    T up[NV], dn[NV], Fu[NV], Fd[NV];
                    face_values(P, W0, S, up, dn);
                    if (d == 0) { phys_flux<0>(P, up, Fu); phys_flux<0>(P, dn, Fd); }
                    else if (d == 1) { phys_flux<1>(P, up, Fu); phys_flux<1>(P, dn, Fd); }
                    else { phys_flux<2>(P, up, Fu); phys_flux<2>(P, dn, Fd); }
#pragma unroll
                    for (int q = 0; q < NV; ++q) dU[q] -= Fu[q] - Fd[q];
                }
            }
            __syncthreads();
            if (active) {
                T up[NV], dn[NV];
#pragma unroll
                for (int q = 0; q < NV; ++q) {
                    const T c = W0[q] = sm.w[q][ly][lx];
                    S[q] = limited_slope<LIM>(c - sm.w[q][ly - dy][lx - dx], sm.w[q][ly + dy][lx + dx] - c);
                }
                face_values(P, W0, S, up, dn);
#pragma unroll
                for (int q = 0; q < NV; ++q) up[q] = far ? dn[q] : up[q];
                half_step(P, up, dU, up);
#pragma unroll
                for (int q = 0; q < NV; ++q) up1[q] = up[q];
                if (!ring_x) {
#pragma unroll
                    for (int q = 0; q < NV; ++q) up1[slot<1>(q)] = up[q];
                }
                if (far) {
#pragma unroll
                    for (int q = 0; q < NV; ++q) sm.f[q][face] = up1[q];
                }
            }
            if (post) break;
            __syncthreads();

            T Un[NV], Hn[NV], Kn[NV];
            const bool more = own && k + 2 <= z1, halo = own && k + 1 < z1;
            if (more) load9(plane(k + 2), P.n, col, Un);
            if (halo) load9(plane(k + 1), P.n, hcol, Hn);
            if (halo && corner) load9(plane(k + 1), P.n, kcol, Kn);
            if (active && !far) {
                T R[NV];
#pragma unroll
                for (int q = 0; q < NV; ++q) R[q] = sm.f[q][face];
                glm_hlld(P, up1, R, up1);
#pragma unroll
                for (int q = 0; q < NV; ++q) sm.f[q][face] = up1[q];
            }
            if (own) {
#pragma unroll
                for (int q = 0; q < NV; ++q) {
                    Wm[q] = sm.w[q][ly][lx];
                    sm.w[q][ly][lx] = Wp[q];
                }
                if (more) to_prim<false>(P, Un, Wp);
            }
            if (halo) {
                to_prim<false>(P, Hn, W0);
#pragma unroll
                for (int q = 0; q < NV; ++q) sm.w[q][hj + 2][hi + 2] = W0[q];
                if (corner) {
                    to_prim<false>(P, Kn, W0);
#pragma unroll
                    for (int q = 0; q < NV; ++q) sm.w[q][kj + 2][ki + 2] = W0[q];
                }
            }
            __syncthreads();
        }
    }
    if (!speed_acc) return;
    // block maxima: wave maxima by shuffles, then the first wave over the waves
    for (int o = 32; o > 0; o >>= 1) {
        smax = fmax(smax, __shfl_xor(smax, o));
        dmax = fmax(dmax, __shfl_xor(dmax, o));
    }
    const int w = tid / 64;
    if ((tid & 63) == 0) { sm.red[0][w] = smax; sm.red[1][w] = dmax; }
    __syncthreads();
    if (tid == 0) {
        for (int q = 1; q < Geo::NT / 64; ++q) {
            smax = fmax(smax, sm.red[0][q]);
            dmax = fmax(dmax, sm.red[1][q]);
        }
        atomicMax(&speed_acc[0], (unsigned long long)__double_as_longlong(smax));
        atomicMax(&speed_acc[1], (unsigned long long)__double_as_longlong(dmax));
    }
}

// max over cells of sum_d (|u_d| + cf_d) and of max_d (|u_d| + cf_d): block
// maxima through LDS, one atomicMax per block on the bit patterns of the
// non-negative doubles (which order like the values)
template <typename T>
__global__ __launch_bounds__(256) void k_speeds(Par<T> P, const T *__restrict__ u,
                                                unsigned long long *__restrict__ acc)
{
    __shared__ double red[2][256];
    double s = 0.0, m = 0.0;
    for (int c = blockIdx.x * 256 + threadIdx.x; c < P.n; c += gridDim.x * 256) {
        T W[NV];
        load_prim<true>(P, u, c, W);
        double sum = 0.0;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const double v = (double)fabs(W[1 + d]) + (double)fast_speed<true>(P, W, W[5 + d]);
            sum += v;
            m = fmax(m, v);
        }
        s = fmax(s, sum);
    }
    red[0][threadIdx.x] = s;
    red[1][threadIdx.x] = m;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            red[0][threadIdx.x] = fmax(red[0][threadIdx.x], red[0][threadIdx.x + w]);
            red[1][threadIdx.x] = fmax(red[1][threadIdx.x], red[1][threadIdx.x + w]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        atomicMax(&acc[0], (unsigned long long)__double_as_longlong(red[0][0]));
        atomicMax(&acc[1], (unsigned long long)__double_as_longlong(red[1][0]));
    }
}

// dt = cfl dx / smax and ch = max speed into device scalars; resets the
// accumulators for the next reduction
__global__ void k_speeds_finish(double cfl, double dx, unsigned long long *acc, double *dt_out,
                                double *ch_out)
{
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    const double s = __longlong_as_double((long long)atomicExch(&acc[0], 0ull));
    const double m = __longlong_as_double((long long)atomicExch(&acc[1], 0ull));
    if (dt_out) *dt_out = cfl * dx / s;
    if (ch_out) *ch_out = m;
}

// dt and ch from device scalars (or the host values) -> the dynamic
// parameters (h, c, ch, ch^2, damp) of the step (one thread)
template <typename T>
__global__ void k_params(T *dyn, const double *dt_dev, const double *ch_dev, double dt_host,
                         double ch_host, double dx, double alpha)
{
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    const double dt = dt_dev ? *dt_dev : dt_host;
    const double ch = ch_dev ? *ch_dev : ch_host;
    dyn[0] = (T)(dt / (2.0 * dx));
    dyn[1] = (T)(dt / dx);
    dyn[2] = (T)ch;
    dyn[3] = (T)(ch * ch);
    dyn[4] = (T)exp(-alpha * ch * dt / dx);
}

}  // namespace mhd

size_t mhd_scratch_bytes(int dtype, int nx, int ny, int nz)
{
    // single precision: six face states of 9 values per cell, plus the step's
    // device-side parameters
    return dtype == 0 ? 0 : 6 * 9 * (size_t)nx * ny * nz * sizeof(float) + 512;
}

template <typename T, int LIM, int TX, int TY>
static void launch_mhd_tiles(const mhd::Par<T> &P, const mhd::Dynamic &D, const MhdScalars &sc,
                             const void *u_in, void *u_out, unsigned long long *acc, int num_cus,
                             hipStream_t st)
{
    const int ntx = (P.nx + TX - 1) / TX, nty = (P.ny + TY - 1) / TY;
    // z-ranges: as many as the chip holds workgroups, as long as that leaves
    // four planes to a range (a range recomputes the plane below it and the
    // plane above it). Shorter ranges, down to one plane, where all of them find a
    // CU of their own: there a step takes the time of one range, 6 to 7 us a plane
    // (16^3 box with MC limiter: 43 us in ranges of four planes, 21 us in ranges
    // of one; 32^3: 44 and 22 us; 64^3, whose ranges of one to three planes share
    // CUs: 67 us in ranges of four, 63 to 85 in shorter ones).
    const int resident = 2 * num_cus, ntiles = ntx * nty;
    int nseg = std::max(1, resident / ntiles);
    nseg = std::min(nseg, (P.nz + 3) / 4);
    int zlen = (P.nz + nseg - 1) / nseg;
    for (int z = std::min(zlen - 1, 3); z >= 1 && ntiles * ((P.nz + z - 1) / z) <= num_cus; --z)
        zlen = z;
    nseg = (P.nz + zlen - 1) / zlen;
    const int nitem = ntiles * nseg, per_xcd = (nitem + 7) / 8;
    hipLaunchKernelGGL((mhd::k_step<T, LIM, TX, TY>), dim3(8 * per_xcd), dim3(tile_threads(TX, TY)), 0,
                       st, P, D, sc.dt, sc.ch, (const T *)u_in, (T *)u_out, ntx, nty, zlen, nitem,
                       per_xcd, acc);
}

template <typename T>
static mhd::Par<T> make_par(int nx, int ny, int nz, const MhdScalars &sc)
{
    mhd::Par<T> P{};
    P.nx = nx; P.ny = ny; P.nz = nz; P.n = nx * ny * nz;
    P.gamma = (T)sc.gamma; P.gm1 = (T)(sc.gamma - 1.0); P.inv_gm1 = (T)(1.0 / (sc.gamma - 1.0));
    P.rho_floor = (T)sc.rho_floor; P.p_floor = (T)sc.p_floor;
    P.h = (T)(sc.dt / (2.0 * sc.dx));
    P.c = (T)(sc.dt / sc.dx);
    P.ch = (T)sc.ch; P.ch2 = (T)(sc.ch * sc.ch); P.ich2 = (T)(1.0 / (2.0 * sc.ch));
    P.damp = (T)exp(-sc.alpha * sc.ch * sc.dt / sc.dx);
    return P;
}

static int run_mhd_f64(int limiter, int nx, int ny, int nz, const void *u_in, void *u_out,
                       const MhdScalars &sc, const double *dt_dev, const double *ch_dev, double cfl,
                       double *dt_next, double *ch_next, unsigned long long *acc, int num_cus,
                       hipStream_t st)
{
    const mhd::Par<double> P = make_par<double>(nx, ny, nz, sc);
    const mhd::Dynamic D{ dt_dev, ch_dev, sc.dx, sc.alpha };
    unsigned long long *a = dt_next || ch_next ? acc : nullptr;
    switch (limiter) {
    case 1: launch_mhd_tiles<double, 1, 24, 8>(P, D, sc, u_in, u_out, a, num_cus, st); break;
    case 2: launch_mhd_tiles<double, 2, 24, 8>(P, D, sc, u_in, u_out, a, num_cus, st); break;
    default: launch_mhd_tiles<double, 0, 24, 8>(P, D, sc, u_in, u_out, a, num_cus, st); break;
    }
    if (a)
        hipLaunchKernelGGL(mhd::k_speeds_finish, dim3(1), dim3(64), 0, st, cfl, sc.dx, a, dt_next,
                           ch_next);
    return (int)hipGetLastError();
}

static int run_mhd_f32(int limiter, int nx, int ny, int nz, const void *u_in, void *u_out,
                       const MhdScalars &sc, const double *dt_dev, const double *ch_dev,
                       void *scratch, double cfl, double *dt_next, double *ch_next,
                       unsigned long long *acc, hipStream_t st)
{
    using T = float;
    const mhd::Par<T> P = make_par<T>(nx, ny, nz, sc);
    const size_t n = (size_t)P.n;
    T *fs = (T *)scratch;
    T *dyn = nullptr;
    if (dt_dev || ch_dev) {
        dyn = (T *)(((uintptr_t)(fs + 54 * n) + 255) & ~(uintptr_t)255);
        hipLaunchKernelGGL(mhd::k_params<T>, dim3(1), dim3(64), 0, st, dyn, dt_dev, ch_dev, sc.dt,
                           sc.ch, sc.dx, sc.alpha);
    }
    const T *u = (const T *)u_in;
    T *out = (T *)u_out;
    const dim3 grid((nx + 63) / 64, (ny + 3) / 4, nz), block(256);
    switch (limiter) {
    case 1: hipLaunchKernelGGL((mhd::k_predict<T, 1>), grid, block, 0, st, P, dyn, u, fs); break;
    case 2: hipLaunchKernelGGL((mhd::k_predict<T, 2>), grid, block, 0, st, P, dyn, u, fs); break;
    default: hipLaunchKernelGGL((mhd::k_predict<T, 0>), grid, block, 0, st, P, dyn, u, fs); break;
    }
    // z-ranges: about 1024 work items, at least 2 planes each
    const int ntx = (nx + mhd::MTX - 1) / mhd::MTX, nty = (ny + mhd::MTY - 1) / mhd::MTY;
    int nseg = (1024 + ntx * nty - 1) / (ntx * nty);
    nseg = nseg < 1 ? 1 : (nseg > (nz + 1) / 2 ? (nz + 1) / 2 : nseg);
    const int zlen = (nz + nseg - 1) / nseg;
    nseg = (nz + zlen - 1) / zlen;
    const int nitem = ntx * nty * nseg, per_xcd = (nitem + 7) / 8;
    unsigned long long *a = dt_next || ch_next ? acc : nullptr;
    hipLaunchKernelGGL(mhd::k_sweep<T>, dim3(8 * per_xcd), dim3(mhd::MT), 0, st, P, dyn, u, fs, out,
                       ntx, nty, zlen, nitem, per_xcd, a);
    if (a)
        hipLaunchKernelGGL(mhd::k_speeds_finish, dim3(1), dim3(64), 0, st, cfl, sc.dx, a, dt_next,
                           ch_next);
    return (int)hipGetLastError();
}

int launch_mhd_step(int dtype, int limiter, int nx, int ny, int nz, const void *u_in, void *u_out,
                    const MhdScalars &sc, const double *dt_dev, const double *ch_dev,
                    void *scratch, double cfl, double *dt_next, double *ch_next,
                    unsigned long long *acc, int num_cus, hipStream_t s)
{
    if (dtype == 0)
        return run_mhd_f64(limiter, nx, ny, nz, u_in, u_out, sc, dt_dev, ch_dev, cfl, dt_next,
                           ch_next, acc, num_cus, s);
    return run_mhd_f32(limiter, nx, ny, nz, u_in, u_out, sc, dt_dev, ch_dev, scratch, cfl, dt_next,
                       ch_next, acc, s);
}

template <typename T>
static int run_speeds(int nx, int ny, int nz, const void *u, const MhdScalars &sc, double cfl,
                      double *dt_dev, double *ch_dev, unsigned long long *acc, hipStream_t st)
{
    mhd::Par<T> P{};
    P.nx = nx; P.ny = ny; P.nz = nz; P.n = nx * ny * nz;
    P.gamma = (T)sc.gamma; P.gm1 = (T)(sc.gamma - 1.0); P.inv_gm1 = (T)(1.0 / (sc.gamma - 1.0));
    P.rho_floor = (T)sc.rho_floor; P.p_floor = (T)sc.p_floor;
    int blocks = (P.n + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(mhd::k_speeds<T>, dim3(blocks), dim3(256), 0, st, P, (const T *)u, acc);
    hipLaunchKernelGGL(mhd::k_speeds_finish, dim3(1), dim3(64), 0, st, cfl, sc.dx, acc, dt_dev,
                       ch_dev);
    return (int)hipGetLastError();
}

int launch_mhd_speeds(int dtype, int nx, int ny, int nz, const void *u, const MhdScalars &sc,
                      double cfl, double *dt_dev, double *ch_dev, unsigned long long *acc,
                      hipStream_t s)
{
    if (dtype == 0) return run_speeds<double>(nx, ny, nz, u, sc, cfl, dt_dev, ch_dev, acc, s);
    return run_speeds<float>(nx, ny, nz, u, sc, cfl, dt_dev, ch_dev, acc, s);
}

}  // namespace gd
