// Reverse-mode adjoint of the Godunov step (gfx950, FP64), for a fixed dt.
//
// The step is U -> U' = U - dt/dx sum_faces (signed F), with every face flux
// F(W_L, W_R) a function of the predicted states of its two cells, each of
// which depends on the primitive state of the cell and its limited slopes.
// The adjoint runs the chain backwards in gather form -- every output value
// is a sum written by exactly one thread, in a fixed order, with no atomics
// -- so it is bitwise deterministic. Two kernels share a scratch area over the
// cells whose predicted states the step uses: the extended box [-2, n+2)^3 of a
// ghosted patch, or the periodic box itself, whose neighbours wrap (x fastest):
//   1 march    per 24x8 column tile of predicted cells and z-range: the step's
//              tile march (godunov_tile.h) with the reverse of each face in
//              place of its flux -- slopes, predicted state and face states
//              from the staged primitives, dL/dF = dt/dx (lam_right - lam_left)
//              (+ dL/dbflux on the patch boundary) reversed through the Riemann
//              solver and the face floors by the owner of the face's lower cell
//              -- then per cell the reverse predictor: dL/dW (direct part),
//              dL/dS, and a 2-bit code per slope recording the limiter branch;
//   2 input    per input cell: dL/dW gathered from its own predictor term
//              and the slope adjoints of itself and its neighbours split by
//              the recorded branches, reversed through the primitive
//              conversion, plus the identity term lam_out.
// At kinks (limiter switches, min/max of wave speeds, the HLLC region and the
// floors) the derivative of the branch the forward step takes is used, with
// the forward step's tie rules. Indices are 32-bit: the host rejects boxes
// whose scratch arrays would not fit.
#include "godunov_internal.h"
#include "godunov_math.h"
#include "godunov_tile.h"

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

namespace gd {

namespace adj {

enum { LIM_MINMOD = 0, LIM_MC = 1, LIM_NONE = 2 };
enum { RS_HLLC = 0, RS_HLL = 1 };

// column tile of the march: its columns, then a wave of ring columns
constexpr int CTX = 24, CTY = 8;
using Tile = TileGeom<CTX, CTY>;

struct Geo {
    int nx, ny, nz, ng, periodic;
    int ex, ey, ez;            // scratch box: n + 4 (ghosted) or n (periodic)
    int E;                     // cells of the scratch box
    int lo;                    // first predicted index: -1 (ghosted) or 0
    int px, py, pz;            // predicted extents: n + 2 (ghosted) or n
    int vin;                   // input variable stride
    int gx, gy, gz;            // input extents
    int nint;                  // interior cells
    int ntx, nty, nseg, zlen;  // tiles and z-segments of the march
    int nitem, per_xcd;        // its work items, and items per XCD slice
    double gamma, inv_gm1, rho_floor, p_floor, lam, c;   // lam = dt/(2dx), c = dt/dx
};

// Per-cell records of 20 doubles, stored in blocks of 64 consecutive cells
// with the fields of a block contiguous ([E/64][20][64]): a wavefront reads
// one field of 64 neighbouring cells as one 512-byte segment, and all the
// fields of those cells lie in one 10 KB span. Records are written with
// streaming (non-temporal) stores: the next kernel reads them long after.
constexpr int NF = 20;
// fields: dL/dS at d*5+q, direct dL/dW at 15+q
constexpr int F_SB = 0, F_WD = 15;

__device__ __forceinline__ int rec(int e, int f) { return ((e >> 6) * NF + f) * 64 + (e & 63); }

struct Scratch {
    double *ad;        // adjoint record of each extended cell
    unsigned *code;    // [E] limiter branch per slope, 2 bits at 2(d*5+q)
};

__device__ __forceinline__ int depth_out(int i, int n) { return i < 0 ? -i : (i >= n ? i - n + 1 : 0); }

__device__ __forceinline__ bool is_read(const Geo &g, int i, int j, int k)
{
    int di = depth_out(i, g.nx), dj = depth_out(j, g.ny), dk = depth_out(k, g.nz);
    int nout = (di > 0) + (dj > 0) + (dk > 0);
    if (nout == 0) return true;
    if (nout == 1) return di + dj + dk <= 2;
    if (nout == 2) return di <= 1 && dj <= 1 && dk <= 1;
    return false;
}

__device__ __forceinline__ bool is_predicted(const Geo &g, int i, int j, int k)
{
    return g.periodic ||
           depth_out(i, g.nx) + depth_out(j, g.ny) + depth_out(k, g.nz) <= 1;
}

// i mod n for i in [-3, n+3); the general form only for boxes narrower than 3
__device__ __forceinline__ int wrap(int i, int n)
{
    if (i < 0) i += n;
    else if (i >= n) i -= n;
    if ((unsigned)i >= (unsigned)n) { i %= n; if (i < 0) i += n; }
    return i;
}

// scratch index of cell (i, j, k): the extended box of a ghosted patch, the
// wrapped interior of a periodic box
__device__ __forceinline__ int ext(const Geo &g, int i, int j, int k)
{
    if (g.periodic) {
        i = wrap(i, g.nx); j = wrap(j, g.ny); k = wrap(k, g.nz);
        return (k * g.ny + j) * g.nx + i;
    }
    return ((k + 2) * g.ey + (j + 2)) * g.ex + (i + 2);
}

__device__ __forceinline__ int interior_index(const Geo &g, int i, int j, int k)
{
    return (k * g.ny + j) * g.nx + i;
}

// What decides a branch -- primitives, slopes, face states, wave speeds and S* --
// is computed by the forward step's functions or by its expressions with the
// same products fused, so that near ties the adjoint takes the branch that the
// step took.

// Conserved -> primitive with floors.
__device__ __forceinline__ void to_prim(const Geo &g, const double U[5], double W[5],
                                        double &inv_rho)
{
    const Phys<double> ph{ g.gamma, g.gamma - 1.0, g.inv_gm1, g.rho_floor, g.p_floor };
    int unused = 0;
    prim_from_cons(U, W, inv_rho, ph, unused);
}

// Branch of a limited slope: 0 zero slope, 1 the a-branch, 2 the b-branch,
// 3 the symmetric branch (a+b)/2 or |a+b|/2.
template <int LIM>
__device__ __forceinline__ unsigned slope_branch(double a, double b)
{
    if (LIM == LIM_NONE) return 3u;
    bool same = (a > 0.0 && b > 0.0) || (a < 0.0 && b < 0.0);
    if (!same) return 0u;
    if (LIM == LIM_MINMOD) return fabs(a) <= fabs(b) ? 1u : 2u;
    double m1 = 2.0 * fabs(a), m2 = 2.0 * fabs(b), m3 = 0.5 * fabs(a + b);
    bool first = m1 <= m2;
    double m = first ? m1 : m2;
    if (m <= m3) return first ? 1u : 2u;
    return 3u;
}

// d slope / d a and d slope / d b of a recorded branch
template <int LIM>
__device__ __forceinline__ void branch_partials(unsigned br, double &pa, double &pb)
{
    const double one = LIM == LIM_MC ? 2.0 : 1.0;
    pa = br == 1u ? one : (br == 3u ? 0.5 : 0.0);
    pb = br == 2u ? one : (br == 3u ? 0.5 : 0.0);
}

// ------------------------------------------------------------ Riemann adjoints

// Forward quantities of the HLLC / HLL flux in rotated form, kept for the
// reverse sweep; y = 1 / sqrt(gamma p rho).
struct Fwd {
    double yL, yR, cL, cR, SL, SR;
    bool slL, srL;      // S_L took the left candidate, S_R the left candidate
};

__device__ __forceinline__ void speeds(double g, const double L[5], const double R[5], Fwd &f)
{
#pragma clang fp contract(off)
    const double gl = g * L[4], gr = g * R[4];
    f.yL = fast_rsqrt(gl * L[0]);
    f.yR = fast_rsqrt(gr * R[0]);
    f.cL = gl * f.yL;
    f.cR = gr * f.yR;
    double a = L[1] - f.cL, b = R[1] - f.cR;
    f.slL = a <= b;
    f.SL = f.slL ? a : b;
    double c = L[1] + f.cL, d = R[1] + f.cR;
    f.srL = c >= d;
    f.SR = f.srL ? c : d;
}

__device__ __forceinline__ void speeds_adjoint(double g, const Fwd &f, double SLb, double SRb,
                                               double Lb[5], double Rb[5])
{
    const double sl = f.slL ? SLb : 0.0, sr = f.srL ? SRb : 0.0;
    Lb[1] += sl + sr;
    Rb[1] += (SLb - sl) + (SRb - sr);
    const double hl = 0.5 * (sr - sl), hr = 0.5 * ((SRb - sr) - (SLb - sl));
    // c = sqrt(g p / rho): dc/dp = c / (2p) = g y / 2, dc/drho = -c / (2 rho)
    // = -c^2 y / 2
    Lb[4] += hl * (g * f.yL);
    Lb[0] -= hl * (f.cL * f.cL * f.yL);
    Rb[4] += hr * (g * f.yR);
    Rb[0] -= hr * (f.cR * f.cR * f.yR);
}

// Adjoint of the physical flux and of the conserved vector of a rotated
// primitive state W, accumulated into Wb: Fb . dF/dW + Ub . dU/dW.
__device__ __forceinline__ void flux_cons_adjoint(double inv_gm1, const double W[5],
                                                  const double Fb[5], const double Ub[5],
                                                  double Wb[5])
{
    const double r = W[0], u = W[1], v = W[2], w = W[3], p = W[4];
    const double q2 = u * u + v * v + w * w;
    const double E = p * inv_gm1 + 0.5 * r * q2;
    // energy adjoint collected from F4 = u (E + p) and U4 = E
    double Eb = Fb[4] * u + Ub[4];
    // F0 = r u, F1 = r u^2 + p, F2 = r u v, F3 = r u w, F4 = u (E + p)
    Wb[0] += Fb[0] * u + Fb[1] * u * u + Fb[2] * u * v + Fb[3] * u * w;
    Wb[1] += Fb[0] * r + 2.0 * Fb[1] * r * u + Fb[2] * r * v + Fb[3] * r * w + Fb[4] * (E + p);
    Wb[2] += Fb[2] * r * u;
    Wb[3] += Fb[3] * r * u;
    Wb[4] += Fb[1] + Fb[4] * u;
    // U0 = r, U1 = r u, U2 = r v, U3 = r w
    Wb[0] += Ub[0] + Ub[1] * u + Ub[2] * v + Ub[3] * w;
    Wb[1] += Ub[1] * r;
    Wb[2] += Ub[2] * r;
    Wb[3] += Ub[3] * r;
    // E = p/(g-1) + r q2 / 2
    Wb[0] += Eb * 0.5 * q2;
    Wb[1] += Eb * r * u;
    Wb[2] += Eb * r * v;
    Wb[3] += Eb * r * w;
    Wb[4] += Eb * inv_gm1;
}

__device__ __forceinline__ void phys_flux(double inv_gm1, const double W[5], double F[5],
                                          double U[5])
{
    const double r = W[0], u = W[1], v = W[2], w = W[3], p = W[4];
    const double E = p * inv_gm1 + 0.5 * r * (u * u + v * v + w * w);
    F[0] = r * u; F[1] = r * u * u + p; F[2] = r * u * v; F[3] = r * u * w; F[4] = u * (E + p);
    U[0] = r; U[1] = r * u; U[2] = r * v; U[3] = r * w; U[4] = E;
}

// Reverse of the HLLC flux in the form the step evaluates it: the physical flux
// of the star state of the side K the face lies on, (a S, a S^2 + p*, a S v_K,
// a S w_K, S (E* + p*)) with m = rho_K (S_K - u_K), a = m / (S_K - S), p* =
// p_K + m (S - u_K), E* = ((S_K - u_K) E_K - p_K u_K + p* S) / (S_K - S); S is
// S* in the star regions and u_K in the upwind ones, where the flux is that of K
// and no longer depends on the wave speeds: a is rho_K there, E* is E_K, and 1 /
// (S_K - S) and m stand for nothing and are zero (the quotients would give the
// same in exact arithmetic only, and 0/0 where the sound speed is lost in u_K).
// One path for all regions, a third fewer operations than through
// F_K + S_K (U*_K - U_K), and 4 of 7 reciprocals gone.
__device__ __forceinline__ void hllc_adjoint(double g, double inv_gm1, const double L[5],
                                             const double R[5], const double Fb[5], double Lb[5],
                                             double Rb[5])
{
    Fwd f;
    speeds(g, L, R, f);
    double dL, dR, mL, mR, iden, Sst;
    {
#pragma clang fp contract(off)
        dL = f.SL - L[1];
        dR = f.SR - R[1];
        mL = L[0] * dL;
        mR = R[0] * dR;
        iden = fast_rcp(mL - mR);
        Sst = fma(-mR, R[1], fma(mL, L[1], R[4] - L[4])) * iden;
    }
    const bool supL = f.SL >= 0.0;
    const bool left = supL || Sst >= 0.0;
    const bool star = !supL && (left || !(f.SR <= 0.0));
    const double r = left ? L[0] : R[0], u = left ? L[1] : R[1], v = left ? L[2] : R[2];
    const double w = left ? L[3] : R[3], p = left ? L[4] : R[4];
    const double SK = left ? f.SL : f.SR, m = star ? (left ? mL : mR) : 0.0;
    const double S = star ? Sst : u;
    const double dK = SK - u, t = S - u;
    const double id = star ? fast_rcp(SK - S) : 0.0;
    const double q2 = u * u + v * v + w * w;
    const double EK = p * inv_gm1 + 0.5 * r * q2;
    const double ps = p + m * t;
    const double Es = star ? id * (dK * EK - p * u + ps * S) : EK;
    const double a = star ? m * id : r, mass = a * S;

    // the flux: mass, mass S + p*, mass v, mass w, S (E* + p*)
    const double eb = Fb[4] * S;
    double psb = eb + Fb[1];
    const double massb = Fb[0] + Fb[1] * S + Fb[2] * v + Fb[3] * w;
    double Sb = Fb[4] * (Es + ps) + Fb[1] * mass;
    double vb = Fb[2] * mass, wb = Fb[3] * mass;
    // E* = id N
    const double Nb = eb * id;
    double dKb = Nb * EK;
    const double EKb = star ? Nb * dK : eb;
    psb += Nb * S;
    Sb += Nb * ps;
    // mass = a S, a = m id, id = 1 / (S_K - S)
    const double ab = massb * S;
    Sb += massb * a;
    const double db = -id * (eb * Es + ab * a);
    // p* = p + m (S - u)
    const double mb = ab * id + psb * t;
    Sb += psb * m - db;
    // m = r (S_K - u)
    dKb += mb * r;
    const double h = EKb * r;
    const double rb = EKb * 0.5 * q2 + (star ? mb * dK : ab);
    double ub = h * u - Nb * p - psb * m - dKb;
    const double pb = psb - Nb * u + EKb * inv_gm1;
    vb += h * v;
    wb += h * w;
    ub += star ? 0.0 : Sb;
    const double SKb = star ? db + dKb : 0.0;
    // S* = num / den, num = p_R - p_L + m_L u_L - m_R u_R, den = m_L - m_R
    const double numb = star ? Sb * iden : 0.0, denb = -numb * S;
    const double mLb = numb * L[1] + denb, mRb = -(numb * R[1] + denb);
    Lb[0] = mLb * dL + (left ? rb : 0.0);
    Lb[1] = numb * mL - mLb * L[0] + (left ? ub : 0.0);
    Lb[2] = left ? vb : 0.0;
    Lb[3] = left ? wb : 0.0;
    Lb[4] = (left ? pb : 0.0) - numb;
    Rb[0] = mRb * dR + (left ? 0.0 : rb);
    Rb[1] = (left ? 0.0 : ub) - numb * mR - mRb * R[0];
    Rb[2] = left ? 0.0 : vb;
    Rb[3] = left ? 0.0 : wb;
    Rb[4] = (left ? 0.0 : pb) + numb;
    speeds_adjoint(g, f, mLb * L[0] + (left ? SKb : 0.0), mRb * R[0] + (left ? 0.0 : SKb), Lb, Rb);
}

__device__ __forceinline__ void hll_adjoint(double g, double inv_gm1, const double L[5],
                                            const double R[5], const double Fb[5], double Lb[5],
                                            double Rb[5])
{
    Fwd f;
    speeds(g, L, R, f);
    const double zero[5] = { 0, 0, 0, 0, 0 };
    if (f.SL >= 0.0) { flux_cons_adjoint(inv_gm1, L, Fb, zero, Lb); return; }
    if (f.SR <= 0.0) { flux_cons_adjoint(inv_gm1, R, Fb, zero, Rb); return; }
    double FL[5], FR[5], UL[5], UR[5];
    phys_flux(inv_gm1, L, FL, UL);
    phys_flux(inv_gm1, R, FR, UR);
    const double iD = fast_rcp(f.SR - f.SL);
    double FLb[5], FRb[5], ULb[5], URb[5], SLb = 0.0, SRb = 0.0, Db = 0.0;
    for (int q = 0; q < 5; ++q) {
        double F = (f.SR * FL[q] - f.SL * FR[q] + f.SL * f.SR * (UR[q] - UL[q])) * iD;
        double Gb = Fb[q] * iD;
        Db -= Gb * F;
        FLb[q] = f.SR * Gb;
        FRb[q] = -f.SL * Gb;
        URb[q] = f.SL * f.SR * Gb;
        ULb[q] = -URb[q];
        SRb += Gb * FL[q] + f.SL * Gb * (UR[q] - UL[q]);
        SLb += -Gb * FR[q] + f.SR * Gb * (UR[q] - UL[q]);
    }
    SRb += Db;
    SLb -= Db;
    flux_cons_adjoint(inv_gm1, L, FLb, ULb, Lb);
    flux_cons_adjoint(inv_gm1, R, FRb, URb, Rb);
    speeds_adjoint(g, f, SLb, SRb, Lb, Rb);
}

// Reverse of the flux through a face, all in the rotated order of its axis: from
// dL/dF and the face states before the floors (raised here) to their adjoints.
template <int RS>
__device__ __forceinline__ void face_reverse(const Geo &g, double L[5], double R[5],
                                             const double Fb[5], double Lb[5], double Rb[5])
{
    const bool flL0 = L[0] < g.rho_floor, flL4 = L[4] < g.p_floor;
    const bool flR0 = R[0] < g.rho_floor, flR4 = R[4] < g.p_floor;
    if (flL0) L[0] = g.rho_floor;
    if (flL4) L[4] = g.p_floor;
    if (flR0) R[0] = g.rho_floor;
    if (flR4) R[4] = g.p_floor;
    for (int q = 0; q < 5; ++q) Lb[q] = Rb[q] = 0.0;
    if (RS == RS_HLL) hll_adjoint(g.gamma, g.inv_gm1, L, R, Fb, Lb, Rb);
    else hllc_adjoint(g.gamma, g.inv_gm1, L, R, Fb, Lb, Rb);
    if (flL0) Lb[0] = 0.0;
    if (flL4) Lb[4] = 0.0;
    if (flR0) Rb[0] = 0.0;
    if (flR4) Rb[4] = 0.0;
}

// Position of component q in the rotated order of axis D.
template <int D>
__device__ constexpr int rot(int q) { return q == 0 || q == 4 ? q : 1 + (q - 1 - D + 3) % 3; }

// dL/dbflux of face fi of axis D (of n_d cells), at sheet position `at`, added
// to dL/dF in rotated order. Faces 0 and n of a periodic box are one face: both
// sheets hold its flux.
template <int D>
__device__ __forceinline__ void add_bflux(const Geo &g, const double *__restrict__ lam_bflux, int fi,
                                          int at, double Fb[5])
{
    const int n_d = D == 0 ? g.nx : (D == 1 ? g.ny : g.nz);
    if (!lam_bflux || (fi != 0 && fi != n_d)) return;
    const int sxs = g.nz * g.ny, sys = g.nz * g.nx, szs = g.ny * g.nx;
    const int base = D == 0 ? 0 : (D == 1 ? 10 * sxs : 10 * sxs + 10 * sys);
    const int size = D == 0 ? sxs : (D == 1 ? sys : szs);
    if (fi == 0 || g.periodic)
        for (int q = 0; q < 5; ++q) Fb[rot<D>(q)] += lam_bflux[base + q * size + at];
    if (fi == n_d || g.periodic)
        for (int q = 0; q < 5; ++q) Fb[rot<D>(q)] += lam_bflux[base + 5 * size + q * size + at];
}

// ------------------------------------------------------------ 1: march

// A column of cells: its offsets within a plane of the input and of the
// interior arrays, and how far outside the patch it lies along x and y.
struct Column {
    int in, inner;
    int di, dj;
    bool inside;
};

__device__ __forceinline__ Column make_column(const Geo &g, int i, int j)
{
    Column c;
    if (g.periodic) {
        c.in = c.inner = wrap(j, g.ny) * g.nx + wrap(i, g.nx);
        c.di = c.dj = 0;
        c.inside = true;
        return c;
    }
    c.di = depth_out(i, g.nx);
    c.dj = depth_out(j, g.ny);
    c.inside = c.di == 0 && c.dj == 0;
    // columns more than two cells out are never read (they may lie outside the
    // array)
    c.in = c.di <= 2 && c.dj <= 2 ? (j + g.ng) * g.gx + (i + g.ng) : 0;
    c.inner = c.inside ? j * g.nx + i : 0;
    return c;
}

// whether the step reads the column's cell `dk` planes outside the patch
__device__ __forceinline__ bool reads(const Column &c, int dk)
{
    const int nout = (c.di > 0) + (c.dj > 0) + (dk > 0), sum = c.di + c.dj + dk;
    return nout == 0 || (nout == 1 && sum <= 2) || (nout == 2 && c.di <= 1 && c.dj <= 1 && dk <= 1);
}

struct MarchSmem {
    double w[2][5][CTY + 4][CTX + 4];    // primitives of planes k and k-1, two-deep halo
    // one slot per x and y face of planes k and k-1 (TileGeom::xface / yface, y
    // faces in rotated order): the face's right state, then its adjoint
    double f[2][5][Tile::NF];
    double lam[5][CTY + 2][CTX + 2];     // dL/dU' of plane k and its ring
};

// The march of the step (godunov_tile) with reversed faces. Per plane k:
//   I   slopes, predictor and face states of plane k; the z face below it,
//       which completes the face-state adjoints of plane k-1; the reverse
//       predictor of plane k-1 and its record;
//   II  the plane's x and y faces; plane k+1 staged, plane k+2 and dL/dU' of
//       plane k+1 loaded.
// Two waves per SIMD: the reverse solves need the registers, and the LDS holds
// two workgroups per CU then, so planes and faces have two buffers and no third
// barrier. Bound by the latency of the reverse solves. Slopes are formed twice
// and the reverse predictor goes axis by axis, so that nothing of a plane's
// slopes is held across the z face: held, 72 registers spilled and the kernel
// took 343 us on the 128^3 box, so 268. Before, one kernel wrote slopes and
// predicted states (20 doubles a cell, 116 us) and another read them back (285
// us): an adjoint step 0.56 -> 0.42 ms. Tile waves run unmasked (masked lane by
// lane, 26 registers of the minmod and 64 of the MC variant spilled, now 8 and
// 35): a 112 x 84 x 60 ghosted patch with MC limiter and flux adjoints
// 0.267 -> 0.174 -> 0.157 ms, ten steps of a 128^3 box and their adjoint
// 7.74 -> 5.63 -> 5.36 ms.
template <int LIM, int RS>
__global__ __launch_bounds__(Tile::NT) __attribute__((amdgpu_waves_per_eu(2))) void k_march(
    Geo g, const double *__restrict__ u, const double *__restrict__ lam_out,
    const double *__restrict__ lam_bflux, Scratch s)
{
    __shared__ MarchSmem sm;
    // workgroups are dealt to the eight XCDs in turn: give each XCD a
    // contiguous range of work items, so that neighbouring tiles share its L2
    const int item = (blockIdx.x & 7) * g.per_xcd + (blockIdx.x >> 3);
    if (item >= g.nitem) return;
    const int bx = item % g.ntx, br = item / g.ntx;
    // tiles and z-segments cover the predicted range [lo, lo + p)^3
    const int x0 = bx * CTX + g.lo, y0 = (br % g.nty) * CTY + g.lo;
    const int kb = (br / g.nty) * g.zlen + g.lo, ke = min(kb + g.zlen, g.lo + g.pz);
    const int ax = min(CTX, g.lo + g.px - x0), ay = min(CTY, g.lo + g.py - y0);
    const int tid = threadIdx.x;

    auto depth = [&](int k) { return g.periodic ? 0 : depth_out(k, g.nz); };
    auto load_u = [&](const Column &c, int k, double U[5]) {
        const double *p = u + (g.periodic ? wrap(k, g.nz) : k + g.ng) * (g.gx * g.gy);
        const bool ok = reads(c, depth(k));
        for (int q = 0; q < 5; ++q) U[q] = ok ? p[q * g.vin + c.in] : (q == 0 || q == 4 ? 1.0 : 0.0);
    };
    auto load_lam = [&](const Column &c, int k, double L[5]) {
        const int kk = g.periodic ? wrap(k, g.nz) : k;
        const bool ok = c.inside && kk >= 0 && kk < g.nz;
        const double *p = lam_out + kk * (g.nx * g.ny);
        for (int q = 0; q < 5; ++q) L[q] = ok ? p[q * g.nint + c.inner] : 0.0;
    };

    if (__builtin_amdgcn_readfirstlane(tid >> 6) < Tile::NINT / 64) {
        // ---- the tile's columns
        // lanes outside a clipped tile compute on its first column, and do not
        // write: what a masked branch may or may not set would keep its
        // registers throughout the branch
        const bool own = tid % CTX < ax && tid / CTX < ay;
        const bool live = __builtin_amdgcn_readfirstlane(tid) / CTX < ay;
        const int ci = own ? tid % CTX : 0, cj = own ? tid / CTX : 0;
        const int i = x0 + ci, j = y0 + cj, lx = ci + 2, ly = cj + 2;
        const Column c = make_column(g, i, j);
        const int xlo = Tile::xface(ci, cj), xhi = Tile::xface(ci + 1, cj);
        const int ylo = Tile::yface(ci, cj), yhi = Tile::yface(ci, cj + 1);
        // whether the column's upper x and y faces and its z faces exist (at
        // the planes, or below the planes, that do)
        const bool in_i = g.periodic || c.di == 0, in_j = g.periodic || c.dj == 0;
        const bool has_x = in_j && i + 1 >= 0 && i + 1 <= g.nx;
        const bool has_y = in_i && j + 1 >= 0 && j + 1 <= g.ny;
        const bool has_z = in_i && in_j;

        // planes k-2 and k+1 of the column; the upper z state of plane k-1 and
        // the adjoint of its lower z face's right state; the upper x and y
        // states, then (after the solves) their adjoints; dL/dU' of plane k
        double Wmm[5], Wp[5], zprev[5], zlo[5], up1[5], up2[5], lam0[5];
        for (int q = 0; q < 5; ++q) zprev[q] = zlo[q] = up1[q] = up2[q] = Wmm[q] = Wp[q] = lam0[q] = 0.0;
        double ir;
        {
            double Ua[5], Ub[5], Uc[5];
            load_u(c, kb - 2, Ua);
            load_u(c, kb - 1, Ub);
            load_u(c, kb, Uc);
            load_lam(c, kb - 1, lam0);
            to_prim(g, Uc, Wp, ir);
            to_prim(g, Ub, Uc, ir);
            to_prim(g, Ua, Ub, ir);
            if (own) {
                for (int q = 0; q < 5; ++q) {
                    sm.w[0][q][ly][lx] = Uc[q];
                    sm.w[1][q][ly][lx] = Ub[q];   // plane kb-2: the z slopes of kb-1
                }
            }
        }
        __syncthreads();
        int b = 0;
        for (int k = kb - 1;; ++k, b ^= 1) {
            const bool inner = k >= kb && k < ke;
            // ---- I
            // dL/dF of the z face below the plane, from dL/dU' of plane k-1
            // (still in LDS) and of plane k
            double Fz[5], nx1[5], nx2[5], zm[5], zp[5];
            for (int q = 0; q < 5; ++q) Fz[q] = zm[q] = zp[q] = nx1[q] = nx2[q] = 0.0;
            for (int q = 0; q < 5; ++q)
                Fz[rot<2>(q)] = g.c * lam0[q] - g.c * sm.lam[q][cj + 1][ci + 1];
            if (own) {
                for (int q = 0; q < 5; ++q) sm.lam[q][cj + 1][ci + 1] = lam0[q];
            }
            if (live && (g.periodic || c.di + c.dj + depth(k) <= 1)) {
                double W[5], Sx[5], Sy[5], Sz[5], Ws[5];
                for (int q = 0; q < 5; ++q) {
                    const double w = W[q] = sm.w[b][q][ly][lx];
                    Sx[q] = limited_slope<LIM>(w - sm.w[b][q][ly][lx - 1], sm.w[b][q][ly][lx + 1] - w);
                    Sy[q] = limited_slope<LIM>(w - sm.w[b][q][ly - 1][lx], sm.w[b][q][ly + 1][lx] - w);
                    Sz[q] = limited_slope<LIM>(w - sm.w[b ^ 1][q][ly][lx], Wp[q] - w);
                }
                predictor(W, fast_rcp(W[0]), Sx, Sy, Sz, g.lam, g.gamma, Ws);
                for (int q = 0; q < 5; ++q) {
                    zm[q] = Ws[q] - 0.5 * Sz[q];
                    zp[q] = Ws[q] + 0.5 * Sz[q];
                    nx1[q] = Ws[q] + 0.5 * Sx[q];
                    nx2[yslot(q)] = Ws[q] + 0.5 * Sy[q];
                }
                if (own && inner) {
                    for (int q = 0; q < 5; ++q) {
                        sm.f[b][q][xlo] = Ws[q] - 0.5 * Sx[q];
                        sm.f[b][yslot(q)][ylo] = Ws[q] - 0.5 * Sy[q];
                    }
                }
            }
            // the z face below the plane
            double zl[5], zr[5];
            for (int q = 0; q < 5; ++q) zl[q] = zr[q] = 0.0;
            __builtin_amdgcn_sched_barrier(0);
            if (live && has_z && k >= kb && (g.periodic || (k >= 0 && k <= g.nz))) {
                double L[5], R[5], Lb[5], Rb[5];
                for (int q = 0; q < 5; ++q) {
                    L[rot<2>(q)] = zprev[q];
                    R[rot<2>(q)] = zm[q];
                }
                add_bflux<2>(g, lam_bflux, k, j * g.nx + i, Fz);
                face_reverse<RS>(g, L, R, Fz, Lb, Rb);
                for (int q = 0; q < 5; ++q) {
                    zl[q] = Lb[rot<2>(q)];
                    zr[q] = Rb[rot<2>(q)];
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            if (live && k > kb && (g.periodic || c.di + c.dj + depth(k - 1) <= 1)) {
                // the adjoints of plane k-1's face states: the left state of an
                // upper face is W* + S/2, the right state of a lower one W* - S/2
                const int e = ext(g, i, j, k - 1);
                double Wsb[5], W[5];
                for (int q = 0; q < 5; ++q) {
                    Wsb[q] = ((up1[q] + sm.f[b ^ 1][q][xlo]) +
                              (up2[yslot(q)] + sm.f[b ^ 1][yslot(q)][ylo])) + (zl[q] + zlo[q]);
                    W[q] = sm.w[b ^ 1][q][ly][lx];
                }
                // reverse of the predictor, axis by axis:
                //   rho* = rho - lam (sum_d u_d S_d,rho + rho divu)
                //   u_m* = u_m - lam (sum_d u_d S_d,m + S_m,p / rho)
                //   p*   = p - lam (sum_d u_d S_d,p + gamma p divu)
                const double inv_rho = fast_rcp(W[0]), lam = g.lam;
                const double divub = -lam * (Wsb[0] * W[0] + g.gamma * Wsb[4] * W[4]);
                double Wb0 = Wsb[0], Wb4 = Wsb[4];
                unsigned code = 0u;
                for (int d = 0; d < 3; ++d) {
                    __builtin_amdgcn_sched_barrier(0);
                    double S[5], Sb[5], dot = 0.0;
                    for (int q = 0; q < 5; ++q) {
                        const double w = W[q];
                        const double a = w - (d == 0 ? sm.w[b ^ 1][q][ly][lx - 1]
                                                     : (d == 1 ? sm.w[b ^ 1][q][ly - 1][lx] : Wmm[q]));
                        const double h = (d == 0 ? sm.w[b ^ 1][q][ly][lx + 1]
                                                 : (d == 1 ? sm.w[b ^ 1][q][ly + 1][lx]
                                                           : sm.w[b][q][ly][lx])) - w;
                        S[q] = limited_slope<LIM>(a, h);
                        code |= slope_branch<LIM>(a, h) << (2 * (d * 5 + q));
                        const double vl = d == 0 ? up1[q] : (d == 1 ? up2[yslot(q)] : zl[q]);
                        const double vr = d == 0 ? sm.f[b ^ 1][q][xlo]
                                                 : (d == 1 ? sm.f[b ^ 1][yslot(q)][ylo] : zlo[q]);
                        Sb[q] = (0.5 * vl - 0.5 * vr) - lam * Wsb[q] * W[1 + d];
                        dot += Wsb[q] * S[q];
                    }
                    Sb[4] -= lam * Wsb[1 + d] * inv_rho;
                    Sb[1 + d] += divub;
                    Wb0 += lam * (Wsb[1 + d] * S[4] * inv_rho * inv_rho - Wsb[0] * S[1 + d]);
                    Wb4 -= lam * g.gamma * Wsb[4] * S[1 + d];
                    const double wd = Wsb[1 + d] - lam * dot;
                    if (own) {
                        for (int q = 0; q < 5; ++q)
                            __builtin_nontemporal_store(Sb[q], &s.ad[rec(e, F_SB + d * 5 + q)]);
                        __builtin_nontemporal_store(wd, &s.ad[rec(e, F_WD + 1 + d)]);
                    }
                }
                if (own) {
                    __builtin_nontemporal_store(Wb0, &s.ad[rec(e, F_WD)]);
                    __builtin_nontemporal_store(Wb4, &s.ad[rec(e, F_WD + 4)]);
                    s.code[e] = code;
                }
            }
            for (int q = 0; q < 5; ++q) {
                up1[q] = nx1[q];
                up2[q] = nx2[q];
            }
            for (int q = 0; q < 5; ++q) {
                zlo[q] = zr[q];
                zprev[q] = zp[q];
            }
            if (k == ke) break;
            __syncthreads();

            // ---- II
            double Un[5], lamn[5];
            load_u(c, k + 2, Un);
            load_lam(c, k + 1, lamn);
            if (live && inner) {
                // a face between cells that are not both there has no adjoint
                const bool at_k = g.periodic || (k >= 0 && k < g.nz);
                double R[5], Fb[5], Lb[5], Rb[5];
                for (int q = 0; q < 5; ++q) Lb[q] = Rb[q] = 0.0;
                if (has_x && at_k) {
                    for (int q = 0; q < 5; ++q) {
                        R[q] = sm.f[b][q][xhi];
                        Fb[q] = g.c * sm.lam[q][cj + 1][ci + 2] - g.c * lam0[q];
                    }
                    add_bflux<0>(g, lam_bflux, i + 1, k * g.ny + j, Fb);
                    face_reverse<RS>(g, up1, R, Fb, Lb, Rb);
                }
                for (int q = 0; q < 5; ++q) up1[q] = Lb[q];
                if (own) {
                    for (int q = 0; q < 5; ++q) sm.f[b][q][xhi] = Rb[q];
                }
                __builtin_amdgcn_sched_barrier(0);
                for (int q = 0; q < 5; ++q) Lb[q] = Rb[q] = 0.0;
                if (has_y && at_k) {
                    for (int q = 0; q < 5; ++q) {
                        R[q] = sm.f[b][q][yhi];
                        Fb[yslot(q)] = g.c * sm.lam[q][cj + 2][ci + 1] - g.c * lam0[q];
                    }
                    add_bflux<1>(g, lam_bflux, j + 1, k * g.nx + i, Fb);
                    face_reverse<RS>(g, up2, R, Fb, Lb, Rb);
                }
                for (int q = 0; q < 5; ++q) up2[q] = Lb[q];
                if (own) {
                    for (int q = 0; q < 5; ++q) sm.f[b][q][yhi] = Rb[q];
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            // the column moves up
            for (int q = 0; q < 5; ++q) {
                Wmm[q] = sm.w[b ^ 1][q][ly][lx];
                lam0[q] = lamn[q];
            }
            if (own) {
                for (int q = 0; q < 5; ++q) sm.w[b ^ 1][q][ly][lx] = Wp[q];
            }
            to_prim(g, Un, Wp, ir);
            __syncthreads();
        }
    } else {
        // ---- a ring column: the state its face with the tile needs (the left
        // and bottom columns hold the face's left state and reverse it), dL/dU'
        // of its cell, and the primitives of its cell and the halo cell behind
        // it, the first four lanes of a corner cell too
        const int r = tid - Tile::NINT;
        const bool own = r < 2 * (ax + ay);
        const bool ring_x = r >= 2 * ax;
        const int e = ring_x ? r - 2 * ax : r;
        const bool far = e >= (ring_x ? ay : ax);             // right or top
        const int at = far ? e - (ring_x ? ay : ax) : e;
        const int ci = ring_x ? (far ? ax : -1) : at, cj = ring_x ? at : (far ? ay : -1);
        const int hi = ring_x ? (far ? ax + 1 : -2) : at, hj = ring_x ? at : (far ? ay + 1 : -2);
        const int ki = (r & 1) ? ax : -1, kj = (r & 2) ? ay : -1;
        const bool corner = r < 4;
        const int i = x0 + ci, j = y0 + cj, lx = ci + 2, ly = cj + 2;
        const Column c = make_column(g, i, j);
        const Column ch = make_column(g, x0 + hi, y0 + hj), ck = make_column(g, x0 + ki, y0 + kj);
        const int face = ring_x ? Tile::xface(ci + !far, cj) : Tile::yface(ci, cj + !far);
        // the face's index along its axis, and whether it exists
        const int fi = (ring_x ? i : j) + !far;
        const bool has = own && fi >= 0 && fi <= (ring_x ? g.nx : g.ny) &&
                         (g.periodic || (ring_x ? c.dj : c.di) == 0);
        const double side = far ? -0.5 : 0.5;

        double Wm[5], Wp[5], up1[5], lam0[5], ir;
        for (int q = 0; q < 5; ++q) Wm[q] = Wp[q] = up1[q] = lam0[q] = 0.0;
        if (own) {
            double Ub[5], Uc[5];
            load_u(c, kb - 1, Ub);
            load_u(c, kb, Uc);
            load_lam(c, kb - 1, lam0);
            to_prim(g, Uc, Wp, ir);
            to_prim(g, Ub, Uc, ir);
            for (int q = 0; q < 5; ++q) sm.w[0][q][ly][lx] = Uc[q];
        }
        __syncthreads();
        int b = 0;
        for (int k = kb - 1;; ++k, b ^= 1) {
            const bool inner = k >= kb && k < ke;
            const bool at_k = g.periodic || (k >= 0 && k < g.nz);
            // ---- I
            if (own && inner) {
                if (has && at_k) {
                    double W[5], Sx[5], Sy[5], Sz[5], Ws[5];
                    for (int q = 0; q < 5; ++q) {
                        const double w = W[q] = sm.w[b][q][ly][lx];
                        Sx[q] = limited_slope<LIM>(w - sm.w[b][q][ly][lx - 1],
                                                   sm.w[b][q][ly][lx + 1] - w);
                        Sy[q] = limited_slope<LIM>(w - sm.w[b][q][ly - 1][lx],
                                                   sm.w[b][q][ly + 1][lx] - w);
                        Sz[q] = limited_slope<LIM>(w - Wm[q], Wp[q] - w);
                    }
                    predictor(W, fast_rcp(W[0]), Sx, Sy, Sz, g.lam, g.gamma, Ws);
                    double st[5];
                    for (int q = 0; q < 5; ++q) st[q] = Ws[q] + side * (ring_x ? Sx[q] : Sy[q]);
                    for (int q = 0; q < 5; ++q) up1[q] = st[q];
                    if (!ring_x)
                        for (int q = 0; q < 5; ++q) up1[yslot(q)] = st[q];
                    if (far)
                        for (int q = 0; q < 5; ++q) sm.f[b][q][face] = up1[q];
                }
                for (int q = 0; q < 5; ++q) sm.lam[q][cj + 1][ci + 1] = lam0[q];
            }
            if (k == ke) break;
            __syncthreads();

            // ---- II
            double Un[5], Hn[5], Kn[5], lamn[5];
            if (own) {
                load_u(c, k + 2, Un);
                load_lam(c, k + 1, lamn);
                load_u(ch, k + 1, Hn);
                if (corner) load_u(ck, k + 1, Kn);
            }
            if (own && inner && !far) {
                double Lb[5], Rb[5];
                for (int q = 0; q < 5; ++q) Rb[q] = 0.0;
                if (has && at_k) {
                    double R[5], d[5], Fb[5];
                    for (int q = 0; q < 5; ++q) {
                        R[q] = sm.f[b][q][face];
                        d[q] = g.c * sm.lam[q][cj + 1 + !ring_x][ci + 1 + ring_x] - g.c * lam0[q];
                    }
                    for (int q = 0; q < 5; ++q) Fb[q] = d[q];
                    if (ring_x) {
                        add_bflux<0>(g, lam_bflux, fi, k * g.ny + j, Fb);
                    } else {
                        for (int q = 0; q < 5; ++q) Fb[yslot(q)] = d[q];
                        add_bflux<1>(g, lam_bflux, fi, k * g.nx + i, Fb);
                    }
                    face_reverse<RS>(g, up1, R, Fb, Lb, Rb);
                }
                for (int q = 0; q < 5; ++q) sm.f[b][q][face] = Rb[q];
            }
            if (own) {
                double Wh[5];
                for (int q = 0; q < 5; ++q) {
                    Wm[q] = sm.w[b][q][ly][lx];
                    sm.w[b ^ 1][q][ly][lx] = Wp[q];
                    lam0[q] = lamn[q];
                }
                to_prim(g, Un, Wp, ir);
                to_prim(g, Hn, Wh, ir);
                for (int q = 0; q < 5; ++q) sm.w[b ^ 1][q][hj + 2][hi + 2] = Wh[q];
                if (corner) {
                    to_prim(g, Kn, Wh, ir);
                    for (int q = 0; q < 5; ++q) sm.w[b ^ 1][q][kj + 2][ki + 2] = Wh[q];
                }
            }
            __syncthreads();
        }
    }
}

// ------------------------------------------------------------ 2: input

// dL/dW of extended cell (i, j, k): its predictor term and the slope splits
// of itself (a - b) and of its neighbours along each axis, from the branches
// recorded by the march.
template <int LIM>
__device__ __forceinline__ void gather_wbar(const Geo &g, const Scratch &s, int i, int j, int k,
                                            double Wb[5])
{
    for (int q = 0; q < 5; ++q) Wb[q] = 0.0;
    if (!is_read(g, i, j, k)) return;
    const int e = ext(g, i, j, k);
    const bool self = is_predicted(g, i, j, k);
    const unsigned cs = self ? s.code[e] : 0u;
    if (self)
        for (int q = 0; q < 5; ++q) Wb[q] += s.ad[rec(e, F_WD + q)];
    for (int d = 0; d < 3; ++d) {
        const int dm[3] = { -(d == 0), -(d == 1), -(d == 2) };
        const bool lo = is_predicted(g, i + dm[0], j + dm[1], k + dm[2]);
        const bool hi = is_predicted(g, i - dm[0], j - dm[1], k - dm[2]);
        const int el = lo ? ext(g, i + dm[0], j + dm[1], k + dm[2]) : 0;
        const int eh = hi ? ext(g, i - dm[0], j - dm[1], k - dm[2]) : 0;
        const unsigned cl = lo ? s.code[el] : 0u;
        const unsigned ch = hi ? s.code[eh] : 0u;
        for (int q = 0; q < 5; ++q) {
            const int dq = d * 5 + q;
            double v = 0.0, pa, pb;
            if (self) {
                branch_partials<LIM>((cs >> (2 * dq)) & 3u, pa, pb);
                const double x = s.ad[rec(e, F_SB + dq)];
                v += pa * x - pb * x;
            }
            if (lo) {
                branch_partials<LIM>((cl >> (2 * dq)) & 3u, pa, pb);
                v += pb * s.ad[rec(el, F_SB + dq)];
            }
            if (hi) {
                branch_partials<LIM>((ch >> (2 * dq)) & 3u, pa, pb);
                v -= pa * s.ad[rec(eh, F_SB + dq)];
            }
            Wb[q] += v;
        }
    }
}

__device__ __forceinline__ void prim_adjoint(const Geo &g, const double U[5], const double Wb[5],
                                             double Ub[5])
{
    const bool rho_fl = U[0] < g.rho_floor;
    const double rho = rho_fl ? g.rho_floor : U[0];
    const double ir = fast_rcp(rho);
    const double vel[3] = { U[1] * ir, U[2] * ir, U[3] * ir };
    const double p = (g.gamma - 1.0) *
                     fma(-0.5, fma(U[3], vel[2], fma(U[2], vel[1], U[1] * vel[0])), U[4]);
    const double pb = p < g.p_floor ? 0.0 : Wb[4];
    Ub[4] = (g.gamma - 1.0) * pb;
    const double kb = -(g.gamma - 1.0) * pb;
    double rhob = Wb[0];
    for (int d = 0; d < 3; ++d) {
        // kin = sum_d m_d vel_d / 2, vel_d = m_d / rho
        const double vb = Wb[1 + d] + 0.5 * kb * U[1 + d];
        Ub[1 + d] = 0.5 * kb * vel[d] + vb * ir;
        rhob -= vb * vel[d] * ir;
    }
    Ub[0] = rho_fl ? 0.0 : rhob;
}

// One thread per input cell; blocks of 64 x 4 cover x-rows of the input box.
template <int LIM>
__global__ __launch_bounds__(256) void k_input(Geo g, const double *__restrict__ u,
                                               const double *__restrict__ lam_out,
                                               double *__restrict__ lam_in, Scratch s)
{
    const int ci = blockIdx.x * 64 + threadIdx.x % 64;
    const int cj = blockIdx.y * 4 + threadIdx.x / 64;
    const int ck = blockIdx.z;
    if (ci >= g.gx || cj >= g.gy) return;
    const int c = (ck * g.gy + cj) * g.gx + ci;
    const int o = g.periodic ? 0 : g.ng;
    const int i = ci - o, j = cj - o, k = ck - o;
    double Wb[5] = { 0, 0, 0, 0, 0 };
    const bool read = g.periodic ||
                      (i >= -2 && i < g.nx + 2 && j >= -2 && j < g.ny + 2 && k >= -2 &&
                       k < g.nz + 2 && is_read(g, i, j, k));
    if (read) gather_wbar<LIM>(g, s, i, j, k, Wb);
    double Ub[5] = { 0, 0, 0, 0, 0 };
    if (read) {
        double U[5];
        for (int q = 0; q < 5; ++q) U[q] = u[c + q * g.vin];
        prim_adjoint(g, U, Wb, Ub);
    }
    const bool inside = i >= 0 && i < g.nx && j >= 0 && j < g.ny && k >= 0 && k < g.nz;
    const int ii = inside ? interior_index(g, i, j, k) : 0;
    for (int q = 0; q < 5; ++q) {
        double v = Ub[q];
        if (inside) v += lam_out[q * g.nint + ii];
        __builtin_nontemporal_store(v, &lam_in[c + q * g.vin]);
    }
}

}  // namespace adj

size_t adjoint_scratch_bytes(const PatchDesc &P)
{
    const int pad = P.periodic ? 0 : 4;
    const int64_t E = (int64_t)(P.nx + pad) * (P.ny + pad) * (P.nz + pad);
    const int64_t Ep = (E + 63) / 64 * 64;
    // a record of 20 doubles and one branch word per extended cell
    return (size_t)(adj::NF * Ep) * sizeof(double) + (size_t)Ep * sizeof(unsigned);
}

bool adjoint_fits_32bit(const PatchDesc &P)
{
    const int pad = P.periodic ? 0 : 4;
    const int64_t E = (int64_t)(P.nx + pad) * (P.ny + pad) * (P.nz + pad);
    const int64_t g = P.periodic ? 0 : 2 * (int64_t)P.ng;
    const int64_t vin = (P.nx + g) * (P.ny + g) * (P.nz + g);
    return adj::NF * (E + 63) < INT32_MAX && 5 * vin < INT32_MAX;
}

template <int LIM, int RS>
static int run_adjoint(const PatchDesc &P, const double *u_in, const double *lam_out,
                       const double *lam_bflux, double *lam_in, const Scalars &sc, double dt,
                       double *scratch, int num_cus, hipStream_t st)
{
    adj::Geo g{};
    g.nx = P.nx; g.ny = P.ny; g.nz = P.nz; g.ng = P.ng; g.periodic = P.periodic;
    const int pad = P.periodic ? 0 : 4;
    g.ex = P.nx + pad; g.ey = P.ny + pad; g.ez = P.nz + pad;
    g.E = g.ex * g.ey * g.ez;
    g.lo = P.periodic ? 0 : -1;
    g.px = P.periodic ? P.nx : P.nx + 2;
    g.py = P.periodic ? P.ny : P.ny + 2;
    g.pz = P.periodic ? P.nz : P.nz + 2;
    g.gx = P.periodic ? P.nx : P.nx + 2 * P.ng;
    g.gy = P.periodic ? P.ny : P.ny + 2 * P.ng;
    g.gz = P.periodic ? P.nz : P.nz + 2 * P.ng;
    g.vin = g.gx * g.gy * g.gz;
    g.nint = P.nx * P.ny * P.nz;
    g.ntx = (g.px + adj::CTX - 1) / adj::CTX;
    g.nty = (g.py + adj::CTY - 1) / adj::CTY;
    // z-segments: as many as the chip holds workgroups (two per CU), at least 4
    // planes each (a segment predicts the planes below and above it again)
    {
        const int tiles = g.ntx * g.nty;
        int nseg = std::max(1, 2 * num_cus / tiles);
        nseg = std::max(1, std::min(nseg, g.pz / 4));
        g.zlen = (g.pz + nseg - 1) / nseg;
        g.nseg = (g.pz + g.zlen - 1) / g.zlen;
    }
    g.nitem = g.ntx * g.nty * g.nseg;
    g.per_xcd = (g.nitem + 7) / 8;
    g.gamma = sc.gamma; g.inv_gm1 = 1.0 / (sc.gamma - 1.0);
    g.rho_floor = sc.rho_floor; g.p_floor = sc.p_floor;
    g.lam = dt / (2.0 * P.dx);
    g.c = dt / P.dx;
    adj::Scratch s{};
    const size_t Ep = ((size_t)g.E + 63) / 64 * 64;
    s.ad = scratch;
    s.code = reinterpret_cast<unsigned *>(scratch + adj::NF * Ep);
    hipLaunchKernelGGL((adj::k_march<LIM, RS>), dim3(8 * g.per_xcd), dim3(adj::Tile::NT), 0, st, g,
                       u_in, lam_out, lam_bflux, s);
    hipLaunchKernelGGL(adj::k_input<LIM>, dim3((g.gx + 63) / 64, (g.gy + 3) / 4, g.gz), dim3(256),
                       0, st, g, u_in, lam_out, lam_in, s);
    return (int)hipGetLastError();
}

int launch_adjoint(int limiter, int riemann, const PatchDesc &P, const double *u_in,
                   const double *lam_out, const double *lam_bflux, double *lam_in,
                   const Scalars &sc, double dt, double *scratch, int num_cus, hipStream_t s)
{
    if (riemann == 1) {
        if (limiter == 1) return run_adjoint<1, 1>(P, u_in, lam_out, lam_bflux, lam_in, sc, dt, scratch, num_cus, s);
        if (limiter == 2) return run_adjoint<2, 1>(P, u_in, lam_out, lam_bflux, lam_in, sc, dt, scratch, num_cus, s);
        return run_adjoint<0, 1>(P, u_in, lam_out, lam_bflux, lam_in, sc, dt, scratch, num_cus, s);
    }
    if (limiter == 1) return run_adjoint<1, 0>(P, u_in, lam_out, lam_bflux, lam_in, sc, dt, scratch, num_cus, s);
    if (limiter == 2) return run_adjoint<2, 0>(P, u_in, lam_out, lam_bflux, lam_in, sc, dt, scratch, num_cus, s);
    return run_adjoint<0, 0>(P, u_in, lam_out, lam_bflux, lam_in, sc, dt, scratch, num_cus, s);
}

}  // namespace gd
