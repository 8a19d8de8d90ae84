// The tile march of the Euler step on gfx950: the device routine that one
// workgroup runs over a TX x TY column tile of a patch and a z-range of its
// planes, with the addressing and CFL-reduction helpers it uses. Included by
// every translation unit that instantiates a step kernel.
#pragma once

#include "godunov_cell.h"
#include "godunov_internal.h"
#include "godunov_math.h"

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gd {

// Threads of a tile: TX*TY interior columns, then the 2(TX+TY) ring
// columns, rounded up to whole waves (24x8: 192 + 64 = 256 threads, 4 waves).
constexpr int tile_threads(int tx, int ty) { return ((tx * ty + 2 * (tx + ty) + 63) / 64) * 64; }

// NT, the workgroup size, may exceed tile_threads(TX, TY) (a kernel that runs
// tiles of several shapes in one workgroup size); the surplus threads own no
// column and only pass the barriers.
template <int TX, int TY, int NT_ = tile_threads(TX, TY)>
struct TileGeom {
    static_assert(NT_ >= tile_threads(TX, TY), "workgroup too small for the tile");
    static constexpr int NINT = TX * TY;
    static constexpr int NT = NT_;
    // faces of a plane: the x faces i-1/2 (i = 0..TX) of each row, then the y
    // faces j-1/2 (j = 0..TY) of each column
    static constexpr int NXF = TY * (TX + 1);
    static constexpr int NF = NXF + (TY + 1) * TX;
    static constexpr int NSLOT = (NF + NT - 1) / NT;    // faces per thread
    __device__ static constexpr int xface(int i, int j) { return j * (TX + 1) + i; }
    __device__ static constexpr int yface(int i, int j) { return NXF + j * TX + i; }
    // (i, j) of face t; true for an x face
    __device__ static bool face_ij(int t, int &i, int &j)
    {
        const bool isx = t < NXF;
        const int u = isx ? t : t - NXF;
        i = isx ? u % (TX + 1) : u % TX;
        j = isx ? u / (TX + 1) : u / TX;
        return isx;
    }
};

// Storage slot of primitive component q in a y-face state: y faces are kept in
// their rotated order (rho, v, w, u, p), x faces in the natural one, so a face
// reads and writes slots 0..4 whatever its orientation.
__device__ constexpr int yslot(int q) { return q == 1 ? 3 : (q == 2 ? 1 : (q == 3 ? 2 : q)); }

// ------------------------------------------------------------ addressing

__device__ __forceinline__ int wrap_once(int i, int n) { return i < 0 ? i + n : (i >= n ? i - n : i); }

struct InputView {
    int64_t vstride;          // elements between variables
    int32_t sy, sz;           // row and plane strides
    int32_t nx, ny, nz, ng, periodic;

    // offset of column (i, j) within a plane
    __device__ __forceinline__ int64_t column(int i, int j) const
    {
        if (periodic) {
            i = wrap_once(wrap_once(i, nx), nx);
            j = wrap_once(wrap_once(j, ny), ny);
            return (int64_t)j * sy + i;
        }
        return (int64_t)(j + ng) * sy + (i + ng);
    }
    __device__ __forceinline__ int64_t plane(int k) const
    {
        if (periodic) return (int64_t)wrap_once(wrap_once(k, nz), nz) * sz;
        return (int64_t)(k + ng) * sz;
    }
};

__device__ __forceinline__ InputView make_view(const PatchDesc &P)
{
    InputView v;
    v.nx = P.nx; v.ny = P.ny; v.nz = P.nz; v.ng = P.ng; v.periodic = P.periodic;
    int gx = P.periodic ? P.nx : P.nx + 2 * P.ng;
    int gy = P.periodic ? P.ny : P.ny + 2 * P.ng;
    int gz = P.periodic ? P.nz : P.nz + 2 * P.ng;
    v.sy = gx;
    v.sz = gx * gy;
    v.vstride = (int64_t)gx * gy * gz;
    return v;
}

template <typename T>
__device__ __forceinline__ void load5(const T *__restrict__ p, int64_t vstride, T U[5])
{
#pragma unroll
    for (int q = 0; q < 5; ++q) U[q] = p[q * vstride];
}

// The five variables of a cell whose plane is the same for every lane (p, a
// scalar) and whose place in the plane is a byte offset of its own. A plane
// holds at most (16384 + 128)^2 cells, so the offset fits 32 bits, and the
// loads take a scalar base and a 32-bit vector offset: no vector address
// arithmetic.
template <typename T>
__device__ __forceinline__ void load5_plane(const T *__restrict__ p, int64_t vstride, uint32_t at,
                                            T U[5])
{
#pragma unroll
    for (int q = 0; q < 5; ++q)
        U[q] = *reinterpret_cast<const T *>(reinterpret_cast<const char *>(p + q * vstride) + at);
}

// ------------------------------------------------------------ CFL reduction

// |u| + |v| + |w| + 3c of a conserved state, c = sqrt(g p / rho) evaluated as
// g p / sqrt(g p rho). The CFL kernels and the fused CFL of the step kernels
// share this function, so both give the same dt bit for bit.
template <typename T>
__device__ __forceinline__ double cell_signal(const T U[5], const Phys<T> &ph, int &hits)
{
    T W[5], inv;
    prim_from_cons(U, W, inv, ph, hits);
    T gp = ph.gamma * W[4];
    T c = gp * fast_rsqrt(gp * W[0]);
    return (double)fma(T(3), c, fabs(W[1]) + fabs(W[2]) + fabs(W[3]));
}

__device__ __forceinline__ double wave_max(double v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
    return v;
}

// Block-wide max of v (>= 0) folded into *smax_bits, the bit pattern of a
// non-negative double (which orders like the value). Thread 0 reads the
// running value first and issues the device-wide atomic only when the
// block's maximum exceeds it, so a grid of thousands of workgroups performs
// few same-address atomics. The maximum is turned into dt and cleared for the
// next use by the last workgroup (cfl_finish) or by a one-thread launch
// (cfl_finalize_kernel).
__device__ void cfl_block_max(double v, unsigned long long *smax_bits)
{
    __shared__ double part[16];
    v = wave_max(v);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0) part[wv] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double m = 0.0;
        for (int i = 0; i < (int)(blockDim.x + 63) / 64; ++i) m = fmax(m, part[i]);
        const unsigned long long b = (unsigned long long)__double_as_longlong(m);
        if (b > __atomic_load_n(smax_bits, __ATOMIC_RELAXED)) atomicMax(smax_bits, b);
    }
}

// cfl_block_max, then (with a completion counter) the last workgroup's store
// of dt. A block's maximum has reached the device's atomics before the block
// counts itself, so the last one reads the maximum of all; no fence, which
// would write back the caches.
__device__ __forceinline__ void cfl_finish(double v, const CflOut &co)
{
    cfl_block_max(v, co.smax_bits);
    if (co.done && threadIdx.x == 0) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (atomicAdd(co.done, 1u) == gridDim.x - 1) {
            const unsigned long long b = atomicExch(co.smax_bits, 0ull);
            *co.dt_next = co.cfl / __longlong_as_double((long long)b);
            atomicExch(co.done, 0u);
        }
    }
}


// An index that is used in a rare branch only: computed there, and not kept in
// a register by the whole march.
__device__ __forceinline__ int rarely(int i)
{
    asm volatile("" : "+v"(i));
    return i;
}

// ------------------------------------------------------------ the tile march

template <typename T, int TX, int TY>
struct TileSmem {
    // primitives of plane k with its two-deep x-y halo (the column's own
    // planes k-1 and k+1 live in registers)
    T w[5][TY + 4][TX + 4];
    // one slot per x and y face of a plane, indexed as TileGeom::xface /
    // yface, y faces in rotated component order (yslot): first the right
    // (upper) state of the face, then its flux, written by the one thread
    // that solves the face. Two planes, in turn.
    T f[2][5][TileGeom<TX, TY>::NF];
};

enum { ROLE_NONE = -1, ROLE_INT = 0, ROLE_BOTTOM = 1, ROLE_TOP = 2, ROLE_LEFT = 3, ROLE_RIGHT = 4 };

// One tile: interior columns [x0, x0+TX) x [y0, y0+TY) (clipped to the
// patch), planes [z0, z1). Every face is solved by the owner of the cell on
// its left (lower) side, which keeps that cell's upper-face states in
// registers; only the lower-face states pass through LDS, and the flux goes
// back into the slot its right state came from, where the cell above finds
// it. Per plane k (with a prologue plane z0-1 that only produces the z+ face
// states, and an epilogue plane z1 that only produces the z- face states):
//   I   the x-y flux divergence of plane k-1; slopes, predictor and face
//       states of plane k; the z face below the plane, which completes and
//       stores plane k-1; the loads of the column's plane k+2 and of the halo's
//       plane k+1;
//   II  the plane's x and y faces (interior columns their upper ones, the
//       ring columns to the left and below the tile's first ones); plane k+1
//       staged in LDS, the column's plane k+2 converted.
// Two barriers a plane. Interior columns fill whole waves and the ring columns
// the rest, so the branch between the two is scalar, and both run unmasked:
// lanes without a column compute on the tile's first one, and neither write nor
// count. What a masked branch may or may not set occupies its registers
// throughout the branch, and the registers are what bounds the march: they set
// the waves per SIMD (three in FP64, four to five in FP32), a spilled prefetch
// costs a wait for each value, and vector instructions alone are cheap (a 2%
// gain from 15% fewer). The loads are issued where registers are free, behind
// the z face, with the faces of phase II before their use; U(k-1) before the
// slopes.
// Measured, against both states of every face passed through LDS to a thread
// picked for the face, with four barriers a plane, and then against masked roles
// with loads a plane ahead: 4096 patches of 8^3 to 32^3 FP64 2.03 -> 1.10 -> 0.97
// ms (the first with its tile choice), 250 x 190 x 141 FP32 0.336 -> 0.176 ->
// 0.171 ms, 256^3 FP64 box 1.04 -> 0.640 -> 0.648 ms; two-level step of a 128^3
// box and 1024 small patches 0.761 -> 0.592 -> 0.532 ms (the last with the seams'
// paired accesses and the tiles that choose_batched now takes for its batch).
// STREAM_OUT: write the new state with streaming (non-temporal) stores. The
// batched launches do: there the outputs of many small patches would
// otherwise evict from the L2 the inputs that neighbouring tiles still read
// (7% fewer bytes fetched on the 4096-patch batch, 1.5% faster). A single
// patch keeps ordinary stores: streaming ones raised its write traffic by 8%
// (rows that two tiles share are no longer merged in the L2) at no gain.
template <typename T, int LIM, int RS, int TX, int TY, int NT = tile_threads(TX, TY),
          bool STREAM_OUT = false>
__device__ void godunov_tile(const PatchDesc &P, const T *__restrict__ u_in_base,
                             T *__restrict__ u_out_base, T *__restrict__ bflux_base, T dtdx, T lam,
                             const Phys<T> &ph, int x0, int y0, int z0, int z1,
                             TileSmem<T, TX, TY> &sm, int &hits, bool want_cfl, double &smax)
{
#pragma clang fp contract(off)
    using Geo = TileGeom<TX, TY, NT>;
    static_assert(Geo::NINT % 64 == 0, "interior columns fill whole waves");
    const int tid = threadIdx.x, first = __builtin_amdgcn_readfirstlane(tid);
    const int ax = min(TX, P.nx - x0);
    const int ay = min(TY, P.ny - y0);
    const InputView view = make_view(P);
    const T *__restrict__ uin = u_in_base + P.in_off;

    // ---- role of this thread: an interior column, a ring column, or none
    // (which computes on the tile's first column, and neither writes nor counts)
    const bool tile_wave = first < Geo::NINT;
    const bool live = tile_wave ? first / TX < ay : first - Geo::NINT < 2 * (ax + ay);
    int ci = 0, cj = 0, role = ROLE_NONE;
    if (tid < Geo::NINT) {
        if (tid % TX < ax && tid / TX < ay) {
            ci = tid % TX;
            cj = tid / TX;
            role = ROLE_INT;
        }
    } else {
        int r = tid - Geo::NINT;
        if (r < ax) { ci = r; cj = -1; role = ROLE_BOTTOM; }
        else if (r < 2 * ax) { ci = r - ax; cj = ay; role = ROLE_TOP; }
        else if (r < 2 * ax + ay) { ci = -1; cj = r - 2 * ax; role = ROLE_LEFT; }
        else if (r < 2 * ax + 2 * ay) { ci = ax; cj = r - 2 * ax - ay; role = ROLE_RIGHT; }
    }
    const bool owner = role != ROLE_NONE;
    // a ring column has one face with the tile: an x face for the left and
    // right columns, a y face for the bottom and top rows; the left and bottom
    // columns hold its left (lower) state and solve it
    const bool ring_x = role == ROLE_LEFT || role == ROLE_RIGHT;
    const bool ring_lo = role == ROLE_LEFT || role == ROLE_BOTTOM;
    const int gi = x0 + ci, gj = y0 + cj;     // patch coordinates of the owned column
    const uint32_t col = (uint32_t)view.column(gi, gj) * (uint32_t)sizeof(T);
    // the face solved first (interior: the upper x face)
    const int face1 = tile_wave ? Geo::xface(ci + 1, cj)
                                : (ring_x ? Geo::xface(ci + ring_lo, cj) : Geo::yface(ci, cj + ring_lo));

    // ---- depth-2 halo and depth-1 corner cells of a plane, one per thread
    int hi = 0, hj = 0;
    const int nhalo = 2 * ax + 2 * ay + 4;
    const bool halo = tid < nhalo, halo_wave = first < nhalo;
    if (halo) {
        int h = tid;
        if (h < ax) { hi = h; hj = -2; }
        else if (h < 2 * ax) { hi = h - ax; hj = ay + 1; }
        else if (h < 2 * ax + ay) { hi = -2; hj = h - 2 * ax; }
        else if (h < 2 * ax + 2 * ay) { hi = ax + 1; hj = h - 2 * ax - ay; }
        else {
            int c = h - 2 * ax - 2 * ay;
            hi = (c & 1) ? ax : -1;
            hj = (c & 2) ? ay : -1;
        }
    }
    const uint32_t hcol = (uint32_t)view.column(x0 + hi, y0 + hj) * (uint32_t)sizeof(T);

    // boundary-flux sheets of this patch
    const bool want_flux = bflux_base != nullptr && P.flux_off >= 0;
    T *__restrict__ bf = want_flux ? bflux_base + P.flux_off : nullptr;
    const int64_t sxs = (int64_t)P.nz * P.ny, sys = (int64_t)P.nz * P.nx, szs = (int64_t)P.ny * P.nx;

    T *__restrict__ out = u_out_base + P.out_off;
    const int64_t ostride = (int64_t)P.nx * P.ny * P.nz;
    const double inv_dx = 1.0 / P.dx;
    const uint32_t ocol = (uint32_t)(gj * P.nx + gi) * (uint32_t)sizeof(T);

    // ---- registers of the owned column
    T Wm[5], W0[5], Wp[5], inv0, invp;
    T zprev[5], acc[5];
    T up1[5], up2[5];       // upper-face states, then the fluxes solved from them
    int col_hits = 0, halo_hits = 0;
    const int lx = ci + 2, ly = cj + 2;
    const T half = T(0.5);

    // prologue: planes z0-2 (used by interior columns only), z0-1 and z0
    {
        T Ua[5], Ub[5], Uc[5], inv;
        load5_plane(uin + view.plane(z0 - 2), view.vstride, col, Ua);
        load5_plane(uin + view.plane(z0 - 1), view.vstride, col, Ub);
        load5_plane(uin + view.plane(z0), view.vstride, col, Uc);
        int below = 0;
        prim_from_cons(Ua, Wm, inv, ph, below);
        if (tile_wave) col_hits += below;
        prim_from_cons(Ub, W0, inv0, ph, col_hits);
        prim_from_cons(Uc, Wp, invp, ph, col_hits);
#pragma unroll
        for (int q = 0; q < 5; ++q) {
            if (owner) sm.w[q][ly][lx] = W0[q];
            zprev[q] = acc[q] = up1[q] = up2[q] = T(0);
        }
    }
    __syncthreads();
    int b = 0;
#pragma unroll 1
    for (int k = z0 - 1;; ++k, b ^= 1) {
        const bool pre = k < z0;
        const bool post = k == z1;
        T(&f)[5][Geo::NF] = sm.f[b];

        // ---- I
        if (live) {
            if (tile_wave && k > z0) {
                const T(&g)[5][Geo::NF] = sm.f[b ^ 1];
#pragma unroll
                for (int q = 0; q < 5; ++q)
                    acc[q] = ((up1[q] - g[q][Geo::xface(ci, cj)]) +
                              (up2[yslot(q)] - g[yslot(q)][Geo::yface(ci, cj)])) + acc[q];
            }
            T Uold[5];
            load5_plane(uin + view.plane(max(k - 1, z0 - 1)), view.vstride, col, Uold);
            T Sx[5], Sy[5], Sz[5], Ws[5];
#pragma unroll
            for (int q = 0; q < 5; ++q) {
                T c = W0[q];
                Sx[q] = limited_slope<LIM>(c - sm.w[q][ly][lx - 1], sm.w[q][ly][lx + 1] - c);
                Sy[q] = limited_slope<LIM>(c - sm.w[q][ly - 1][lx], sm.w[q][ly + 1][lx] - c);
                Sz[q] = limited_slope<LIM>(c - Wm[q], Wp[q] - c);
            }
            predictor(W0, inv0, Sx, Sy, Sz, lam, ph.gamma, Ws);
            if (tile_wave) {
                T zm[5], zpn[5], dx[5], dy[5];
#pragma unroll
                for (int q = 0; q < 5; ++q) {
                    zm[q] = fma(-half, Sz[q], Ws[q]);
                    zpn[q] = fma(half, Sz[q], Ws[q]);
                    dx[q] = fma(-half, Sx[q], Ws[q]);
                    up1[q] = fma(half, Sx[q], Ws[q]);
                    dy[yslot(q)] = fma(-half, Sy[q], Ws[q]);
                    up2[yslot(q)] = fma(half, Sy[q], Ws[q]);
                }
                // the lowest of the six densities and of the six pressures: a
                // fused multiply-add is monotone, so it is the one of the
                // largest slope; only below the floor are the states looked at
                const T rmin = fma(-half, fmax(fmax(fabs(Sx[0]), fabs(Sy[0])), fabs(Sz[0])), Ws[0]);
                const T pmin = fma(-half, fmax(fmax(fabs(Sx[4]), fabs(Sy[4])), fabs(Sz[4])), Ws[4]);
                if (__builtin_expect(rmin < ph.rho_floor || pmin < ph.p_floor, 0)) {
                    // the prologue and epilogue planes use (and count) one state
                    int none = 0;
                    int &xy = pre || post ? none : col_hits;
                    zm[0] = floored(zm[0], ph.rho_floor, pre ? none : col_hits);
                    zm[4] = floored(zm[4], ph.p_floor, pre ? none : col_hits);
                    zpn[0] = floored(zpn[0], ph.rho_floor, post ? none : col_hits);
                    zpn[4] = floored(zpn[4], ph.p_floor, post ? none : col_hits);
                    dx[0] = floored(dx[0], ph.rho_floor, xy);
                    dx[4] = floored(dx[4], ph.p_floor, xy);
                    up1[0] = floored(up1[0], ph.rho_floor, xy);
                    up1[4] = floored(up1[4], ph.p_floor, xy);
                    dy[0] = floored(dy[0], ph.rho_floor, xy);
                    dy[4] = floored(dy[4], ph.p_floor, xy);
                    up2[0] = floored(up2[0], ph.rho_floor, xy);
                    up2[4] = floored(up2[4], ph.p_floor, xy);
                }
                if (owner) {
#pragma unroll
                    for (int q = 0; q < 5; ++q) {
                        f[q][Geo::xface(ci, cj)] = dx[q];
                        f[q][Geo::yface(ci, cj)] = dy[q];
                    }
                }
                if (!pre) {
                    // the z face below the plane; completes plane k-1
                    T F[5];
                    face_flux<RS, 2, SQ_Z>(zprev, zm, ph, F);
                    if (want_flux && owner && (k == 0 || k == P.nz)) {
                        T *sheet = bf + 10 * sxs + 10 * sys + (k == 0 ? 0 : 5 * szs);
                        const int at = rarely(gj) * P.nx + rarely(gi);
#pragma unroll
                        for (int q = 0; q < 5; ++q) sheet[q * szs + at] = F[q];
                    }
                    if (k > z0) {
                        // U' = U - dt/dx (acc + F_z(k-1/2)), acc = div_xy(k-1) - F_z(k-3/2)
                        T Un[5];
                        T *o = out + (int64_t)(k - 1) * P.nx * P.ny;
#pragma unroll
                        for (int q = 0; q < 5; ++q) Un[q] = fma(-dtdx, acc[q] + F[q], Uold[q]);
                        if (owner) {
#pragma unroll
                            for (int q = 0; q < 5; ++q) {
                                T *dst = reinterpret_cast<T *>(
                                    reinterpret_cast<char *>(o + q * ostride) + ocol);
                                if constexpr (STREAM_OUT) __builtin_nontemporal_store(Un[q], dst);
                                else *dst = Un[q];
                            }
                        }
                        if (want_cfl && owner) {
                            // signal speed of the new state, exactly as cfl_dt computes it
                            int unused = 0;
                            smax = fmax(smax, cell_signal(Un, ph, unused) * inv_dx);
                        }
                    }
#pragma unroll
                    for (int q = 0; q < 5; ++q) acc[q] = -F[q];
                }
#pragma unroll
                for (int q = 0; q < 5; ++q) zprev[q] = zpn[q];
            } else if (!pre && !post) {
                // a ring column: the one state its face with the tile needs,
                // direction and side selected per lane
                T st[5];
#pragma unroll
                for (int q = 0; q < 5; ++q)
                    st[q] = fma(ring_lo ? half : -half, ring_x ? Sx[q] : Sy[q], Ws[q]);
                st[0] = floored(st[0], ph.rho_floor, col_hits);
                st[4] = floored(st[4], ph.p_floor, col_hits);
                const T y[5] = { st[0], st[2], st[3], st[1], st[4] };
#pragma unroll
                for (int q = 0; q < 5; ++q) up1[q] = ring_x ? st[q] : y[q];
                if (owner && !ring_lo) {
#pragma unroll
                    for (int q = 0; q < 5; ++q) f[q][face1] = up1[q];
                }
            }
        }
        if (post) break;
        __builtin_amdgcn_sched_barrier(0);
        T Upf[5], Hpf[5];
        load5_plane(uin + view.plane(k + 2), view.vstride, col, Upf);
        load5_plane(uin + view.plane(k + 1), view.vstride, hcol, Hpf);
        __syncthreads();

        // ---- II
        if (!pre && live) {
            T R[5], G[5];
#pragma unroll
            for (int q = 0; q < 5; ++q) R[q] = f[q][face1];
            riemann<RS, SQ_XY>(up1, R, ph, G);
#pragma unroll
            for (int q = 0; q < 5; ++q) up1[q] = G[q];
            if (tile_wave ? owner : ring_lo) {
#pragma unroll
                for (int q = 0; q < 5; ++q) f[q][face1] = G[q];
                if (want_flux) {
                    // the face's index along its axis: gi+1 (an interior
                    // column's upper face, or the left ring's), gj+1 for the
                    // bottom ring
                    if (tile_wave || ring_x) {
                        if (gi + 1 == (tile_wave ? P.nx : 0)) {
                            T *sheet = bf + (tile_wave ? 5 * sxs : 0);
                            const int at = k * P.ny + rarely(gj);
#pragma unroll
                            for (int q = 0; q < 5; ++q) sheet[q * sxs + at] = G[q];
                        }
                    } else if (gj + 1 == 0) {
                        T *sheet = bf + 10 * sxs;
                        const int at = k * P.nx + rarely(gi);
#pragma unroll
                        for (int q = 0; q < 5; ++q) sheet[q * sys + at] = G[yslot(q)];
                    }
                }
            }
            if (tile_wave) {
                const int face2 = Geo::yface(ci, cj + 1);
#pragma unroll
                for (int q = 0; q < 5; ++q) R[q] = f[q][face2];
                riemann<RS, SQ_XY>(up2, R, ph, G);
#pragma unroll
                for (int q = 0; q < 5; ++q) up2[q] = G[q];
                if (owner) {
#pragma unroll
                    for (int q = 0; q < 5; ++q) f[q][face2] = G[q];
                    if (want_flux && gj + 1 == P.ny) {
                        T *sheet = bf + 10 * sxs + 5 * sys;
                        const int at = k * P.nx + rarely(gi);
#pragma unroll
                        for (int q = 0; q < 5; ++q) sheet[q * sys + at] = G[yslot(q)];
                    }
                }
            }
        }
        // the column moves up: plane k+1 staged, plane k+2 from its loads
#pragma unroll
        for (int q = 0; q < 5; ++q) {
            Wm[q] = W0[q];
            W0[q] = Wp[q];
        }
        inv0 = invp;
        if (owner) {
#pragma unroll
            for (int q = 0; q < 5; ++q) sm.w[q][ly][lx] = W0[q];
        }
        if (live) {
            int own = 0;
            prim_from_cons_march(Upf, Wp, invp, ph, own);
            // (a ring column uses planes up to z1, an interior one z1+1)
            if (tile_wave || k + 2 <= z1) col_hits += own;
        }
        if (halo_wave && k + 1 < z1) {
            T Wh[5], invh;
            prim_from_cons_march(Hpf, Wh, invh, ph, halo_hits);
            if (halo) {
#pragma unroll
                for (int q = 0; q < 5; ++q) sm.w[q][hj + 2][hi + 2] = Wh[q];
            }
        }
        __syncthreads();
    }
    hits += (owner ? col_hits : 0) + (halo ? halo_hits : 0);
}

__device__ __forceinline__ void flush_hits(int hits, unsigned long long *counter)
{
    if (hits) atomicAdd(counter, (unsigned long long)hits);
}

// One patch. Workgroups are dispatched round-robin over the 8 XCDs (each
// with its own L2); the block index is remapped so that each XCD works
// through a contiguous range of items, ordered z-segment-major then tile
// row-major, so that tiles sharing halo columns run on the same L2.
// Occupancy target: three waves per SIMD in FP64 (168 VGPRs), four in FP32.
template <typename T>
constexpr int waves_per_eu() { return sizeof(T) == 8 ? 3 : 4; }

}  // namespace gd
