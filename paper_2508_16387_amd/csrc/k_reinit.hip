// k_reinit.hip -- level-set reinitialization (section "Level set method",
// eq. reinit): pseudo-time steps of
//     d phi / d tau + S(phi_0) (|grad phi| - 1) = 0,
//     S(phi_0) = phi_0 / sqrt(phi_0^2 + eps^2),
// with the upwind (Godunov) |grad phi| of one-sided differences a = D^- phi,
// b = D^+ phi per active axis:
//     S > 0: sum_d max(max(a_d, 0)^2, min(b_d, 0)^2)
//     S < 0: sum_d max(min(a_d, 0)^2, max(b_d, 0)^2)
// and forward-Euler steps dtau = 0.5 min_d h_d (Jacobi: every cell reads the
// previous iterate).  First-layer cells (a face neighbour on the other side
// of the zero level set, phi >= 0 counting as the non-negative side) keep
// phi_0, which is the paper's fixed-first-layer treatment; with a narrow
// band only cells with |phi_0| < band move.  Both are expressed as S = 0.
//
// Boundary images: one layer, periodic axes wrap, transmissive and wall
// boundaries repeat the boundary cell (the zero-gradient and mirror images
// of phi coincide for one layer).
//
// Work decomposition (MI355X): over the whole grid a thread owns one column
// of RZ_FULL consecutive planes, a block 256 consecutive columns (row after
// row, so that no lane falls past the end of a row); in a narrow band the
// blocks are 64 x 4 tiles of one plane, the compact shape that fewest of the
// band's cells touch, and only those on a list run.  A cell reads its own
// value, S and its x and y neighbours (cache lines that its block loads
// anyway); its z neighbours are the thread's own planes.  All planes of a
// block are compile-time known, so their loads are in flight together and no
// wavefront waits for a barrier; blocks are renumbered so that each XCD takes
// a contiguous run of tiles, whose shared rows and planes meet in its L2.
// The Godunov term of an axis is the square of max(s a, -s b, 0), s the sign
// of S: seven instructions where both signs' forms took fifteen.  Measured at
// 200x160x144: 31.3 us per step with rows exchanged through LDS, a barrier
// per plane and 64-wide tiles (a quarter of the lanes past the row's end),
// 23 us now, bound by FP64 issue and the Infinity Cache about equally.
//
// The speed kernel also writes the second iterate's start.  In a narrow band
// it appends the blocks that hold any cell with S != 0 to the list; over the
// whole grid nearly all do, and one counter for all of them (5760 blocks'
// atomics, two thirds of its 79 us) is left out.  The iterate is kept in two buffers
// that both start as phi_0; a frozen cell never changes, so it is never
// written -- a narrow band costs only the blocks it touches.  Per iteration
// and moving cell the algorithmic traffic is phi and S read, phi written: 24
// bytes.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "m2c.h"
#include "m2c_reinit.h"

namespace m2c {
namespace {

constexpr int RX = 64, RY = 4;
// Planes per block: 4 over the whole grid (us per step with 2, 4 and 8: 64^3
// 3.7, 4.2, 5.6; 128^3 12.2, 11.9, 12.7; 256^3 113, 99, 96: fewer leave more
// z neighbours to be read twice, more leave small grids too few blocks); 1
// in a narrow band, where the tile of one plane is the one that fewest idle
// cells share (band of six cells, with 1, 2 and 4: 64^3 3.5, 3.7, 4.1; 128^3
// 7.1, 6.6, 7.1; 256^3 19.8, 16.5, 16.9, so two would be the better choice
// from 128^3 on).
constexpr int RZ_FULL = 4, RZ_BAND = 1;

__device__ __forceinline__ int image(int i, int n, int periodic)
{
    return i < 0 ? (periodic ? i + n : 0) : (i >= n ? (periodic ? i - n : n - 1) : i);
}

struct Tile {
    int i, j, k0;
    bool live;                        // inside the grid (else clamped to it)
};

// BAND: 64 x 4 tile b of one plane; otherwise 256 consecutive columns of
// RZ_FULL planes.
template <bool BAND>
__device__ __forceinline__ Tile tile_of(const ReinitGrid& g, uint32_t b)
{
    Tile t;
    if (BAND) {
        const uint32_t bx = b % (uint32_t)g.bx, r = b / (uint32_t)g.bx;
        const uint32_t by = r % (uint32_t)g.by, bz = r / (uint32_t)g.by;
        const int i = (int)(bx * RX + threadIdx.x % RX), j = (int)(by * RY + threadIdx.x / RX);
        t.live = i < g.nx && j < g.ny;
        t.i = min(i, g.nx - 1);
        t.j = min(j, g.ny - 1);
        t.k0 = (int)bz * RZ_BAND;
    } else {
        const uint32_t pl = (uint32_t)g.nx * (uint32_t)g.ny, nb = (pl - 1) / (RX * RY) + 1;
        const uint32_t bz = b / nb, c = (b - bz * nb) * (RX * RY) + threadIdx.x;
        t.live = c < pl;
        const uint32_t cc = t.live ? c : pl - 1;
        t.j = (int)(cc / (uint32_t)g.nx);
        t.i = (int)(cc - (uint32_t)t.j * (uint32_t)g.nx);
        t.k0 = (int)bz * RZ_FULL;
    }
    return t;
}

// Dispatch is round-robin over the 8 XCDs: block b of n runs on XCD b % 8;
// each XCD's blocks take one contiguous run of tiles.
__device__ __forceinline__ uint32_t xcd_run(uint32_t b, uint32_t n)
{
    const uint32_t q = n / 8, r = n % 8, x = b % 8, idx = b / 8;
    return (x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q) + idx;
}

// Values of one field at a thread's cells of RZ consecutive planes and at
// their neighbours (boundary images applied; every index in range, also for
// threads and planes past the grid, whose cells are not written).
template <int RZ>
struct Stencil {
    double c[RZ + 2];                 // planes k0 - 1 .. k0 + RZ (past the last: repeated)
    double top;                       // z image above the grid's last plane
    double xa[RZ], xb[RZ], ya[RZ], yb[RZ];
    uint32_t cell[RZ];
};

template <int RZ>
__device__ __forceinline__ void load_stencil(const ReinitGrid& g, const Tile& t, const double* __restrict__ phi,
                                             Stencil<RZ>& v)
{
    const uint32_t pl = (uint32_t)g.nx * (uint32_t)g.ny, row = (uint32_t)g.nx * (uint32_t)t.j, col = row + (uint32_t)t.i;
    const uint32_t xm = row + (uint32_t)image(t.i - 1, g.nx, g.per[0]), xp = row + (uint32_t)image(t.i + 1, g.nx, g.per[0]);
    const uint32_t ym = (uint32_t)g.nx * (uint32_t)image(t.j - 1, g.ny, g.per[1]) + (uint32_t)t.i;
    const uint32_t yp = (uint32_t)g.nx * (uint32_t)image(t.j + 1, g.ny, g.per[1]) + (uint32_t)t.i;
    const int last = g.nz - 1;
    v.c[0] = phi[col + pl * (uint32_t)image(t.k0 - 1, g.nz, g.per[2])];
#pragma unroll
    for (int q = 0; q < RZ; ++q) {
        const uint32_t o = pl * (uint32_t)min(t.k0 + q, last);
        v.cell[q] = col + o;
        v.c[1 + q] = phi[col + o];
        v.ya[q] = phi[ym + o];
        v.yb[q] = phi[yp + o];
        v.xa[q] = phi[xm + o];
        v.xb[q] = phi[xp + o];
    }
    v.c[1 + RZ] = phi[col + pl * (uint32_t)min(t.k0 + RZ, last)];
    v.top = phi[col + pl * (uint32_t)image(g.nz, g.nz, g.per[2])];
}

// Upper z neighbour of the thread's plane q.
template <int RZ>
__device__ __forceinline__ double z_above(const ReinitGrid& g, const Tile& t, const Stencil<RZ>& v, int q)
{
    return t.k0 + q == g.nz - 1 ? v.top : v.c[2 + q];
}

template <bool BAND>
__global__ __launch_bounds__(256) void k_reinit_speed(const ReinitGrid g, const double* __restrict__ phi0,
                                                      double eps2, double band, double* __restrict__ S,
                                                      double* __restrict__ tmp, int32_t* __restrict__ list)
{
    constexpr int RZ = BAND ? RZ_BAND : RZ_FULL;
    const uint32_t blk = xcd_run(blockIdx.x, gridDim.x);
    const Tile t = tile_of<BAND>(g, blk);
    int any = 0;
    // (a wavefront past the grid has nothing to do; 1x1x200000, band of two
    // cells, 11 iterations: 309 us with its loads, 252 without)
    if (!BAND || __any(t.live)) {                // wave-uniform
        Stencil<RZ> v;
        load_stencil<RZ>(g, t, phi0, v);
#pragma unroll
        for (int q = 0; q < RZ; ++q) {
            const double p = v.c[1 + q];
            const bool pos = p >= 0.0;
            bool fl = false;
            if (g.act[0]) fl |= (v.xa[q] >= 0.0) != pos || (v.xb[q] >= 0.0) != pos;
            if (g.act[1]) fl |= (v.ya[q] >= 0.0) != pos || (v.yb[q] >= 0.0) != pos;
            if (g.act[2]) fl |= (v.c[q] >= 0.0) != pos || (z_above<RZ>(g, t, v, q) >= 0.0) != pos;
            double s = p / sqrt(p * p + eps2);
            if (fl || (BAND && fabs(p) >= band)) s = 0.0;
            if (t.live && t.k0 + q < g.nz) {
                S[v.cell[q]] = s;
                tmp[v.cell[q]] = p;
                any |= s != 0.0;
            }
        }
    }
    if (!BAND) return;
    any = __syncthreads_or(any);
    // list[0] counts the blocks with moving cells, list[1..] holds them
    if (threadIdx.x == 0 && any) list[1 + atomicAdd(&list[0], 1)] = (int32_t)blk;
}

// a^2 + b^2 + c^2, each square rounded before it is added.
__device__ __forceinline__ double norm2(double a, double b, double c)
{
#pragma clang fp contract(off)
    return a * a + b * b + c * c;
}

// BAND: the block runs tile list[1 + block]; otherwise every tile of the grid
template <bool BAND>
__global__ __launch_bounds__(256) void k_reinit_step(const ReinitGrid g, const double* __restrict__ phi,
                                                     double* __restrict__ out, const double* __restrict__ S,
                                                     const int32_t* __restrict__ list, double dtau)
{
    constexpr int RZ = BAND ? RZ_BAND : RZ_FULL;
    const uint32_t b = xcd_run(blockIdx.x, gridDim.x);
    const Tile t = tile_of<BAND>(g, BAND ? (uint32_t)list[1 + b] : b);
    if (BAND && !__any(t.live)) return;           // wave-uniform
    Stencil<RZ> v;
    double s[RZ];
    load_stencil<RZ>(g, t, phi, v);
#pragma unroll
    for (int q = 0; q < RZ; ++q) s[q] = S[v.cell[q]];
#pragma unroll
    for (int q = 0; q < RZ; ++q) {
        const double p = v.c[1 + q];
        // frozen (S = 0): both buffers hold phi_0
        if (t.live && t.k0 + q < g.nz && s[q] != 0.0) {
            // S > 0: the larger of max(a, 0) and -min(b, 0); S < 0 the same of
            // -a and -b (a, b the one-sided differences): signs are exact, and
            // the larger square is the square of the larger
            auto term = [&](double lo, double hi, double rh) {
                const double rs = copysign(rh, s[q]);
                return fmax(fmax((p - lo) * rs, (p - hi) * rs), 0.0);
            };
            const double g2 = norm2(g.act[0] ? term(v.xa[q], v.xb[q], g.rh[0]) : 0.0,
                                    g.act[1] ? term(v.ya[q], v.yb[q], g.rh[1]) : 0.0,
                                    g.act[2] ? term(v.c[q], z_above<RZ>(g, t, v, q), g.rh[2]) : 0.0);
            out[v.cell[q]] = p - dtau * s[q] * (sqrt(g2) - 1.0);
        }
    }
}

}  // namespace

long long reinit_blocks(const ReinitGrid& g)
{
    return (long long)g.bx * g.by * g.bz;
}

bool reinit_grid(int nx, int ny, int nz, const double h[3], const int32_t bc[6], ReinitGrid& g)
{
    if (nx < 1 || ny < 1 || nz < 1) return false;
    if ((long long)nx * ny * nz > (1LL << 31)) return false;
    g.nx = nx;
    g.ny = ny;
    g.nz = nz;
    const int n[3] = {nx, ny, nz};
    double hmin = INFINITY;
    for (int d = 0; d < 3; ++d) {
        if (!(h[d] > 0.0) || !isfinite(h[d])) return false;
        for (int s = 0; s < 2; ++s)
            if (bc[2 * d + s] < M2C_BC_TRANSMISSIVE || bc[2 * d + s] > M2C_BC_PERIODIC) return false;
        if ((bc[2 * d] == M2C_BC_PERIODIC) != (bc[2 * d + 1] == M2C_BC_PERIODIC)) return false;
        g.per[d] = bc[2 * d] == M2C_BC_PERIODIC;
        g.act[d] = n[d] > 1;
        g.h[d] = h[d];
        g.rh[d] = 1.0 / h[d];
        if (g.act[d]) hmin = fmin(hmin, h[d]);
    }
    g.hmin = isfinite(hmin) ? hmin : fmin(h[0], fmin(h[1], h[2]));
    g.bx = (nx + RX - 1) / RX;
    g.by = (ny + RY - 1) / RY;
    g.rz = RZ_FULL;
    g.bz = (nz + g.rz - 1) / g.rz;
    return true;
}

hipError_t reinit_run(const ReinitGrid& g0, double* phi, double* S, double* tmp, int32_t* list, int iters,
                      double band, hipStream_t s)
{
    ReinitGrid g = g0;
    if (iters <= 0) return hipSuccess;
    // (not recorded into a graph: the band's launches need its block count)
    hipStreamCaptureStatus capturing = hipStreamCaptureStatusNone;
    hipError_t e = hipStreamIsCapturing(s, &capturing);
    if (e != hipSuccess) return e;
    if (capturing != hipStreamCaptureStatusNone) return hipErrorStreamCaptureUnsupported;
    const long long N = (long long)g.nx * g.ny * g.nz;
    const double eps2 = g.hmin * g.hmin;              // smallest cell width, squared
    const double dtau = 0.5 * g.hmin;
    const bool narrow = band > 0.0;
    long long nb;
    if (narrow) {
        g.rz = RZ_BAND;
        g.bz = (g.nz + g.rz - 1) / g.rz;
        nb = reinit_blocks(g);
    } else {
        nb = (((long long)g.nx * g.ny - 1) / (RX * RY) + 1) * ((g.nz + RZ_FULL - 1) / RZ_FULL);
    }
    if (nb > 0x7fffffffLL) return hipErrorInvalidValue;
    if (narrow) {
        e = hipMemsetAsync(list, 0, sizeof(int32_t), s);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_reinit_speed<true>, dim3((unsigned)nb), dim3(256), 0, s, g, phi, eps2, band, S, tmp, list);
    } else {
        hipLaunchKernelGGL(k_reinit_speed<false>, dim3((unsigned)nb), dim3(256), 0, s, g, phi, eps2, band, S, tmp, list);
    }
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (narrow) {
        // the number of moving blocks sizes every step launch
        int32_t nact = 0;
        e = hipMemcpyAsync(&nact, list, sizeof(int32_t), hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess) return e;
        if (nact < 0 || nact > nb) return hipErrorUnknown;
        if (nact == 0) return hipSuccess;
        nb = nact;
    }
    for (int it = 0; it < iters; ++it) {
        const double* src = (it & 1) ? tmp : phi;
        double* dst = (it & 1) ? phi : tmp;
        if (narrow)
            hipLaunchKernelGGL(k_reinit_step<true>, dim3((unsigned)nb), dim3(256), 0, s, g, src, dst, S, list, dtau);
        else
            hipLaunchKernelGGL(k_reinit_step<false>, dim3((unsigned)nb), dim3(256), 0, s, g, src, dst, S, list, dtau);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (iters & 1) e = hipMemcpyAsync(phi, tmp, N * sizeof(double), hipMemcpyDeviceToDevice, s);
    return e;
}

}  // namespace m2c

using namespace m2c;

extern "C" int m2c_reinit_workspace(int32_t nx, int32_t ny, int32_t nz, int64_t* bytes)
{
    const double h[3] = {1.0, 1.0, 1.0};
    const int32_t bc[6] = {0, 0, 0, 0, 0, 0};
    ReinitGrid g;
    if (!bytes || !reinit_grid(nx, ny, nz, h, bc, g)) return M2C_ERR_ARG;
    *bytes = reinit_workspace_bytes(g);
    return M2C_OK;
}

extern "C" int m2c_reinit_field(int32_t nx, int32_t ny, int32_t nz, const double h[3], const int32_t bc[6],
                                double* phi, void* work, int32_t iters, double band, void* hip_stream)
{
    ReinitGrid g;
    if (!h || !bc || !reinit_grid(nx, ny, nz, h, bc, g)) return M2C_ERR_ARG;
    if (iters < 0 || !(band >= 0.0) || !isfinite(band)) return M2C_ERR_ARG;
    if (iters == 0) return M2C_OK;
    if (!phi || !work) return M2C_ERR_ARG;
    const long long N = (long long)nx * ny * nz;
    double* S = (double*)work;
    double* tmp = S + N;
    int32_t* active = (int32_t*)(tmp + N);
    return reinit_run(g, phi, S, tmp, active, iters, band, (hipStream_t)hip_stream) == hipSuccess ? M2C_OK
                                                                                                  : M2C_ERR_DEVICE;
}
