// cslbm.hip -- the C ABI of libcslbm (gfx950) and its single-level helper
// kernels: flags, initialisation, population copies, read-back, vorticity,
// FP64 conservation totals and the finiteness check.  The collide-stream
// kernel itself lives in step.hip.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>
#include <type_traits>
#include <utility>

#include "../../include/cslbm.h"
#include "cm_collide.hpp"
#include "brick.hpp"
#include "exchange.hpp"
#include "internal.hpp"
#include "lattice.hpp"

namespace cslbm {

// ---------------------------------------------------------------------------
// error reporting
// ---------------------------------------------------------------------------
static thread_local std::string g_last_error;

int fail(int code, const char* fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_last_error = buf;
    return code;
}

int check_launch(const char* what)
{
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(CSLBM_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
    return CSLBM_OK;
}

// ---------------------------------------------------------------------------
// auxiliary kernels (one thread per cell, 1D launch over N)
// ---------------------------------------------------------------------------
__device__ __forceinline__ void cell_coords(int64_t c, int nx, int ny, int& x, int& y, int& z)
{
    x = (int)(c % nx);
    y = (int)((c / nx) % ny);
    z = (int)(c / ((int64_t)nx * ny));
}

__global__ void k_prepare_flags(uint8_t* flags, uint32_t* links, int nx, int ny, int nz,
                                int periodic, int64_t N, const BrickMap bm)
{
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= N) return;
    int x, y, z;
    if (bm.table)
        brick_xyz(bm, (int)c, x, y, z);
    else
        cell_coords(c, nx, ny, x, y, z);
    const uint8_t kind = flags[c] & kKindMask;
    uint32_t m = 0;
    bool near_fluid = false;
    if (kind != kFluid && kind != kWall) {
        // some neighbour (periodic wrap on every axis) is fluid: the adjoint
        // step checks such cells' neighbours before writing zeros
#pragma unroll
        for (int i = 1; i < Q; ++i) {
            int64_t src;
            if (bm.table) {
                const int s = brick_neighbour(bm, (int)c, x, y, z, kCx[i], kCy[i], kCz[i]);
                if (s < 0) continue;
                src = s;
            } else {
                const int xs = (x - kCx[i] + nx) % nx, ys = (y - kCy[i] + ny) % ny,
                          zs = (z - kCz[i] + nz) % nz;
                src = xs + (int64_t)nx * (ys + (int64_t)ny * zs);
            }
            near_fluid |= (flags[src] & kKindMask) == kFluid;
        }
    } else {
#pragma unroll
        for (int i = 1; i < Q; ++i) {
            if (leaves_box(x, y, z, kCx[i], kCy[i], kCz[i], nx, ny, nz, periodic)) {
                m |= 1u << i;
                continue;
            }
            int64_t src;
            if (bm.table) {
                // a source that is not stored counts as solid (a valid brick
                // level never lets a fluid cell pull from one)
                const int s = brick_neighbour(bm, (int)c, x, y, z, kCx[i], kCy[i], kCz[i]);
                if (s < 0) {
                    m |= 1u << i;
                    continue;
                }
                src = s;
            } else {
                const int xs = (x - kCx[i] + nx) % nx, ys = (y - kCy[i] + ny) % ny,
                          zs = (z - kCz[i] + nz) % nz;
                src = xs + (int64_t)nx * (ys + (int64_t)ny * zs);
            }
            if ((flags[src] & kKindMask) == kSolid) m |= 1u << i;
        }
    }
    // wall node: the normal is minus the one axis velocity whose pull source
    // is blocked (code k for velocity k = 1..6: n = -c_k), and the blocked
    // sources must be exactly those of the velocities pointing away from the
    // wall (c.n < 0); otherwise code 7
    int wall_code = 0;
    if (kind == kWall) {
        int axis_blocked = 0;
        wall_code = 7;
#pragma unroll
        for (int k = 1; k <= 6; ++k)
            if (m & (1u << k)) {
                ++axis_blocked;
                wall_code = k;
            }
        if (axis_blocked != 1) {
            wall_code = 7;
        } else {
            uint32_t expect = 0;
#pragma unroll
            for (int i = 1; i < Q; ++i) {
                const int cn = -(kCx[i] * kCx[wall_code] + kCy[i] * kCy[wall_code] +
                                 kCz[i] * kCz[wall_code]);
                if (cn < 0) expect |= 1u << i;
            }
            if (expect != m) wall_code = 7;
        }
    }
    flags[c] = kind | (m ? kNearWall : 0) | (near_fluid ? CSLBM_NEAR_FLUID : 0) |
               (uint8_t)(wall_code << kWallNormalShift);
    if (links) links[c] = m;
}

template <typename T>
__global__ void k_init_eq(T* f, float* g, int64_t N, int64_t P, const float* rho, const float* u,
                          const float* s)
{
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= N) return;
    const float r = rho ? rho[c] : 1.0f;
    const float ux = u[c], uy = u[N + c], uz = u[2 * N + c];
    float v[27];
    shifted_equilibrium(v, r, ux, uy, uz);
#pragma unroll
    for (int i = 0; i < Q; ++i) Io<T>::st(f + i * P + c, v[tensor_slot(i)]);
    if (g) {
        const float sc = s ? s[c] : 0.0f;
#pragma unroll
        for (int i = 0; i < QS; ++i) g[i * P + c] = scalar_eq(i, sc, ux, uy, uz);
    }
}

template <typename T>
__global__ void k_set_pop(T* f, float* g, int64_t N, int64_t P, const float* src, const float* gsrc,
                          int shifted)
{
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= N) return;
    float v[Q], u[QS];   // all loads before the first store
#pragma unroll
    for (int i = 0; i < Q; ++i) v[i] = src[i * N + c];
    const bool scalar = g && gsrc;
    if (scalar)
#pragma unroll
        for (int i = 0; i < QS; ++i) u[i] = gsrc[i * N + c];
#pragma unroll
    for (int i = 0; i < Q; ++i) Io<T>::st(f + i * P + c, shifted ? v[i] : v[i] - weight(i));
    if (scalar)
#pragma unroll
        for (int i = 0; i < QS; ++i) g[i * P + c] = u[i];
}

// Population copy between two levels of one storage type, cell list to
// cell list (the kept part of a rebuilt region).  One thread per cell.
template <typename T>
__global__ void __launch_bounds__(256) k_copy_cells(const T* f, const float* g, int64_t P, T* fo,
                                                    float* go, int64_t Po, const int32_t* src,
                                                    const int32_t* dst, int n)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    const int64_t a = src[k], b = dst[k];
    // all loads before the first store: a store between them would order
    // each later load after it (the compiler cannot rule out overlap)
    T v[Q];
    float u[QS];
#pragma unroll
    for (int i = 0; i < Q; ++i) v[i] = f[i * P + a];
    if (g)
#pragma unroll
        for (int i = 0; i < QS; ++i) u[i] = g[i * P + a];
#pragma unroll
    for (int i = 0; i < Q; ++i) fo[i * Po + b] = v[i];
    if (g)
#pragma unroll
        for (int i = 0; i < QS; ++i) go[i * Po + b] = u[i];
}

template <typename T>
__global__ void k_get_pop(const T* f, const float* g, int64_t N, int64_t P, float* dst, float* gdst,
                          int shifted)
{
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= N) return;
    float h[Q], u[QS];   // all loads before the first store
#pragma unroll
    for (int i = 0; i < Q; ++i) h[i] = Io<T>::ld(f + i * P + c);
    const bool scalar = g && gdst;
    if (scalar)
#pragma unroll
        for (int i = 0; i < QS; ++i) u[i] = g[i * P + c];
#pragma unroll
    for (int i = 0; i < Q; ++i) dst[i * N + c] = shifted ? h[i] : h[i] + weight(i);
    if (scalar)
#pragma unroll
        for (int i = 0; i < QS; ++i) gdst[i * N + c] = u[i];
}

// velocity u = (j - F/2)/rho of one cell's stored populations (tensor order)
// with the level's force and buoyancy; returns the density, s the scalar
__device__ __forceinline__ float velocity(const float (&v)[27], const float* g, const float* force,
                                          int64_t P, int64_t c, float beta, float s_ref, float (&u)[3],
                                          float* s = nullptr)
{
    float dr, jx, jy, jz;
    moments0(v, dr, jx, jy, jz);
    float sc = 0.0f;
    if (g)
#pragma unroll
        for (int i = 0; i < QS; ++i) sc += g[i * P + c];
    float Fx = 0.0f, Fy = 0.0f, Fz = 0.0f;
    if (force) {
        Fx = force[c];
        Fy = force[P + c];
        Fz = force[2 * P + c];
    }
    if (g) Fz += beta * (sc - s_ref);
    const float r = 1.0f + dr;
    u[0] = (jx - 0.5f * Fx) / r;
    u[1] = (jy - 0.5f * Fy) / r;
    u[2] = (jz - 0.5f * Fz) / r;
    if (s) *s = sc;
    return r;
}

template <typename T>
__global__ void k_macro(const T* f, const float* g, const float* force, int64_t N, int64_t P,
                        float beta, float s_ref, float* rho, float* u, float* s)
{
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= N) return;
    float v[27];
#pragma unroll
    for (int i = 0; i < Q; ++i) v[tensor_slot(i)] = Io<T>::ld(f + i * P + c);
    float w[3], sc;
    const float r = velocity(v, g, force, P, c, beta, s_ref, w, &sc);
    if (rho) rho[c] = r;
    if (u) {
        u[c] = w[0];
        u[N + c] = w[1];
        u[2 * N + c] = w[2];
    }
    if (s) s[c] = sc;
}

// |curl u| and |u| of the stored state by central differences (periodic wrap
// on periodic axes, one-sided differences at non-periodic faces).  A
// workgroup walks a tx x ty tile along z: every thread reads one cell's
// populations of the plane (the tile and one cell around it), its velocity
// goes to a ring of four planes in LDS (one barrier a plane: the slot written
// next is not among the three being read), and the output threads take their
// differences there.  Against a velocity field written to temporary memory
// and differenced by a second kernel (below): 492 / 578 us at 256^3 FP32, 334 /
// 396 binary16, 71 / 78 us at 128^3 with scalar, 26 / 34 us at 2x600x600 binary16,
// 110 / 106 us at 65x200x200 with scalar (the worst of 450 boxes; 1.4 times
// as fast on average).  At 256^3 it is bound by
// the lines at the tiles' edges, which its two neighbours fetch as well (the
// read-back of density and velocity alone takes 388 us).
constexpr int kVortWidth = 64;      // widest tile
constexpr int kVortThreads = 704;   // most cells of a tile and its rim

struct VortArgs {
    const void* f;
    const float* g;
    const float* force;
    int nx, ny, nz, periodic;
    int ntx, nty, cz;   // tiles along x and y, planes per workgroup
    int tx, ty;         // cells of a tile (k_vorticity)
    int64_t plane;
    float beta, s_ref;
    float* out;
    float* speed;
};

// the cell an index of the tile's rim stands for: outside the box it wraps on
// a periodic axis and repeats the face cell on the others (never read there)
__device__ __forceinline__ int vort_cell(int i, int n, bool periodic)
{
    return periodic ? (i % n + n) % n : min(max(i, 0), n - 1);
}

// offsets of the two differenced points along an axis (0 at a face); the
// distance between them is 1 or 2 cells, or 0 along a single cell
__device__ __forceinline__ void vort_points(int i, int n, bool periodic, int& lo, int& hi)
{
    lo = !periodic && i == 0 ? 0 : 1;
    hi = !periodic && i == n - 1 ? 0 : 1;
}

__device__ __forceinline__ float vort_slope(float hi, float lo, int h)
{
    return h > 0 ? (hi - lo) * (h == 1 ? 1.0f : 0.5f) : 0.0f;
}

// grad[a][b] = d u_a / d x_b and the cell's velocity, to cell c
__device__ __forceinline__ void vort_store(const VortArgs& a, int64_t c, const float (&grad)[3][3],
                                           float ux, float uy, float uz)
{
    const float wx = grad[2][1] - grad[1][2], wy = grad[0][2] - grad[2][0], wz = grad[1][0] - grad[0][1];
    __builtin_nontemporal_store(sqrtf(wx * wx + wy * wy + wz * wz), a.out + c);
    if (a.speed) __builtin_nontemporal_store(sqrtf(ux * ux + uy * uy + uz * uz), a.speed + c);
}

template <typename T>
__global__ void __launch_bounds__(kVortThreads) k_vorticity(const VortArgs a)
{
    __shared__ float ring[4][3][kVortThreads];
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const int64_t nxy = (int64_t)nx * ny, P = a.plane;
    const T* f = static_cast<const T*>(a.f);
    const int blk = xcd_block(blockIdx.x, gridDim.x);
    const int bx = blk % a.ntx, by = (blk / a.ntx) % a.nty, bz = blk / (a.ntx * a.nty);
    const int t = threadIdx.x;
    const int rx = a.tx + 2;
    const bool in_region = t < rx * (a.ty + 2);
    const int x = vort_cell(bx * a.tx - 1 + t % rx, nx, a.periodic & 1);
    const int y = vort_cell(by * a.ty - 1 + t / rx, ny, a.periodic & 2);
    const int ox = t % a.tx, oy = t / a.tx;
    const int X = bx * a.tx + ox, Y = by * a.ty + oy;
    const bool out = oy < a.ty && X < nx && Y < ny;
    const int centre = (oy + 1) * rx + ox + 1;
    int xlo, xhi, ylo, yhi;
    vort_points(X, nx, a.periodic & 1, xlo, xhi);
    vort_points(Y, ny, a.periodic & 2, ylo, yhi);
    const int z0 = bz * a.cz, z1 = min(z0 + a.cz, nz);
    for (int p = z0 - 1; p <= z1; ++p) {
        if (in_region) {
            const int64_t c = x + (int64_t)nx * y + nxy * vort_cell(p, nz, a.periodic & 4);
            float v[27];
#pragma unroll
            for (int i = 0; i < Q; ++i) v[tensor_slot(i)] = Io<T>::ld(f + i * P + c);
            float u[3];
            velocity(v, a.g, a.force, P, c, a.beta, a.s_ref, u);
#pragma unroll
            for (int k = 0; k < 3; ++k) ring[p & 3][k][t] = u[k];
        }
        __syncthreads();
        if (!out || p <= z0) continue;
        const int z = p - 1;
        int zlo, zhi;
        vort_points(z, nz, a.periodic & 4, zlo, zhi);
        const float (&here)[3][kVortThreads] = ring[z & 3];
        const float (&below)[3][kVortThreads] = ring[(z - zlo) & 3];
        const float (&above)[3][kVortThreads] = ring[(z + zhi) & 3];
        float grad[3][3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            grad[k][0] = vort_slope(here[k][centre + xhi], here[k][centre - xlo], xlo + xhi);
            grad[k][1] = vort_slope(here[k][centre + yhi * rx], here[k][centre - ylo * rx], ylo + yhi);
            grad[k][2] = vort_slope(above[k][centre], below[k][centre], zlo + zhi);
        }
        vort_store(a, X + (int64_t)nx * Y + nxy * z, grad, here[0][centre], here[1][centre], here[2][centre]);
    }
}

// The same for small boxes, whose walk along z would be a chain of memory round
// trips with few workgroups: one tile per workgroup, every cell of it and of
// one cell around it at once, one barrier.  Against the walk: 4.0 / 17.2 us at
// 16^3, 4.1 / 13.2 us at 32^3, 5.7 / 13.1 us at 48x48x40; bound by the launch
// and one round trip.
template <typename T, int TX, int TY, int TZ>
__global__ void __launch_bounds__(((TX + 2) * (TY + 2) * (TZ + 2) + 63) / 64 * 64)
    k_vorticity_box(const VortArgs a)
{
    constexpr int RX = TX + 2, RY = TY + 2, RZ = TZ + 2, R = RX * RY * RZ;
    __shared__ float u[3][R];
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const int64_t nxy = (int64_t)nx * ny;
    const int blk = xcd_block(blockIdx.x, gridDim.x);
    const int bx = blk % a.ntx, by = (blk / a.ntx) % a.nty, bz = blk / (a.ntx * a.nty);
    const int t = threadIdx.x;
    if (t < R) {
        const int64_t c = vort_cell(bx * TX - 1 + t % RX, nx, a.periodic & 1) +
                          (int64_t)nx * vort_cell(by * TY - 1 + t / RX % RY, ny, a.periodic & 2) +
                          nxy * vort_cell(bz * TZ - 1 + t / (RX * RY), nz, a.periodic & 4);
        const T* f = static_cast<const T*>(a.f);
        float v[27];
#pragma unroll
        for (int i = 0; i < Q; ++i) v[tensor_slot(i)] = Io<T>::ld(f + i * a.plane + c);
        float w[3];
        velocity(v, a.g, a.force, a.plane, c, a.beta, a.s_ref, w);
#pragma unroll
        for (int k = 0; k < 3; ++k) u[k][t] = w[k];
    }
    __syncthreads();
    const int ox = t % TX, oy = t / TX % TY, oz = t / (TX * TY);
    const int X = bx * TX + ox, Y = by * TY + oy, Z = bz * TZ + oz;
    if (oz >= TZ || X >= nx || Y >= ny || Z >= nz) return;
    const int centre = ((oz + 1) * RY + oy + 1) * RX + ox + 1;
    int xlo, xhi, ylo, yhi, zlo, zhi;
    vort_points(X, nx, a.periodic & 1, xlo, xhi);
    vort_points(Y, ny, a.periodic & 2, ylo, yhi);
    vort_points(Z, nz, a.periodic & 4, zlo, zhi);
    float grad[3][3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        grad[k][0] = vort_slope(u[k][centre + xhi], u[k][centre - xlo], xlo + xhi);
        grad[k][1] = vort_slope(u[k][centre + yhi * RX], u[k][centre - ylo * RX], ylo + yhi);
        grad[k][2] = vort_slope(u[k][centre + zhi * RX * RY], u[k][centre - zlo * RX * RY], zlo + zhi);
    }
    vort_store(a, X + (int64_t)nx * Y + nxy * Z, grad, u[0][centre], u[1][centre], u[2][centre]);
}

// Tiles and planes of k_vorticity.  Rows are cut into equal tiles of at most 64
// cells, and a tile has as many rows as the threads allow: with 64 x 8 tiles
// throughout, 2x600x600 took 253 us (34 in two passes, 26 so), 80x300x300 294
// (binary16; 229, 222).  The planes then follow from the workgroups a CU gets:
// it takes its turns at them plane by plane, and one alone leaves the memory
// idle at its barriers (65x200x200 with scalar: 115 us with one, 110 with two).
// False where a CU would get more than the three that fit, that is on flat
// boxes, whose tiles are many and read two planes more than they write
// (1024x1024x1: 58 us against 44 in two passes; 575x278x105: 669, 670), for
// binary16 rows of less than half a tile (24x393x519 166 us against 152;
// 20x524x186 50 against 56), and where the rims' scalar and force come from
// beyond the 256 MB of last-level cache too (142x282x362: 630 against 573; 80x300x300
// 308, 297; but 48x497x516 438, 519).
static bool plan_vorticity(VortArgs& a, bool half)
{
    constexpr int64_t cus = 256;
    if (half && a.nx < kVortWidth / 2) return false;
    const int64_t bytes = (int64_t)a.nx * a.ny * a.nz * (Q * (half ? 2 : 4) + QS * 4 + 12);
    if (a.g && a.force && bytes > (256 << 20)) return false;
    a.ntx = (a.nx + kVortWidth - 1) / kVortWidth;
    a.tx = (a.nx + a.ntx - 1) / a.ntx;
    const int rows = kVortThreads / (a.tx + 2) - 2;
    const int nt0 = (a.ny + rows - 1) / rows;
    double best = 1e300;
    int64_t share = 0;   // workgroups per CU
    for (int nty = nt0; nty <= 2 * nt0 && nty <= nt0 + 64 && nty <= a.ny; ++nty) {
        const int ty = (a.ny + nty - 1) / nty;
        const int64_t tiles = (int64_t)a.ntx * ((a.ny + ty - 1) / ty);
        const double plane = std::max(0.9, (a.tx + 2.0) * (ty + 2.0) * 5.6e-3);   // us
        const int64_t r0 = (tiles + cus - 1) / cus;
        for (int64_t r = r0; r < r0 + 4; ++r) {
            const int64_t chunks = std::min<int64_t>(a.nz, r * cus / tiles);
            const int cz = (int)((a.nz + chunks - 1) / chunks);
            const int64_t per_cu = (tiles * ((a.nz + cz - 1) / cz) + cus - 1) / cus;
            const double cost = (cz + 2.0) * (per_cu == 1 ? 1.35 : (double)per_cu) * plane;
            if (cost < best) {
                best = cost;
                share = per_cu;
                a.nty = (a.ny + ty - 1) / ty;
                a.ty = ty;
                a.cz = cz;
            }
        }
    }
    return share <= 3;
}

// the same from a dense velocity field [3][N]
__global__ void __launch_bounds__(256) k_curl(const VortArgs a, const float* u)
{
    const int64_t nxy = (int64_t)a.nx * a.ny, N = nxy * a.nz;
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= N) return;
    int p[3];
    cell_coords(c, a.nx, a.ny, p[0], p[1], p[2]);
    const int n[3] = {a.nx, a.ny, a.nz};
    const int64_t stride[3] = {1, a.nx, nxy};
    float grad[3][3];
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        const bool periodic = a.periodic & (1 << b);
        int lo, hi;
        vort_points(p[b], n[b], periodic, lo, hi);
        const int64_t cl = c + (vort_cell(p[b] - lo, n[b], periodic) - p[b]) * stride[b];
        const int64_t ch = c + (vort_cell(p[b] + hi, n[b], periodic) - p[b]) * stride[b];
#pragma unroll
        for (int k = 0; k < 3; ++k) grad[k][b] = vort_slope(u[k * N + ch], u[k * N + cl], lo + hi);
    }
    vort_store(a, c, grad, u[c], u[N + c], u[2 * N + c]);
}

static int vorticity_two_passes(const cslbm_level* L, const VortArgs& a, hipStream_t stream)
{
    const int64_t N = cells_of(L);
    float* u = nullptr;
    CSLBM_HIP_TRY(hipMallocAsync((void**)&u, 3 * N * sizeof(float), stream));
    const dim3 grid((unsigned)((N + 255) / 256)), block(256);
    if (L->storage == CSLBM_F32)
        hipLaunchKernelGGL(k_macro<float>, grid, block, 0, stream, (const float*)L->f, L->g, L->force, N,
                           L->plane, a.beta, a.s_ref, nullptr, u, nullptr);
    else
        hipLaunchKernelGGL(k_macro<_Float16>, grid, block, 0, stream, (const _Float16*)L->f, L->g, L->force,
                           N, L->plane, a.beta, a.s_ref, nullptr, u, nullptr);
    int rc = check_launch("k_macro");
    if (!rc) {
        hipLaunchKernelGGL(k_curl, grid, block, 0, stream, a, u);
        rc = check_launch("k_curl");
    }
    const hipError_t ef = hipFreeAsync(u, stream);
    if (rc) return rc;
    if (ef != hipSuccess) return fail(CSLBM_ERR_HIP, "hipFreeAsync: %s", hipGetErrorString(ef));
    return CSLBM_OK;
}

template <int TX, int TY, int TZ>
static void launch_vorticity_box(VortArgs a, bool half, hipStream_t st)
{
    a.ntx = (a.nx + TX - 1) / TX;
    a.nty = (a.ny + TY - 1) / TY;
    const dim3 grid((unsigned)((int64_t)a.ntx * a.nty * ((a.nz + TZ - 1) / TZ)));
    const dim3 block(((TX + 2) * (TY + 2) * (TZ + 2) + 63) / 64 * 64);
    if (half)
        hipLaunchKernelGGL((k_vorticity_box<_Float16, TX, TY, TZ>), grid, block, 0, st, a);
    else
        hipLaunchKernelGGL((k_vorticity_box<float, TX, TY, TZ>), grid, block, 0, st, a);
}

// FP64 conservation: per-block partial sums (count, sum h, sum c h, sum g),
// then one block adds the partials in a fixed order.
constexpr int kRedBlocks = 1024;
constexpr int kRedThreads = 256;
constexpr int kRedVals = 6;

template <typename T>
__global__ void __launch_bounds__(kRedThreads)
    k_conserved_partials(const T* f, const float* g, const uint8_t* flags, int64_t N, int64_t P,
                         double* partials)
{
    double acc[kRedVals] = {0, 0, 0, 0, 0, 0};
    for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < N;
         c += (int64_t)gridDim.x * blockDim.x) {
        if (flags) {
            const int kind = flags[c] & kKindMask;
            if (kind == kSolid || kind == kGhost) continue;
        }
        double dr = 0.0, jx = 0.0, jy = 0.0, jz = 0.0;
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            const double h = (double)Io<T>::ld(f + i * P + c);
            dr += h;
            jx += kCx[i] * h;
            jy += kCy[i] * h;
            jz += kCz[i] * h;
        }
        double sc = 0.0;
        if (g)
#pragma unroll
            for (int i = 0; i < QS; ++i) sc += (double)g[i * P + c];
        acc[0] += 1.0;
        acc[1] += dr;
        acc[2] += jx;
        acc[3] += jy;
        acc[4] += jz;
        acc[5] += sc;
    }
    __shared__ double sm[kRedVals][kRedThreads];
#pragma unroll
    for (int k = 0; k < kRedVals; ++k) sm[k][threadIdx.x] = acc[k];
    __syncthreads();
    for (int w = kRedThreads / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
#pragma unroll
            for (int k = 0; k < kRedVals; ++k) sm[k][threadIdx.x] += sm[k][threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0)
#pragma unroll
        for (int k = 0; k < kRedVals; ++k) partials[blockIdx.x * kRedVals + k] = sm[k][0];
}

__global__ void __launch_bounds__(kRedThreads) k_conserved_final(const double* partials, int nblocks,
                                                                 double* out)
{
    double acc[kRedVals] = {0, 0, 0, 0, 0, 0};
    for (int b = threadIdx.x; b < nblocks; b += blockDim.x)
#pragma unroll
        for (int k = 0; k < kRedVals; ++k) acc[k] += partials[b * kRedVals + k];
    __shared__ double sm[kRedVals][kRedThreads];
#pragma unroll
    for (int k = 0; k < kRedVals; ++k) sm[k][threadIdx.x] = acc[k];
    __syncthreads();
    for (int w = kRedThreads / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
#pragma unroll
            for (int k = 0; k < kRedVals; ++k) sm[k][threadIdx.x] += sm[k][threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        out[0] = sm[0][0] + sm[1][0];   // sum rho = cells + sum h
        out[1] = sm[2][0];
        out[2] = sm[3][0];
        out[3] = sm[4][0];
        out[4] = sm[5][0];
    }
}

// Scratch of the allocation-free conservation call: the per-block partials
// of k_conserved_partials (every block writes its own entries, so nothing
// needs clearing between calls).  One copy per GPU, held until the process
// ends; host code uses the device address from hipGetSymbolAddress, never
// the symbol itself.
constexpr int64_t kScratchDoubles = (int64_t)kRedBlocks * kRedVals;
static __device__ __align__(256) double scratch[kScratchDoubles];

constexpr int kMaxDevices = 64;
static double* g_scratch_ptr[kMaxDevices] = {};
static std::mutex g_scratch_mutex;

// Device address of `scratch` on the current device, looked up once per
// device (with that device current).
static int scratch_of_current_device(double** out)
{
    int dev = -1;
    CSLBM_HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices)
        return fail(CSLBM_ERR_UNSUPPORTED, "device index %d outside [0, %d)", dev, kMaxDevices);
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr)
            return fail(CSLBM_ERR_HIP, "hipGetSymbolAddress(scratch) on device %d: %s", dev,
                        hipGetErrorString(e));
        g_scratch_ptr[dev] = static_cast<double*>(ptr);
    }
    *out = g_scratch_ptr[dev];
    return CSLBM_OK;
}

template <typename T>
__global__ void k_count_nonfinite(const T* f, const float* g, int64_t N, int64_t P,
                                  unsigned long long* count)
{
    unsigned long long bad = 0;
    for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < N;
         c += (int64_t)gridDim.x * blockDim.x) {
#pragma unroll
        for (int i = 0; i < Q; ++i) bad += !isfinite(Io<T>::ld(f + i * P + c));
        if (g)
#pragma unroll
            for (int i = 0; i < QS; ++i) bad += !isfinite(g[i * P + c]);
    }
    if (bad) atomicAdd(count, bad);
}

// ---------------------------------------------------------------------------
// host side: validation and launches
// ---------------------------------------------------------------------------
int64_t cells_of(const cslbm_level* L)
{
    return L->brick_table ? (int64_t)L->n_bricks * kBrickCells : (int64_t)L->nx * L->ny * L->nz;
}

BrickMap brick_map(const cslbm_level* L)
{
    BrickMap m;
    m.table = L->brick_table;
    m.origin = L->brick_origin;
    m.bnx = L->nx / kBrickEdge;
    m.bny = L->ny / kBrickEdge;
    m.bnz = L->nz / kBrickEdge;
    return m;
}

int validate_shape(const cslbm_level* L)
{
    if (!L) return fail(CSLBM_ERR_ARG, "level is NULL");
    if (L->nx < 1 || L->ny < 1 || L->nz < 1)
        return fail(CSLBM_ERR_SHAPE, "level size %d x %d x %d must be positive", L->nx, L->ny, L->nz);
    const int64_t N = cells_of(L);
    if (N > 0x7fffffffLL)
        return fail(CSLBM_ERR_SHAPE, "level has %lld cells; at most 2^31-1 are supported",
                    (long long)N);
    if (L->nz > 65535 || L->ny > 65535)
        return fail(CSLBM_ERR_SHAPE, "ny and nz must be at most 65535");
    if (L->plane < N)
        return fail(CSLBM_ERR_SHAPE, "plane stride %lld is smaller than nx*ny*nz = %lld",
                    (long long)L->plane, (long long)N);
    if (L->storage != CSLBM_F32 && L->storage != CSLBM_F16S)
        return fail(CSLBM_ERR_UNSUPPORTED, "unknown storage format %d", L->storage);
    if (!L->f) return fail(CSLBM_ERR_ARG, "f is NULL");
    if ((L->g == nullptr) != (L->g_next == nullptr))
        return fail(CSLBM_ERR_ARG, "g and g_next must both be set or both be NULL");
    if ((L->periodic & 7) != 7 && !L->flags)
        return fail(CSLBM_ERR_ARG, "a non-periodic axis needs a flags array (periodic = %d)",
                    L->periodic);
    if (L->wall_cells < 0 || (L->wall_cells > 0 && !L->flags))
        return fail(CSLBM_ERR_ARG, "wall_cells = %d needs a flags array holding them", L->wall_cells);
    if (L->brick_table) {
        if (L->nx % kBrickEdge || L->ny % kBrickEdge || L->nz % kBrickEdge)
            return fail(CSLBM_ERR_SHAPE, "a brick level's box %d x %d x %d must be a multiple of 8",
                        L->nx, L->ny, L->nz);
        const int64_t nb = (int64_t)(L->nx / 8) * (L->ny / 8) * (L->nz / 8);
        if (L->n_bricks < 1 || L->n_bricks > nb)
            return fail(CSLBM_ERR_ARG, "n_bricks = %d outside [1, %lld]", L->n_bricks, (long long)nb);
        if (!L->brick_origin) return fail(CSLBM_ERR_ARG, "brick_origin is NULL");
        if (!L->flags) return fail(CSLBM_ERR_ARG, "a brick level needs flags");
        if (L->periodic & 7) return fail(CSLBM_ERR_UNSUPPORTED, "a brick level has no periodic axis");
        if (L->force) return fail(CSLBM_ERR_UNSUPPORTED, "a brick level has no force field");
    }
    return CSLBM_OK;
}

int validate_params(const cslbm_level* L)
{
    const cslbm_params& p = L->p;
    if (!(p.nu > 0.0) || !std::isfinite(p.nu))
        return fail(CSLBM_ERR_ARG, "viscosity nu = %g must be positive (S4..8 in (0, 2))", p.nu);
    for (int g = 0; g < 4; ++g)
        if (!(p.nu_hi[g] > 0.0) || !std::isfinite(p.nu_hi[g]))
            return fail(CSLBM_ERR_ARG, "artificial viscosity nu_hi[%d] = %g must be positive", g,
                        p.nu_hi[g]);
    if (p.adaptive) {
        if (!(p.g_max > 0.0)) return fail(CSLBM_ERR_ARG, "g_max = %g must be positive", p.g_max);
        if (!(p.b > 0.0) || !(p.a + p.b > 0.0))
            return fail(CSLBM_ERR_ARG,
                        "adaptive factor a*x + b must stay positive on [0, 1] (a = %g, b = %g)",
                        p.a, p.b);
    }
    if (L->g && !(p.tau_s > 0.5))
        return fail(CSLBM_ERR_ARG, "scalar relaxation time tau_s = %g must exceed 1/2", p.tau_s);
    if (p.grad_mode != 0 && p.grad_mode != 1)
        return fail(CSLBM_ERR_ARG, "grad_mode = %d must be 0 or 1", p.grad_mode);
    if (p.gmax_running && p.grad_mode != 1)
        return fail(CSLBM_ERR_ARG, "gmax_running needs grad_mode 1");
    return CSLBM_OK;
}

static inline unsigned blocks_for(int64_t n, int threads) { return (unsigned)((n + threads - 1) / threads); }

// After the state of a gradient-mode level was written: its velocity field.
static int refresh_velocity(const cslbm_level* L, hipStream_t stream)
{
    if (L->p.grad_mode != 1 || !L->vel) return CSLBM_OK;
    const int64_t N = cells_of(L);
    const dim3 grid(blocks_for(N, 256)), block(256);
    const float beta = (float)L->p.beta, sref = (float)L->p.s_ref;
    if (L->storage == CSLBM_F32)
        hipLaunchKernelGGL(k_macro<float>, grid, block, 0, stream, (const float*)L->f, L->g, L->force,
                           N, L->plane, beta, sref, nullptr, L->vel, nullptr);
    else
        hipLaunchKernelGGL(k_macro<_Float16>, grid, block, 0, stream, (const _Float16*)L->f, L->g,
                           L->force, N, L->plane, beta, sref, nullptr, L->vel, nullptr);
    return check_launch("k_macro");
}

Rates make_rates(const cslbm_params& p)
{
    Rates r;
    r.S = (float)(1.0 / (3.0 * p.nu + 0.5));
    for (int g = 0; g < 4; ++g) r.nu3[g] = (float)(3.0 * p.nu_hi[g]);
    r.a = (float)p.a;
    r.b = (float)p.b;
    r.inv_gmax = p.adaptive ? (float)(1.0 / p.g_max) : 0.0f;
    r.adaptive = p.adaptive ? 1 : 0;
    return r;
}

// Block of 256 threads: bx consecutive x (a multiple of 64, so waves cover
// contiguous row segments) by 256/bx rows.  bx is the largest of 256, 128, 64
// that leaves the fewest idle lanes per row (nx = 384 -> 128, nx = 512 ->
// 256, nx = 96 -> 128).
}  // namespace cslbm

using namespace cslbm;

extern "C" {

int64_t cslbm_plane_stride(int32_t nx, int32_t ny, int32_t nz)
{
    if (nx < 1 || ny < 1 || nz < 1) return fail(CSLBM_ERR_SHAPE, "sizes must be positive");
    const int64_t N = (int64_t)nx * ny * nz;
    // round up to 256 elements and add 3*256 so consecutive planes start at
    // offsets that differ by an odd number of 1 KiB blocks
    return ((N + 255) / 256) * 256 + 3 * 256;
}

int64_t cslbm_level_bytes(int32_t nx, int32_t ny, int32_t nz, int32_t storage, int32_t with_scalar)
{
    const int64_t plane = cslbm_plane_stride(nx, ny, nz);
    if (plane < 0) return plane;
    if (storage != CSLBM_F32 && storage != CSLBM_F16S)
        return fail(CSLBM_ERR_UNSUPPORTED, "unknown storage format %d", storage);
    const int64_t elem = storage == CSLBM_F32 ? 4 : 2;
    return 27 * plane * elem + (with_scalar ? 7 * plane * 4 : 0);
}

int cslbm_prepare_flags(const cslbm_level* L, hipStream_t stream)
{
    int rc = validate_shape(L);
    if (rc) return rc;
    if (!L->flags) return fail(CSLBM_ERR_ARG, "flags is NULL");
    const int64_t N = cells_of(L);
    hipLaunchKernelGGL(k_prepare_flags, dim3(blocks_for(N, 256)), dim3(256), 0, stream, L->flags,
                       L->links, L->nx, L->ny, L->nz, L->periodic, N, brick_map(L));
    return check_launch("k_prepare_flags");
}

int cslbm_init_equilibrium(cslbm_level* L, const float* rho, const float* u, const float* s,
                           hipStream_t stream)
{
    int rc = validate_shape(L);
    if (rc) return rc;
    if (!u) return fail(CSLBM_ERR_ARG, "u is NULL");
    const int64_t N = cells_of(L);
    const dim3 grid(blocks_for(N, 256)), block(256);
    if (L->storage == CSLBM_F32)
        hipLaunchKernelGGL(k_init_eq<float>, grid, block, 0, stream, (float*)L->f, L->g, N, L->plane,
                           rho, u, s);
    else
        hipLaunchKernelGGL(k_init_eq<_Float16>, grid, block, 0, stream, (_Float16*)L->f, L->g, N,
                           L->plane, rho, u, s);
    rc = check_launch("k_init_eq");
    return rc ? rc : refresh_velocity(L, stream);
}

int cslbm_set_populations(cslbm_level* L, const float* f, const float* g, int32_t shifted,
                          hipStream_t stream)
{
    int rc = validate_shape(L);
    if (rc) return rc;
    if (!f) return fail(CSLBM_ERR_ARG, "source populations are NULL");
    const int64_t N = cells_of(L);
    const dim3 grid(blocks_for(N, 256)), block(256);
    if (L->storage == CSLBM_F32)
        hipLaunchKernelGGL(k_set_pop<float>, grid, block, 0, stream, (float*)L->f, L->g, N, L->plane,
                           f, g, shifted);
    else
        hipLaunchKernelGGL(k_set_pop<_Float16>, grid, block, 0, stream, (_Float16*)L->f, L->g, N,
                           L->plane, f, g, shifted);
    rc = check_launch("k_set_pop");
    return rc ? rc : refresh_velocity(L, stream);
}

int cslbm_get_populations(const cslbm_level* L, float* f, float* g, int32_t shifted,
                          hipStream_t stream)
{
    int rc = validate_shape(L);
    if (rc) return rc;
    if (!f) return fail(CSLBM_ERR_ARG, "destination is NULL");
    const int64_t N = cells_of(L);
    const dim3 grid(blocks_for(N, 256)), block(256);
    if (L->storage == CSLBM_F32)
        hipLaunchKernelGGL(k_get_pop<float>, grid, block, 0, stream, (const float*)L->f, L->g, N,
                           L->plane, f, g, shifted);
    else
        hipLaunchKernelGGL(k_get_pop<_Float16>, grid, block, 0, stream, (const _Float16*)L->f, L->g,
                           N, L->plane, f, g, shifted);
    return check_launch("k_get_pop");
}

int cslbm_copy_cells(const cslbm_level* src, const int32_t* src_cells, cslbm_level* dst,
                     const int32_t* dst_cells, int32_t n_cells, hipStream_t stream)
{
    int rc = validate_shape(src);
    if (rc) return rc;
    rc = validate_shape(dst);
    if (rc) return rc;
    if (src->storage != dst->storage)
        return fail(CSLBM_ERR_UNSUPPORTED, "copying between storage formats is not supported");
    if (n_cells < 0 || (n_cells > 0 && (!src_cells || !dst_cells)))
        return fail(CSLBM_ERR_ARG, "bad cell lists");
    if ((src->g != nullptr) != (dst->g != nullptr))
        return fail(CSLBM_ERR_ARG, "both levels or neither must carry the scalar");
    if (src->f == dst->f) return fail(CSLBM_ERR_ARG, "source and destination states alias");
    if (n_cells == 0) return CSLBM_OK;
    const dim3 grid(blocks_for(n_cells, 256)), block(256);
    if (src->storage == CSLBM_F32)
        hipLaunchKernelGGL(k_copy_cells<float>, grid, block, 0, stream, (const float*)src->f, src->g,
                           src->plane, (float*)dst->f, dst->g, dst->plane, src_cells, dst_cells,
                           n_cells);
    else
        hipLaunchKernelGGL(k_copy_cells<_Float16>, grid, block, 0, stream, (const _Float16*)src->f,
                           src->g, src->plane, (_Float16*)dst->f, dst->g, dst->plane, src_cells,
                           dst_cells, n_cells);
    return check_launch("k_copy_cells");
}

int cslbm_step(cslbm_level* L, int32_t n_steps, hipStream_t stream)
{
    int rc = validate_shape(L);
    if (rc) return rc;
    rc = validate_params(L);
    if (rc) return rc;
    if (n_steps < 0) return fail(CSLBM_ERR_ARG, "n_steps = %d is negative", n_steps);
    if (!L->f_next) return fail(CSLBM_ERR_ARG, "f_next is NULL");
    if (L->f == L->f_next) return fail(CSLBM_ERR_ARG, "f and f_next alias");
    if (L->g && L->g == L->g_next) return fail(CSLBM_ERR_ARG, "g and g_next alias");
    const bool grad = L->p.grad_mode == 1;
    if (grad) {
        if (L->flags)
            return fail(CSLBM_ERR_UNSUPPORTED,
                        "the finite-difference gradient mode needs a fully periodic level without flags");
        if (!L->vel || !L->vel_next || L->vel == L->vel_next)
            return fail(CSLBM_ERR_ARG, "grad_mode 1 needs distinct vel and vel_next buffers");
        if (L->p.gmax_running && !L->gmax_buf)
            return fail(CSLBM_ERR_ARG, "gmax_running needs gmax_buf");
    }

    auto swap_buffers = [&]() {
        std::swap(L->f, L->f_next);
        std::swap(L->g, L->g_next);
    };
    int n = 0;
    // fused pairs: an even number of them, so that the buffers' roles after
    // n_steps are those of n_steps single steps, and at least one single step
    // after them, so that f_next holds the state before the last step
    if (n_steps >= 5 && step_pair_kind(L) != PairKind::kNone)
        for (const int paired = (n_steps - 1) / 4 * 4; n < paired; n += 2) {
            rc = launch_step_pair(L, L->f, L->f_next, L->g, L->g_next, stream);
            if (rc) return rc;
            swap_buffers();
        }
    for (; n < n_steps; ++n) {
        rc = grad ? launch_step_grad(L, L->f, L->f_next, L->g, L->g_next, L->vel, L->vel_next, stream)
                  : launch_step_into(L, L->f, L->f_next, L->g, L->g_next, stream);
        if (rc) return rc;
        if (grad) std::swap(L->vel, L->vel_next);
        swap_buffers();
    }
    return CSLBM_OK;
}

int cslbm_read_macro(const cslbm_level* L, float* rho, float* u, float* s, hipStream_t stream)
{
    int rc = validate_shape(L);
    if (rc) return rc;
    if (s && !L->g) return fail(CSLBM_ERR_ARG, "scalar requested but the level has no g");
    const int64_t N = cells_of(L);
    const dim3 grid(blocks_for(N, 256)), block(256);
    const float beta = (float)L->p.beta, sref = (float)L->p.s_ref;
    if (L->storage == CSLBM_F32)
        hipLaunchKernelGGL(k_macro<float>, grid, block, 0, stream, (const float*)L->f, L->g, L->force,
                           N, L->plane, beta, sref, rho, u, s);
    else
        hipLaunchKernelGGL(k_macro<_Float16>, grid, block, 0, stream, (const _Float16*)L->f, L->g,
                           L->force, N, L->plane, beta, sref, rho, u, s);
    return check_launch("k_macro");
}

int cslbm_vorticity(const cslbm_level* L, float* omega, float* speed, hipStream_t stream)
{
    int rc = validate_shape(L);
    if (rc) return rc;
    if (L->brick_table) return fail(CSLBM_ERR_UNSUPPORTED, "vorticity of a brick level");
    if (!omega) return fail(CSLBM_ERR_ARG, "omega is NULL");
    VortArgs a;
    a.f = L->f;
    a.g = L->g;
    a.force = L->force;
    a.nx = L->nx;
    a.ny = L->ny;
    a.nz = L->nz;
    a.periodic = L->periodic & 7;
    a.plane = L->plane;
    a.beta = (float)L->p.beta;
    a.s_ref = (float)L->p.s_ref;
    a.out = omega;
    a.speed = speed;
    // small boxes: the smallest tile that gives a CU one workgroup at most
    // (48x48x40: 16x6x4 5.7 us, 16x4x4 6.9, 8x4x4 7.8), 16x4x4 for a few more;
    // at 1024 of those the walk is as fast (64^3: 12.5 against 13.4 us)
    auto tiles_of = [&](int tx, int ty) {
        return (int64_t)blocks_for(L->nx, tx) * blocks_for(L->ny, ty) * blocks_for(L->nz, 4);
    };
    const bool half = L->storage != CSLBM_F32;
    const int64_t wide = tiles_of(16, 4);
    if (wide <= 768) {
        if (tiles_of(8, 4) <= 256)
            launch_vorticity_box<8, 4, 4>(a, half, stream);
        else if (wide > 256 && tiles_of(16, 6) <= 256)
            launch_vorticity_box<16, 6, 4>(a, half, stream);
        else
            launch_vorticity_box<16, 4, 4>(a, half, stream);
        return check_launch("k_vorticity_box");
    }
    if (!plan_vorticity(a, half)) return vorticity_two_passes(L, a, stream);
    const dim3 grid((unsigned)((int64_t)a.ntx * a.nty * ((L->nz + a.cz - 1) / a.cz)));
    const dim3 block((unsigned)(((a.tx + 2) * (a.ty + 2) + 63) / 64 * 64));
    if (half)
        hipLaunchKernelGGL(k_vorticity<_Float16>, grid, block, 0, stream, a);
    else
        hipLaunchKernelGGL(k_vorticity<float>, grid, block, 0, stream, a);
    return check_launch("k_vorticity");
}

int cslbm_conserved_f64(const cslbm_level* L, double out[5], hipStream_t stream)
{
    int rc = validate_shape(L);
    if (rc) return rc;
    if (!out) return fail(CSLBM_ERR_ARG, "out is NULL");
    const int64_t N = cells_of(L);
    double* dmem = nullptr;
    CSLBM_HIP_TRY(hipMallocAsync((void**)&dmem, (kRedBlocks * kRedVals + 8) * sizeof(double), stream));
    double* partials = dmem;
    double* dout = dmem + kRedBlocks * kRedVals;
    if (L->storage == CSLBM_F32)
        hipLaunchKernelGGL(k_conserved_partials<float>, dim3(kRedBlocks), dim3(kRedThreads), 0, stream,
                           (const float*)L->f, L->g, L->flags, N, L->plane, partials);
    else
        hipLaunchKernelGGL(k_conserved_partials<_Float16>, dim3(kRedBlocks), dim3(kRedThreads), 0,
                           stream, (const _Float16*)L->f, L->g, L->flags, N, L->plane, partials);
    rc = check_launch("k_conserved_partials");
    if (!rc) {
        hipLaunchKernelGGL(k_conserved_final, dim3(1), dim3(kRedThreads), 0, stream, partials,
                           kRedBlocks, dout);
        rc = check_launch("k_conserved_final");
    }
    double host[5] = {0, 0, 0, 0, 0};
    if (!rc) {
        const hipError_t e = hipMemcpyAsync(host, dout, sizeof host, hipMemcpyDeviceToHost, stream);
        if (e != hipSuccess) rc = fail(CSLBM_ERR_HIP, "copy of the totals: %s", hipGetErrorString(e));
    }
    const hipError_t ef = hipFreeAsync(dmem, stream);
    const hipError_t es = hipStreamSynchronize(stream);
    if (rc) return rc;
    if (ef != hipSuccess) return fail(CSLBM_ERR_HIP, "hipFreeAsync: %s", hipGetErrorString(ef));
    if (es != hipSuccess) return fail(CSLBM_ERR_HIP, "hipStreamSynchronize: %s", hipGetErrorString(es));
    std::memcpy(out, host, sizeof host);
    return CSLBM_OK;
}

int cslbm_conserved_f64_noalloc(const cslbm_level* L, double* totals, hipStream_t stream)
{
    int rc = validate_shape(L);
    if (rc) return rc;
    if (!totals) return fail(CSLBM_ERR_ARG, "totals is NULL");
    // the reduction grid is fixed (grid-stride loop), so every level fits
    static_assert((int64_t)kRedBlocks * kRedVals <= kScratchDoubles, "partials exceed the scratch");
    double* partials = nullptr;
    rc = scratch_of_current_device(&partials);
    if (rc) return rc;
    const int64_t N = cells_of(L);
    if (L->storage == CSLBM_F32)
        hipLaunchKernelGGL(k_conserved_partials<float>, dim3(kRedBlocks), dim3(kRedThreads), 0, stream,
                           (const float*)L->f, L->g, L->flags, N, L->plane, partials);
    else
        hipLaunchKernelGGL(k_conserved_partials<_Float16>, dim3(kRedBlocks), dim3(kRedThreads), 0,
                           stream, (const _Float16*)L->f, L->g, L->flags, N, L->plane, partials);
    rc = check_launch("k_conserved_partials");
    if (rc) return rc;
    hipLaunchKernelGGL(k_conserved_final, dim3(1), dim3(kRedThreads), 0, stream, partials,
                       kRedBlocks, totals);
    return check_launch("k_conserved_final");
}

int cslbm_check_finite(const cslbm_level* L, int64_t* n_bad, hipStream_t stream)
{
    int rc = validate_shape(L);
    if (rc) return rc;
    if (!n_bad) return fail(CSLBM_ERR_ARG, "n_bad is NULL");
    const int64_t N = cells_of(L);
    unsigned long long* dcount = nullptr;
    CSLBM_HIP_TRY(hipMallocAsync((void**)&dcount, sizeof(unsigned long long), stream));
    rc = CSLBM_OK;
    hipError_t e = hipMemsetAsync(dcount, 0, sizeof(unsigned long long), stream);
    if (e != hipSuccess) rc = fail(CSLBM_ERR_HIP, "hipMemsetAsync: %s", hipGetErrorString(e));
    if (!rc) {
        const unsigned nb = (unsigned)std::min<int64_t>(blocks_for(N, 256), 4096);
        if (L->storage == CSLBM_F32)
            hipLaunchKernelGGL(k_count_nonfinite<float>, dim3(nb), dim3(256), 0, stream,
                               (const float*)L->f, L->g, N, L->plane, dcount);
        else
            hipLaunchKernelGGL(k_count_nonfinite<_Float16>, dim3(nb), dim3(256), 0, stream,
                               (const _Float16*)L->f, L->g, N, L->plane, dcount);
        rc = check_launch("k_count_nonfinite");
    }
    unsigned long long host = 0;
    if (!rc) {
        e = hipMemcpyAsync(&host, dcount, sizeof host, hipMemcpyDeviceToHost, stream);
        if (e != hipSuccess) rc = fail(CSLBM_ERR_HIP, "copy of the count: %s", hipGetErrorString(e));
    }
    const hipError_t ef = hipFreeAsync(dcount, stream);
    const hipError_t es = hipStreamSynchronize(stream);
    if (rc) return rc;
    if (ef != hipSuccess) return fail(CSLBM_ERR_HIP, "hipFreeAsync: %s", hipGetErrorString(ef));
    if (es != hipSuccess) return fail(CSLBM_ERR_HIP, "hipStreamSynchronize: %s", hipGetErrorString(es));
    *n_bad = (int64_t)host;
    if (host) return fail(CSLBM_ERR_NONFINITE, "%llu non-finite values in the state", host);
    return CSLBM_OK;
}

int cslbm_abi_sizes(int64_t* params_bytes, int64_t* level_bytes, int64_t* scale_bytes)
{
    if (params_bytes) *params_bytes = (int64_t)sizeof(cslbm_params);
    if (level_bytes) *level_bytes = (int64_t)sizeof(cslbm_level);
    if (scale_bytes) *scale_bytes = (int64_t)sizeof(cslbm_scale);
    return CSLBM_OK;
}

const char* cslbm_last_error(void) { return g_last_error.c_str(); }

}  // extern "C"
