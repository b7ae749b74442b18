// step_pair.hip -- two collide-stream steps of a fully periodic FP32 level in
// one pass over memory (gfx950).
//
// k_step is bound by HBM: 27 reads and 27 writes per lattice update, at the
// rate its access pattern reaches without any arithmetic.  Here a workgroup
// walks a column of cells (a TX x TY tile of the x-y plane) along z.  For
// every plane it computes the first step on the tile and one cell around it
// (one thread per cell), puts the new populations of that plane into LDS, and
// its output threads take the second step's pulled populations from there:
// those with c_z = -1 complete the output plane below, those with c_z = 0 and
// +1 wait in 27 registers for the planes to come.  A pair of steps reads the
// state once and writes it once; what it pays is the first step of the
// halo cells (a tile's perimeter, and two planes per workgroup).  Small levels
// take k_step_pair_box below.
//
// Two planes of LDS where they fit (without the scalar): one barrier a plane,
// and waves may run a plane's first step while others are at the second step
// of the plane before.  One plane and two barriers: 424 -> 457 us per step at
// 256^3.  The next plane's loads are issued before the barrier, as soon as
// the plane in the registers is in LDS (after it: 457 -> 490 us); earlier
// they need 27 more registers, which spill at four waves per SIMD, and at three
// were slower (530-580 us).
//
// What bounds it: VALU issue, busy 79-81 % of the time at 256^3; HBM moves
// 4.5-5.1 TB/s (over cards: the halo lines that are read again vary).  Per step, pair against k_step: 418 / 645 us at 256^3, 55 / 83 us
// at 128^3, 60 / 104 us at 181x118x77 (rows off the cache lines), 28 / 38 us
// at 96^3; with force and scalar 76 / 108 us at 128^3.  binary16 levels stay
// with k_step: it already issues VALU instructions 87 % of the time.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "../../include/cslbm.h"
#include "cm_collide.hpp"
#include "exchange.hpp"
#include "internal.hpp"
#include "lattice.hpp"

namespace cslbm {

struct PairArgs {
    const float* f;
    float* fo;
    const float* g;
    float* go;
    const float* force;
    int nx, ny, nz;
    int ntx, nty;   // tiles along x and y
    int ty;         // rows of a tile (at most TY)
    int cz;         // output planes of a workgroup
    int64_t plane;
    Rates r;
    float beta, s_ref, inv_tau_s;
};

template <int TX, int TY>
struct PairShape {
    static constexpr int RX = TX + 2, RY = TY + 2;
    static constexpr int kRegion = RX * RY;   // first-step cells of a plane
    static constexpr int kThreads = (kRegion + 63) / 64 * 64;   // of a full-height tile
};

// Uniform plane bases stay in one SGPR pair that walks from plane to plane,
// and a lane adds its 32-bit byte offset.  The empty asm statements keep the
// compiler from forming 27 bases ahead of the z loop (they spilled into
// VGPR lanes) or one 64-bit lane address per plane.
using GlobalFloat = __attribute__((address_space(1))) float;
using GlobalChar = __attribute__((address_space(1))) char;

struct PlaneWalk {
    int64_t at = 0, step;   // bytes
    __device__ __forceinline__ explicit PlaneWalk(int64_t plane) : step(plane * 4) {}
    __device__ __forceinline__ void next()
    {
        at += step;
        asm volatile("" : "+s"(at));
    }
    __device__ __forceinline__ GlobalFloat* lane(const float* base, uint32_t off) const
    {
        GlobalChar* b = (GlobalChar*)base + at;
        asm volatile("" : "+s"(b));
        return (GlobalFloat*)(b + off);
    }
};

// The cell update of k_step on pulled populations, bit for bit, in the two
// halves of cm_collide; the scalar's update is in the second.  Neither half has
// a branch (pair_args folds adaptive = 0 into a and b), since the compiler
// fuses multiplications into additions inside one basic block only.
struct PulledCell {
    CellMomentum m;
    float F[3], s;
};

template <bool kScalar>
__device__ __forceinline__ PulledCell pulled_transform(const PairArgs& a, float (&v)[27],
                                                       const float (&gv)[QS], const float (&F)[3])
{
    PulledCell c{{}, {F[0], F[1], F[2]}, 0.0f};
    if (kScalar) {
        c.s = (gv[0] + (gv[1] + gv[2])) + ((gv[3] + gv[4]) + (gv[5] + gv[6]));
        c.F[2] += a.beta * (c.s - a.s_ref);
    }
    c.m = cm_collide_transform(v, c.F[0], c.F[1], c.F[2]);
    return c;
}

// Ends the first half here where the second stands behind a branch, which
// would draw any part of the first into itself.
__device__ __forceinline__ void pin(float (&v)[27], CellMomentum& m)
{
#pragma unroll
    for (int q = 0; q < 27; ++q) asm volatile("" : "+v"(v[q]));
    asm volatile("" : "+v"(m.px));
    asm volatile("" : "+v"(m.py));
    asm volatile("" : "+v"(m.pz));
}

template <bool kScalar>
__device__ __forceinline__ void pulled_relax(const PairArgs& a, const PulledCell& c, float (&v)[27],
                                             float (&gv)[QS])
{
    Rates r = a.r;
    r.adaptive = 1;
    const CellMacro mc = cm_collide_relax(v, c.m, r, c.F[0], c.F[1], c.F[2]);
    if (kScalar)
#pragma unroll
        for (int i = 0; i < QS; ++i) {
            const float ge = scalar_eq(i, c.s, mc.ux, mc.uy, mc.uz);
            gv[i] = gv[i] - (gv[i] - ge) * a.inv_tau_s;
        }
}

template <bool kForce, bool kScalar, int TX, int TY, int kWaves>
__global__ void __launch_bounds__((PairShape<TX, TY>::kThreads))
    __attribute__((amdgpu_waves_per_eu(kWaves))) k_step_pair(const PairArgs a)
{
    using S = PairShape<TX, TY>;
    constexpr int R = S::kRegion;
    constexpr int kPlane = (kScalar ? Q + QS : Q) * R;   // floats of a first-step plane
    constexpr bool kTwo = 2 * kPlane * sizeof(float) <= 160 * 1024;
    __shared__ float lds[kPlane * (kTwo ? 2 : 1)];

    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const int64_t nxy = (int64_t)nx * ny;
    const int64_t P = a.plane;
    // x-fastest tiles, each XCD a contiguous range: neighbouring tiles walk z
    // side by side on one XCD and find their shared lines in its L2
    const int blk = xcd_block(blockIdx.x, gridDim.x);
    const int bx = blk % a.ntx, by = (blk / a.ntx) % a.nty, bz = blk / (a.ntx * a.nty);
    const int t = threadIdx.x;
    // first-step cell of this thread and its pull offsets (threads past the
    // tile's rows repeat cells of the last row and store nothing)
    const int rx = t % S::RX, ry = min(t / S::RX, S::RY - 1);
    const bool in_region = t < (a.ty + 2) * S::RX;
    const int x = ((bx * TX - 1 + rx) % nx + nx) % nx;
    const int y = ((by * a.ty - 1 + ry) % ny + ny) % ny;
    const int xs[3] = {x == nx - 1 ? 0 : x + 1, x, x == 0 ? nx - 1 : x - 1};
    const int ys[3] = {(y == ny - 1 ? 0 : y + 1) * nx, y * nx, (y == 0 ? ny - 1 : y - 1) * nx};
    // second-step cell
    const int ox = t & (TX - 1), oy = t / TX;
    const int X = bx * TX + ox, Y = by * a.ty + oy;
    const bool out = oy < a.ty && X < nx && Y < ny;
    const uint32_t ocell = (uint32_t)(X + nx * Y) * 4u;
    float* wr = lds + t;
    const float* rd = lds + (oy + 1) * S::RX + ox + 1;
    int other = kPlane;   // distance to the other plane's buffer
    const int z0 = bz * a.cz, z1 = min(z0 + a.cz, nz);

    float pre[27], gpre[QS], fpre[3];   // first-step cell: pulled, then collided
    auto fetch = [&](int p) {
        const int z = p < 0 ? p + nz : (p >= nz ? p - nz : p);
        // formed again for every plane: kept across the loop they are nine
        // 64-bit lane offsets
        int qx[3] = {xs[0], xs[1], xs[2]}, qy[3] = {ys[0], ys[1], ys[2]};
        asm volatile("" : "+v"(qx[0]), "+v"(qx[1]), "+v"(qx[2]), "+v"(qy[0]), "+v"(qy[1]), "+v"(qy[2]));
        const int64_t zo[3] = {(z == nz - 1 ? 0 : z + 1) * nxy, z * nxy, (z == 0 ? nz - 1 : z - 1) * nxy};
        const float* const fz[3] = {a.f + zo[0], a.f + zo[1], a.f + zo[2]};
        PlaneWalk w(P);
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            pre[tensor_slot(i)] = *w.lane(fz[kCz[i] + 1], (uint32_t)(qx[kCx[i] + 1] + qy[kCy[i] + 1]) * 4u);
            w.next();
        }
        if (kScalar) {
            const float* const gz[3] = {a.g + zo[0], a.g + zo[1], a.g + zo[2]};
            PlaneWalk wg(P);
#pragma unroll
            for (int i = 0; i < QS; ++i) {
                gpre[i] = *wg.lane(gz[kSz[i] + 1], (uint32_t)(qx[kSx[i] + 1] + qy[kSy[i] + 1]) * 4u);
                wg.next();
            }
        }
        if (kForce) {
            PlaneWalk wf(P);
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                fpre[d] = *wf.lane(a.force + zo[1], (uint32_t)(qx[1] + qy[1]) * 4u);
                wf.next();
            }
        }
    };
    // Waits for the fetched plane.  Placed before the stores of a plane, so
    // that the next plane's collision does not wait for those stores as well
    // (loads and stores share one counter).
    auto arrived = [&]() {
#pragma unroll
        for (int q = 0; q < 27; q += 9)
            asm volatile("" : : "v"(pre[q]), "v"(pre[q + 1]), "v"(pre[q + 2]), "v"(pre[q + 3]), "v"(pre[q + 4]),
                         "v"(pre[q + 5]), "v"(pre[q + 6]), "v"(pre[q + 7]), "v"(pre[q + 8]));
        if (kScalar)
            asm volatile("" : : "v"(gpre[0]), "v"(gpre[1]), "v"(gpre[2]), "v"(gpre[3]), "v"(gpre[4]),
                         "v"(gpre[5]), "v"(gpre[6]));
        if (kForce) asm volatile("" : : "v"(fpre[0]), "v"(fpre[1]), "v"(fpre[2]));
    };
    // second-step populations gathered so far.  now: output plane p - 1 (those
    // with c_z = +1 and 0 already read); later: output plane p (c_z = +1)
    float now[27], later[9], gnow[QS], glater = 0.0f;
#pragma unroll
    for (int q = 0; q < 27; ++q) now[q] = 0.0f;
#pragma unroll
    for (int q = 0; q < 9; ++q) later[q] = 0.0f;
#pragma unroll
    for (int q = 0; q < QS; ++q) gnow[q] = 0.0f;

    fetch(z0 - 1);
    arrived();
    for (int p = z0 - 1; p <= z1; ++p) {
        // first step on plane p
        float F1[3] = {0.0f, 0.0f, 0.0f};
        if (kForce)
#pragma unroll
            for (int d = 0; d < 3; ++d) F1[d] = fpre[d];
        PulledCell c1 = pulled_transform<kScalar>(a, pre, gpre, F1);
        pin(pre, c1.m);
        // the second half and the stores to LDS in one block: with the whole
        // update before them, 74 -> 88 us per step at 128^3 with scalar
        if (!kTwo) __syncthreads();   // the previous plane has been read
        if (in_region) {
            pulled_relax<kScalar>(a, c1, pre, gpre);
#pragma unroll
            for (int i = 0; i < Q; ++i) wr[i * R] = pre[tensor_slot(i)];
            if (kScalar)
#pragma unroll
                for (int i = 0; i < QS; ++i) wr[(Q + i) * R] = gpre[i];
        }
        // without a branch: a conditional fetch keeps both versions of the
        // registers (past the last plane it reloads that plane)
        fetch(min(p + 1, z1));
        __syncthreads();
        // second step on output plane p - 1
        const bool store = out && p > z0;
        if (store) {
#pragma unroll
            for (int i = 0; i < Q; ++i)
                if (kCz[i] == -1) now[tensor_slot(i)] = rd[i * R - kCx[i] - kCy[i] * S::RX];
            if (kScalar) gnow[6] = rd[(Q + 6) * R];
            float F2[3] = {0.0f, 0.0f, 0.0f};
            if (kForce) {
                PlaneWalk w(P);
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    F2[d] = *w.lane(a.force + (p - 1) * nxy, ocell);
                    w.next();
                }
            }
            const PulledCell c2 = pulled_transform<kScalar>(a, now, gnow, F2);
            pulled_relax<kScalar>(a, c2, now, gnow);
        }
        arrived();
        if (store) {
            uint32_t oc = ocell;
            asm volatile("" : "+v"(oc));
            PlaneWalk w(P);
#pragma unroll
            for (int i = 0; i < Q; ++i) {
                __builtin_nontemporal_store(now[tensor_slot(i)], w.lane(a.fo + (p - 1) * nxy, oc));
                w.next();
            }
            if (kScalar) {
                PlaneWalk wg(P);
#pragma unroll
                for (int i = 0; i < QS; ++i) {
                    __builtin_nontemporal_store(gnow[i], wg.lane(a.go + (p - 1) * nxy, oc));
                    wg.next();
                }
            }
        }
        if (out) {
            int k = 0;
#pragma unroll
            for (int i = 0; i < Q; ++i)
                if (kCz[i] == 0) now[tensor_slot(i)] = rd[i * R - kCx[i] - kCy[i] * S::RX];
#pragma unroll
            for (int i = 0; i < Q; ++i)
                if (kCz[i] == 1) {
                    now[tensor_slot(i)] = later[k];
                    later[k++] = rd[i * R - kCx[i] - kCy[i] * S::RX];
                }
            if (kScalar) {
#pragma unroll
                for (int i = 0; i < 5; ++i) gnow[i] = rd[(Q + i) * R - kSx[i] - kSy[i] * S::RX];
                gnow[5] = glater;
                glater = rd[(Q + 5) * R];
            }
        }
        if (kTwo) {
            wr += other;
            rd += other;
            other = -other;
        }
    }
}

// Rows per tile and planes per workgroup.  One workgroup runs on a CU at a
// time; the workgroups run in rounds of 256, each computes two planes more
// than it outputs, and a plane takes its first- and second-step waves per SIMD
// and half a wave for the barrier.  Measured at 256^3: 64 x 8 tiles of 128
// planes (256 workgroups) 419 us per step, of 64 planes 456, of 32 planes 463;
// 64 x 9 of 128 planes (232) 512; tiles of 13 rows and one LDS plane 472 (64 us
// against 57 at 128^3, 61 against 61 at 181x118x77).
template <int TX, int TY>
static void plan_tiles(PairArgs& a)
{
    constexpr int64_t slots = 256;
    a.ntx = (a.nx + TX - 1) / TX;
    double best = 1e300;
    const int nt0 = (a.ny + TY - 1) / TY;
    for (int nty = nt0; nty <= 2 * nt0 && nty <= nt0 + 16 && nty <= a.ny; ++nty) {
        const int ty = (a.ny + nty - 1) / nty;
        const int64_t tiles = (int64_t)a.ntx * ((a.ny + ty - 1) / ty);
        const int w1 = ((ty + 2) * (TX + 2) + 63) / 64, w2 = (ty * TX + 63) / 64;
        const double waves = (w1 + 3) / 4 + (w2 + 3) / 4 + 0.5;
        const int64_t r0 = (tiles + slots - 1) / slots;
        for (int64_t r = r0; r < r0 + 4; ++r) {
            const int64_t chunks = std::min<int64_t>(a.nz, r * slots / tiles);
            const int cz = (int)((a.nz + chunks - 1) / chunks);
            const int64_t blocks = tiles * ((a.nz + cz - 1) / cz);
            const double cost = (double)((blocks + slots - 1) / slots) * (cz + 2.5) * waves;
            if (cost < best) {
                best = cost;
                a.nty = (a.ny + ty - 1) / ty;
                a.ty = ty;
                a.cz = cz;
            }
        }
    }
}

template <bool kForce, bool kScalar, int TX, int TY, int kWaves>
static void launch_pair(PairArgs a, hipStream_t st)
{
    plan_tiles<TX, TY>(a);
    const int64_t blocks = (int64_t)a.ntx * a.nty * ((a.nz + a.cz - 1) / a.cz);
    const int threads = (std::max((a.ty + 2) * (TX + 2), a.ty * TX) + 63) / 64 * 64;
    hipLaunchKernelGGL((k_step_pair<kForce, kScalar, TX, TY, kWaves>), dim3((unsigned)blocks),
                       dim3((unsigned)threads), 0, st, a);
}

// The same pair for levels too small to march: one TX x TY x TZ tile per
// workgroup, the first step on it and one cell around it (a thread per cell)
// into LDS, one barrier, the second step from there.  What bounds a small
// step is its launch and the round trip to memory (4.3-4.7 us at 16^3 and at
// 32^3 alike); two and a half times the first step's arithmetic costs less
// than a second trip.  Per step, pair against k_step: 3.8 / 4.7 us at 32^3,
// 6.6 / 8.4 us at 48^3, 10.9 / 12.2 us at 64^3, 16.5 / 21.9 us at 72^3; with
// scalar and force 4.3 / 4.9 us at 32^3, 21.3 / 27.4 us at 72^3.  Larger tiles
// share more but leave SIMDs idle or hold one workgroup per CU: 8x8x8 at 32^3
// 4.9 us, 8x8x4 4.1, 16x6x4 4.6; 4x4x4 at 64^3 17.5.
template <int TX, int TY, int TZ>
struct BoxShape {
    static constexpr int RX = TX + 2, RY = TY + 2, RZ = TZ + 2;
    static constexpr int kRegion = RX * RY * RZ;   // first-step cells
    static constexpr int kThreads = (kRegion + 63) / 64 * 64;
    static constexpr int kCells = TX * TY * TZ;
};

template <bool kForce, bool kScalar, int TX, int TY, int TZ>
__global__ void __launch_bounds__((BoxShape<TX, TY, TZ>::kThreads)) k_step_pair_box(const PairArgs a)
{
    using S = BoxShape<TX, TY, TZ>;
    constexpr int R = S::kRegion;
    __shared__ float lds[(kScalar ? Q + QS : Q) * R];

    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const int nxy = nx * ny;
    const int blk = xcd_block(blockIdx.x, gridDim.x);
    const int bx = blk % a.ntx, by = (blk / a.ntx) % a.nty, bz = blk / (a.ntx * a.nty);
    const int t = threadIdx.x;
    // first-step cell; the box is at least a tile long each way, so one period
    // brings any of them inside
    const int rx = t % S::RX, ry = t / S::RX % S::RY, rz = min(t / (S::RX * S::RY), S::RZ - 1);
    auto wrap = [](int v, int n) { return v < 0 ? v + n : (v >= n ? v - n : v); };
    const int x = wrap(bx * TX - 1 + rx, nx), y = wrap(by * TY - 1 + ry, ny), z = wrap(bz * TZ - 1 + rz, nz);
    const int xs[3] = {x == nx - 1 ? 0 : x + 1, x, x == 0 ? nx - 1 : x - 1};
    const int ys[3] = {(y == ny - 1 ? 0 : y + 1) * nx, y * nx, (y == 0 ? ny - 1 : y - 1) * nx};
    const int zs[3] = {(z == nz - 1 ? 0 : z + 1) * nxy, z * nxy, (z == 0 ? nz - 1 : z - 1) * nxy};
    // second-step cell
    const int ox = t % TX, oy = t / TX % TY, oz = t / (TX * TY);
    const int X = bx * TX + ox, Y = by * TY + oy, Z = bz * TZ + oz;
    const bool out = t < S::kCells && X < nx && Y < ny && Z < nz;
    const uint32_t ocell = (uint32_t)(X + nx * Y + nxy * Z) * 4u;

    float v[27], g[QS], F1[3] = {0.0f, 0.0f, 0.0f}, F2[3] = {0.0f, 0.0f, 0.0f};
    PlaneWalk w(a.plane);
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        v[tensor_slot(i)] = *w.lane(a.f, (uint32_t)(xs[kCx[i] + 1] + ys[kCy[i] + 1] + zs[kCz[i] + 1]) * 4u);
        w.next();
    }
    if (kScalar) {
        PlaneWalk wg(a.plane);
#pragma unroll
        for (int i = 0; i < QS; ++i) {
            g[i] = *wg.lane(a.g, (uint32_t)(xs[kSx[i] + 1] + ys[kSy[i] + 1] + zs[kSz[i] + 1]) * 4u);
            wg.next();
        }
    }
    if (kForce) {
        PlaneWalk wf(a.plane);
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            F1[d] = *wf.lane(a.force, (uint32_t)(xs[1] + ys[1] + zs[1]) * 4u);
            if (out) F2[d] = *wf.lane(a.force, ocell);
            wf.next();
        }
    }
    PulledCell c1 = pulled_transform<kScalar>(a, v, g, F1);
    pin(v, c1.m);
    if (t < R) {
        pulled_relax<kScalar>(a, c1, v, g);
#pragma unroll
        for (int i = 0; i < Q; ++i) lds[i * R + t] = v[tensor_slot(i)];
        if (kScalar)
#pragma unroll
            for (int i = 0; i < QS; ++i) lds[(Q + i) * R + t] = g[i];
    }
    __syncthreads();
    if (!out) return;
    const float* rd = lds + ((oz + 1) * S::RY + oy + 1) * S::RX + ox + 1;
#pragma unroll
    for (int i = 0; i < Q; ++i)
        v[tensor_slot(i)] = rd[i * R - kCx[i] - kCy[i] * S::RX - kCz[i] * S::RX * S::RY];
    if (kScalar)
#pragma unroll
        for (int i = 0; i < QS; ++i)
            g[i] = rd[(Q + i) * R - kSx[i] - kSy[i] * S::RX - kSz[i] * S::RX * S::RY];
    const PulledCell c2 = pulled_transform<kScalar>(a, v, g, F2);
    pulled_relax<kScalar>(a, c2, v, g);
    PlaneWalk wo(a.plane);
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        *wo.lane(a.fo, ocell) = v[tensor_slot(i)];
        wo.next();
    }
    if (kScalar) {
        PlaneWalk wg(a.plane);
#pragma unroll
        for (int i = 0; i < QS; ++i) {
            *wg.lane(a.go, ocell) = g[i];
            wg.next();
        }
    }
}

template <bool kForce, bool kScalar, int TX, int TY, int TZ>
static void launch_box(PairArgs a, hipStream_t st)
{
    a.ntx = (a.nx + TX - 1) / TX;
    a.nty = (a.ny + TY - 1) / TY;
    const int blocks = a.ntx * a.nty * ((a.nz + TZ - 1) / TZ);
    hipLaunchKernelGGL((k_step_pair_box<kForce, kScalar, TX, TY, TZ>), dim3((unsigned)blocks),
                       dim3((unsigned)BoxShape<TX, TY, TZ>::kThreads), 0, st, a);
}

template <bool kForce, bool kScalar>
static void launch_box(const PairArgs& a, int tile, hipStream_t st)
{
    if (tile == 0)
        launch_box<kForce, kScalar, 8, 4, 4>(a, st);
    else if (tile == 1)
        launch_box<kForce, kScalar, 8, 6, 4>(a, st);
    else if constexpr (!kScalar)
        launch_box<kForce, kScalar, 16, 4, 4>(a, st);
}

static PairArgs pair_args(const cslbm_level* L, const void* fin, void* fout, const float* gin, float* gout)
{
    PairArgs a;
    a.f = static_cast<const float*>(fin);
    a.fo = static_cast<float*>(fout);
    a.g = gin;
    a.go = gout;
    a.force = L->force;
    a.nx = L->nx;
    a.ny = L->ny;
    a.nz = L->nz;
    a.ntx = a.nty = a.ty = a.cz = 1;
    a.plane = L->plane;
    a.r = make_rates(L->p);
    if (!a.r.adaptive) {   // the factor 0 * min(G / g_max, 1) + 1 is 1
        a.r.a = 0.0f;
        a.r.b = 1.0f;
    }
    a.beta = (float)L->p.beta;
    a.s_ref = (float)L->p.s_ref;
    a.inv_tau_s = gin ? (float)(1.0 / L->p.tau_s) : 0.0f;
    return a;
}

// Tiles 64 cells wide, or 32 where the rows are multiples of half a cache
// line and 64 would leave more lanes past the row's end (96^3: 28 against 31
// us per step, 80x300x100 with scalar 109, 117).  With other row lengths a
// 32-wide tile writes every line in parts (181x118x77: 72 against 60 us).
static bool narrow_tiles(const cslbm_level* L)
{
    const int w32 = (L->nx + 31) / 32 * 32, w64 = (L->nx + 63) / 64 * 64;
    return L->nx <= 32 || (L->nx % 16 == 0 && w32 < w64);
}

// Whether a pair marches along z: enough cells to give every CU a tile of
// some planes (cells times the used part of the tiles' width; per step at
// 64^3 12.3 us against 12.0 single, 64x64x128 17 against 22) and a few rows
// and planes for the halo to stay small (288x288x8: 26 against 31).  Lane
// offsets in a plane are 32-bit bytes.
// Up to 2^19 cells the small tiles are the better way for fewer than 30 rows
// or planes (with force 96x28x141 19.7 us marching, 16.5 on tiles, 18.1 single;
// 64x23x191 14.8, 13.7, 14.2).
constexpr int64_t kBoxCells = 1 << 19;

static bool marches(const cslbm_level* L)
{
    const int least = std::min(L->ny, L->nz);
    if (least < 8 || (int64_t)L->nx * L->ny >= (1 << 30)) return false;
    if (cells_of(L) <= kBoxCells && least < 30) return false;
    const int tx = narrow_tiles(L) ? 32 : 64;
    const double used = (double)L->nx / ((L->nx + tx - 1) / tx * tx);
    return (double)cells_of(L) * used > (double)(1 << 18);
}

// The tile of k_step_pair_box for a level, -1 where two single steps are
// faster or as fast.  Both sides are estimated in us from fits to the times of
// 900 random boxes of 1k-520k cells (they leave 6-9 %): a pair costs a launch
// and its tiles' first- and second-step waves, counted on average and on the
// CU that has most; a step a launch, its 256-thread blocks, its cells, and
// those that outgrow the L2s.  Which side wins changes with how the tiles fill
// the last round over 256 CUs (with scalar and force 66x62x19: 8.1 us per step
// against 7.8 single; 45x23x77: 7.0 against 8.2), so a limit on the cells alone
// would not do.  A pair has to be ahead by 11 %: 4 of the 525 boxes that pair
// lose more than 2 % (10 % at worst), 17 of 622 would at 5 %.
static int box_tile(const cslbm_level* L)
{
    constexpr int tx[3] = {8, 8, 16}, ty[3] = {4, 6, 4}, tz = 4;
    // launch, wave of the CU with most tiles, wave on average
    constexpr double pair_us[2][3][3] = {{{5.2, 0.22, 0.14}, {5.15, 0.21, 0.12}, {5.2, 0.167, 0.14}},
                                         {{5.0, 0.33, 0.14}, {5.4, 0.24, 0.177}, {}}};
    const int64_t cells = cells_of(L);
    const bool scalar = L->g != nullptr;
    if (cells > kBoxCells) return -1;
    const dim3 b = step_block(L->nx);
    const double rounds = (double)((L->nx + b.x - 1) / b.x) * ((L->ny + b.y - 1) / b.y) * L->nz / 256.0;
    const double spill = std::max((double)cells - 1.2e5, 0.0);
    const double single = scalar ? 4.25 + 0.85 * rounds + 2.25e-5 * (double)cells + 2.45e-5 * spill
                                 : 4.2 + 0.66 * rounds + 1.95e-5 * (double)cells + 1.5e-5 * spill;
    int tile = -1;
    double best = 0.89 * 2.0 * single;
    for (int k = 0; k < (scalar ? 2 : 3); ++k) {
        // one period brings a halo cell inside
        if (L->nx < tx[k] || L->ny < ty[k] || L->nz < tz) continue;
        const int64_t blocks = (int64_t)((L->nx + tx[k] - 1) / tx[k]) * ((L->ny + ty[k] - 1) / ty[k]) *
                               ((L->nz + tz - 1) / tz);
        const int waves = ((tx[k] + 2) * (ty[k] + 2) * (tz + 2) + 63) / 64 + (tx[k] * ty[k] * tz + 63) / 64;
        const double(&c)[3] = pair_us[scalar][k];
        const double most = c[1] + (L->force ? 0.03 : 0.0);
        const double us = c[0] + waves * (most * (double)((blocks + 255) / 256) + c[2] * (double)blocks / 256.0);
        if (us < best) {
            best = us;
            tile = k;
        }
    }
    return tile;
}

// Levels whose pairs of steps run faster fused: fully periodic FP32 boxes
// without flags or gradient mode.
PairKind step_pair_kind(const cslbm_level* L)
{
    if (L->storage != CSLBM_F32 || L->flags || L->brick_table || (L->periodic & 7) != 7 ||
        L->p.grad_mode != 0)
        return PairKind::kNone;
    if (marches(L)) return PairKind::kMarch;
    return box_tile(L) >= 0 ? PairKind::kTiles : PairKind::kNone;
}

int launch_step_pair(const cslbm_level* L, const void* fin, void* fout, const float* gin, float* gout,
                     hipStream_t stream)
{
    const PairArgs a = pair_args(L, fin, fout, gin, gout);
    if (!marches(L)) {
        const int tile = box_tile(L);
        if (gin && L->force)
            launch_box<true, true>(a, tile, stream);
        else if (gin)
            launch_box<false, true>(a, tile, stream);
        else if (L->force)
            launch_box<true, false>(a, tile, stream);
        else
            launch_box<false, false>(a, tile, stream);
        return check_launch("k_step_pair_box");
    }
    const bool narrow = narrow_tiles(L);
    // at most twelve waves (32 x 16: ten), three per SIMD (the scalar takes 154-167 VGPRs)
    if (gin && L->force) {
        if (narrow)
            launch_pair<true, true, 32, 16, 3>(a, stream);
        else
            launch_pair<true, true, 64, 9, 3>(a, stream);
    } else if (gin) {
        if (narrow)
            launch_pair<false, true, 32, 16, 3>(a, stream);
        else
            launch_pair<false, true, 64, 9, 3>(a, stream);
    } else if (L->force) {
        if (narrow)
            launch_pair<true, false, 32, 20, 3>(a, stream);
        else
            launch_pair<true, false, 64, 9, 3>(a, stream);
    } else {
        if (narrow)
            launch_pair<false, false, 32, 20, 3>(a, stream);
        else
            launch_pair<false, false, 64, 9, 3>(a, stream);
    }
    return check_launch("k_step_pair");
}

}  // namespace cslbm
