// gfx950 small-board kernel of libfdtd.
//
// brick_step2 advances a brick of 28 x (RY-4) x (RZ-4) nodes by two full leapfrog
// steps (Model section: B->H then D->E, Eqs. 1-4, twice) from one read of its
// 32 x RY x RZ neighbourhood, with no march along z:
//
//   E^n         on the whole region, i0-2 .. i0+29 (likewise in y and z)
//   H^{n+1/2}   on region indices 0 .. R-2 of each axis
//   E^{n+1}     on 1 .. R-2
//   H^{n+3/2}   on 1 .. R-3
//   E^{n+2}     on 2 .. R-3, the owned nodes, stored with H, D and B
//
// A half wave is one row of 32 nodes.  Every thread keeps its nodes' fields in
// registers through all four half steps; LDS holds E and H for the neighbours.
//
// Why: a board of some 10^4 to 10^5 cells is bound by latency, not by work.  The
// marching kernel (field_step2) walks such a board's few tiles in short z pieces,
// three barriers and a round of prefetched loads per plane behind a chain of five
// dependent loads (work item, descriptor, step counters, tables, fields):
// 14.7 us per pair of steps for 48 x 43 x 30 cells (9.5 in bricks) where a chain of empty
// launches takes 1.7 each.  Here a brick's loads are all in flight at once, addressed from
// kernel arguments alone, and a pair of steps is four barriers.  The price is the
// halo: 19 % (8 x 7) to 33 % (16 x 8) of the nodes computed are owned, which is why
// larger boards, whose compute units are busy anyway, keep the marching kernel, and
// so do boards that step beside others whose launches could share the device.
//
// Every per-node update is written with exactly the expressions of the other
// field kernels, so all give the same bits.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>

#include "fdtd_device.h"
#include "fdtd_internal.h"

namespace fdtd {

namespace {

// the five coefficients of one axis that a half step reads at one index: of H
// (half node a, own axis at the node) or of E (node a, own axis at the half node)
struct Half {
    float cam1, rp, ca, ph, q;
};

struct Yes { static constexpr bool value = true; };
struct No { static constexpr bool value = false; };

template <int RY, int RZ>
struct BrickLds {
    static constexpr int kNodes = 32 * RY * RZ;
    float e[3][kNodes], h[3][kNodes];
    ClassEntry tab[256];
    // [row][0 the H set, 1 the E set]: cam1, rp, ca, ph, q
    alignas(16) float y[RY][2][8], z[RZ][2][8];
};

template <int RY, int RZ, typename CT, bool PL>
__global__ __launch_bounds__(1024)
__attribute__((amdgpu_waves_per_eu(4))) void brick_step2(const BoardDev B, int par, int rel)
{
    constexpr int OX = 28, OY = RY - 4, OZ = RZ - 4, ROWS = RY * RZ, N = (ROWS + 31) / 32;
    constexpr int DY = 32, DZ = 32 * RY;   // LDS strides
    __shared__ BrickLds<RY, RZ> L;
    const int nx = B.nx, ny = B.ny, nz = B.nz;
    const int tid = threadIdx.x;
    const int x = tid & 31;
    int row0 = tid >> 5;   // made opaque before each half step, so that row indices are not kept in registers
    const int i0 = (int)blockIdx.x * OX, j0 = (int)blockIdx.y * OY, k0 = (int)blockIdx.z * OZ;
    const int i = i0 - 2 + x;
    const int sy = B.pitch, sz = B.pitch * (ny + 1), guard = sz * (nz + 1);
    const float* gE = B.f[par][0];
    const float* gH = B.f[par][3];
    const float* gB = B.f[par][6];
    const float* gD = B.d[par][0];
    const uint32_t cs = B.cstride, cs2 = 2u * B.cstride, guardb = (uint32_t)guard * 4u;
    const int64_t step = *(const int64_t*)B.step + rel;   // read by source and probe nodes only
    const float crdx = B.crd_x, crdy = B.crd_y, crdz = B.crd_z;
    auto in_slab = [](int q, int n, int lo, int hi) { return (q < lo) || (hi > 0 && q >= n - hi); };
    const bool px = in_slab(i, nx, B.pml[0], B.pml[1]);
    const bool ibx = (unsigned)i <= (unsigned)nx;

    // ---- the whole neighbourhood in flight: fields, auxiliaries, class
    float ex[N], ey[N], ez[N], hx[N], hy[N], hz[N], bx[N], by[N], bz[N], dx[N], dy[N], dz[N];
    CT id[N];
    auto in_py = [&](int y) { return in_slab(j0 - 2 + y, ny, B.pml[2], B.pml[3]); };
    auto in_pz = [&](int z) { return in_slab(k0 - 2 + z, nz, B.pml[4], B.pml[5]); };
    auto in_board = [&](int y, int z) {
        return ibx && (unsigned)(j0 - 2 + y) <= (unsigned)ny && (unsigned)(k0 - 2 + z) <= (unsigned)nz;
    };
#pragma unroll
    for (int n = 0; n < N; ++n) {
        const int row = row0 + 32 * n, y = row % RY, z = row / RY;
        const int j = j0 - 2 + y, k = k0 - 2 + z;
        const bool py = in_py(y), pz = in_pz(z);
        const uint32_t off = row < ROWS && in_board(y, z) ? (uint32_t)(i + j * sy + k * sz) * 4u : guardb;
        ex[n] = ld_at(gE, off);
        ey[n] = ld_at(gE, off + cs);
        ez[n] = ld_at(gE, off + cs2);
        // H, B and the class where H1 runs, D where E1 runs
        const bool inh = x < 31 && y < RY - 1 && z < RZ - 1, ine = inh && x >= 1 && y >= 1 && z >= 1;
        const uint32_t oh = inh ? off : guardb, oe = ine ? off : guardb;
        hx[n] = ld_at(gH, oh);
        hy[n] = ld_at(gH, oh + cs);
        hz[n] = ld_at(gH, oh + cs2);
        bx[n] = ld_at(gB, (px || py) ? oh : guardb);
        by[n] = ld_at(gB, ((py || pz) ? oh : guardb) + cs);
        bz[n] = ld_at(gB, ((pz || px) ? oh : guardb) + cs2);
        dx[n] = ld_at(gD, (px || py) ? oe : guardb);
        dy[n] = ld_at(gD, ((py || pz) ? oe : guardb) + cs);
        dz[n] = ld_at(gD, ((pz || px) ? oe : guardb) + cs2);
        id[n] = ld_at_t<CT>(B.cls, sizeof(CT) == 1 ? oe >> 2 : oe >> 1);
    }
    const __attribute__((address_space(1))) ClassEntry* __restrict__ ctab =
        (const __attribute__((address_space(1))) ClassEntry*)B.ctab;
    if (sizeof(CT) == 1 && tid < 4 * B.nclass)   // the table word by word
        ((float*)L.tab)[tid] = ((cgfloat*)B.ctab)[tid];
    // coefficient kinds in the order of Half; the H set takes a's half node and the
    // own axis's node, the E set the other way round
    auto coef = [&](int axis, int n1, int idx, int set, int v) {
        const int kind = v == 0 ? kCam1 : v == 1 ? kRp : v == 2 ? kCa : v == 3 ? kPh : kQ;
        const int half = v <= 2 ? 1 - set : set;
        return ((cgfloat*)B.coef[axis])[(kind * 2 + half) * n1 + min(max(idx, 0), n1 - 1)];
    };
    for (int e = tid; e < (RY + RZ) * 10; e += 1024) {
        const int r = e / 10, set = e % 10 / 5, v = e % 5;
        if (r < RY)
            L.y[r][set][v] = coef(1, ny + 1, j0 - 2 + r, set, v);
        else
            L.z[r - RY][set][v] = coef(2, nz + 1, k0 - 2 + r - RY, set, v);
    }
    Half X[2];
#pragma unroll
    for (int set = 0; set < 2; ++set)
        X[set] = Half{coef(0, nx + 1, i, set, 0), coef(0, nx + 1, i, set, 1), coef(0, nx + 1, i, set, 2),
                      coef(0, nx + 1, i, set, 3), coef(0, nx + 1, i, set, 4)};
    auto half_of = [](const float* p) { return Half{p[0], p[1], p[2], p[3], p[4]}; };
    auto class_entry = [&](CT c) {
        ClassEntry ce;
        if (sizeof(CT) == 1) {
            ce = L.tab[c];
        } else {
            ce.inv_x = ctab[c].inv_x;
            ce.inv_y = ctab[c].inv_y;
            ce.inv_z = ctab[c].inv_z;
            ce.flags = ctab[c].flags;
        }
        return ce;
    };

    // ---- B then H from E in LDS, region indices lo .. R-1-hi of each axis
    auto h_half = [&](int lo, int hi) __attribute__((always_inline)) {
        asm volatile("" : "+v"(row0));
#pragma unroll
        for (int n = 0; n < N; ++n) {
            const int row = row0 + 32 * n, y = row % RY, z = row / RY, q = row * 32 + x;
            const bool in = y >= lo && y <= RY - 1 - hi && z >= lo && z <= RZ - 1 - hi && row < ROWS;
            if (!in) continue;   // the whole half wave
            const bool inx = x >= lo && x <= 31 - hi;
            float nhx = 0.f, nhy = 0.f, nhz = 0.f, nbx = 0.f, nby = 0.f, nbz = 0.f;
            if (inx && in_board(y, z)) {
                const bool py = in_py(y), pz = in_pz(z);
                const Half Y = half_of(L.y[y][0]), Z = half_of(L.z[z][0]);
                const float cxe = (L.e[2][q + DY] - ez[n]) * crdy - (L.e[1][q + DZ] - ey[n]) * crdz;
                const float dbx = fmaf(Y.cam1, bx[n], -Y.rp * cxe);
                nhx = fmaf(Z.ca, hx[n], Z.rp * fmaf(X[0].ph, dbx, X[0].q * bx[n]));
                const float cye = (L.e[0][q + DZ] - ex[n]) * crdz - (L.e[2][q + 1] - ez[n]) * crdx;
                const float dby = fmaf(Z.cam1, by[n], -Z.rp * cye);
                nhy = fmaf(X[0].ca, hy[n], X[0].rp * fmaf(Y.ph, dby, Y.q * by[n]));
                const float cze = (L.e[1][q + 1] - ey[n]) * crdx - (L.e[0][q + DY] - ex[n]) * crdy;
                const float dbz = fmaf(X[0].cam1, bz[n], -X[0].rp * cze);
                nhz = fmaf(Y.ca, hz[n], Y.rp * fmaf(Z.ph, dbz, Z.q * bz[n]));
                nbx = (px || py) ? bx[n] + dbx : 0.f;
                nby = (py || pz) ? by[n] + dby : 0.f;
                nbz = (pz || px) ? bz[n] + dbz : 0.f;
            }
            hx[n] = nhx;
            hy[n] = nhy;
            hz[n] = nhz;
            bx[n] = nbx;
            by[n] = nby;
            bz[n] = nbz;
            L.h[0][q] = nhx;
            L.h[1][q] = nhy;
            L.h[2][q] = nhz;
        }
    };
    // ---- D then E from H in LDS, region indices lo .. R-1-hi, at step s
    auto e_half = [&](int lo, int hi, int64_t s, auto last) __attribute__((always_inline)) {
        constexpr bool LAST = decltype(last)::value;
        bool bad = false;
        asm volatile("" : "+v"(row0));
#pragma unroll
        for (int n = 0; n < N; ++n) {
            const int row = row0 + 32 * n, y = row % RY, z = row / RY, q = row * 32 + x;
            const int j = j0 - 2 + y, k = k0 - 2 + z;
            const bool in = y >= lo && y <= RY - 1 - hi && z >= lo && z <= RZ - 1 - hi && row < ROWS;
            if (!in) continue;
            const bool inx = x >= lo && x <= 31 - hi;
            // the nodes this brick owns: the far walls carry nothing
            const bool own = x >= 2 && x <= 29 && y >= 2 && y <= RY - 3 && z >= 2 && z <= RZ - 3 && i < nx &&
                             j < ny && k < nz;
            float nex = 0.f, ney = 0.f, nez = 0.f, ndx = 0.f, ndy = 0.f, ndz = 0.f;
            if (inx && in_board(y, z) && (!LAST || own)) {
                const bool py = in_py(y), pz = in_pz(z);
                const uint32_t o = (uint32_t)(i + j * sy + k * sz) * 4u;
                const Half Y = half_of(L.y[y][1]), Z = half_of(L.z[z][1]);
                const ClassEntry ce = class_entry(id[n]);
                const float chx = (hz[n] - L.h[2][q - DY]) * crdy - (hy[n] - L.h[1][q - DZ]) * crdz;
                const float ddx = fmaf(Y.cam1, dx[n], Y.rp * chx);
                const float exn = fmaf(Z.ca, ex[n], Z.rp * (ce.inv_x * fmaf(X[1].ph, ddx, X[1].q * dx[n])));
                const float chy = (hx[n] - L.h[0][q - DZ]) * crdz - (hz[n] - L.h[2][q - 1]) * crdx;
                const float ddy = fmaf(Z.cam1, dy[n], Z.rp * chy);
                const float eyn = fmaf(X[1].ca, ey[n], X[1].rp * (ce.inv_y * fmaf(Y.ph, ddy, Y.q * dy[n])));
                const float chz = (hy[n] - L.h[1][q - 1]) * crdx - (hx[n] - L.h[0][q - DY]) * crdy;
                float ddz = fmaf(X[1].cam1, dz[n], X[1].rp * chz);
                float ezn = fmaf(Y.ca, ez[n], Y.rp * (ce.inv_z * fmaf(Z.ph, ddz, Z.q * dz[n])));
                const int node = (int)(o >> 2);
                if (ce.flags & kSrcEz) {
                    // the sources' Js of step s; a resistive source solves for E^{n+1}
                    const __attribute__((address_space(1))) int32_t* sn =
                        (const __attribute__((address_space(1))) int32_t*)B.src_node;
                    float js = 0.0f, bs = 0.0f;
                    for (int t = 0; t < B.nsrc; ++t)
                        if (sn[t] == node) {
                            js += ((cgfloat*)B.src_j)[t * B.max_steps + s];
                            bs += ((cgfloat*)B.src_beta)[t];
                        }
                    const float chs = chz - js;
                    ddz = fmaf(X[1].cam1, dz[n], X[1].rp * chs);
                    ezn = fmaf(Y.ca, ez[n], Y.rp * (ce.inv_z * fmaf(Z.ph, ddz, Z.q * dz[n])));
                    if (bs != 0.0f) ezn = conductive_e(ez[n], chs, ce.inv_z, bs);
                }
                nex = (ce.flags & kUpdEx) ? exn : 0.0f;
                ney = (ce.flags & kUpdEy) ? eyn : 0.0f;
                nez = (ce.flags & kUpdEz) ? ezn : 0.0f;
                ndx = ((px || py) && (ce.flags & kUpdEx)) ? dx[n] + ddx : dx[n];
                ndy = ((py || pz) && (ce.flags & kUpdEy)) ? dy[n] + ddy : dy[n];
                ndz = ((pz || px) && (ce.flags & kUpdEz)) ? dz[n] + ddz : dz[n];
                if (own && (ce.flags & kPrbEz)) {
                    const __attribute__((address_space(1))) int32_t* pn =
                        (const __attribute__((address_space(1))) int32_t*)B.prb_node;
                    for (int t = 0; t < B.nprb; ++t)
                        if (pn[t] == node) ((gfloat*)B.prb_series)[t * B.max_steps + s] = nez;
                }
                if (PL && own && (ce.flags & kPlnEz))   // ring slot s mod kPlaneRing, one node plane each
                    st_at(B.plane_ring, (uint32_t)(s & (kPlaneRing - 1)) * ((uint32_t)sz * 4u) + (uint32_t)(i + j * sy) * 4u, nez);
                if constexpr (LAST) {
                    float* dE = B.f[par ^ 1][0];
                    float* dH = B.f[par ^ 1][3];
                    float* dB = B.f[par ^ 1][6];
                    float* dD = B.d[par ^ 1][0];
                    st_at(dE, o, nex);
                    st_at(dE, o + cs, ney);
                    st_at(dE, o + cs2, nez);
                    st_at(dH, o, hx[n]);
                    st_at(dH, o + cs, hy[n]);
                    st_at(dH, o + cs2, hz[n]);
                    if (px || py) {
                        st_at(dB, o, bx[n]);
                        st_at(dD, o, ndx);
                    }
                    if (py || pz) {
                        st_at(dB, o + cs, by[n]);
                        st_at(dD, o + cs, ndy);
                    }
                    if (pz || px) {
                        st_at(dB, o + cs2, bz[n]);
                        st_at(dD, o + cs2, ndz);
                    }
                    bad |= !isfinite(nex + ney + nez);
                }
            }
            if constexpr (!LAST) {
                ex[n] = nex;
                ey[n] = ney;
                ez[n] = nez;
                dx[n] = ndx;
                dy[n] = ndy;
                dz[n] = ndz;
                L.e[0][q] = nex;
                L.e[1][q] = ney;
                L.e[2][q] = nez;
            }
        }
        if (LAST && bad) *(__attribute__((address_space(1))) int32_t*)B.bad = 1;
    };
#pragma unroll
    for (int n = 0; n < N; ++n) {
        const int row = row0 + 32 * n;
        if (row < ROWS) {
            L.e[0][row * 32 + x] = ex[n];
            L.e[1][row * 32 + x] = ey[n];
            L.e[2][row * 32 + x] = ez[n];
        }
    }
    __syncthreads();
    h_half(0, 1);
    __syncthreads();
    e_half(1, 1, step, No{});
    __syncthreads();
    h_half(1, 2);
    __syncthreads();
    e_half(2, 2, step + 1, Yes{});
}

template <int RY, int RZ>
hipError_t launch_t(const BoardDev& b, int par, int rel, bool wide, bool plane, hipStream_t st)
{
    const dim3 grid((b.nx + 27) / 28, (b.ny + RY - 5) / (RY - 4), (b.nz + RZ - 5) / (RZ - 4));
    if (wide) {
        if (plane)
            hipLaunchKernelGGL((brick_step2<RY, RZ, uint16_t, true>), grid, dim3(1024), 0, st, b, par, rel);
        else
            hipLaunchKernelGGL((brick_step2<RY, RZ, uint16_t, false>), grid, dim3(1024), 0, st, b, par, rel);
    } else {
        if (plane)
            hipLaunchKernelGGL((brick_step2<RY, RZ, uint8_t, true>), grid, dim3(1024), 0, st, b, par, rel);
        else
            hipLaunchKernelGGL((brick_step2<RY, RZ, uint8_t, false>), grid, dim3(1024), 0, st, b, par, rel);
    }
    return hipGetLastError();
}

}  // namespace

// Brick shapes (region rows in y and z) and what a pair of steps takes, launch
// included, while every brick has a compute unit to itself (microseconds, boards
// of 14 k to 310 k cells).
static const struct {
    int ry, rz;
    double us;
} kBricks[] = {{8, 7, 9.4}, {8, 8, 10.0}, {12, 8, 13.2}, {10, 10, 15.4}, {16, 8, 16.8}};

static double brick_count(int q, int nx, int ny, int nz)
{
    return std::ceil(nx / 28.0) * std::ceil(ny / (kBricks[q].ry - 4.0)) * std::ceil(nz / (kBricks[q].rz - 4.0));
}

// What a pair of steps in bricks of shape q costs a device that other launches keep
// busy (microseconds): its share of the compute units for a brick's time.
double brick_share(int q, int nx, int ny, int nz, int cus)
{
    return kBricks[q].us * brick_count(q, nx, ny, nz) / std::max(1, cus);
}

// The brick shape for a plain board, -1 where the marching kernel is faster.  A
// second round of bricks costs as much as the first (80 x 72 x 37 cells in 540
// 8 x 8 bricks: 20.8 us; in 252 of 10 x 10: 15.9).  The marching kernel's pair
// takes 15 to 16 us up to about 100 k cells and up to 3.2 us more per further 100 k
// (48 x 43 x 30: 14.7, bricks 9.5; 80 x 72 x 37: 18.2 and 15.9; 130 x 60 x 40: 21.0
// and 17.9); it is left where it is within 5 % of the estimate.  Over 21 boards of
// 6 k to 360 k cells that stepped alone the choice was never the slower one.
int pick_brick(int nx, int ny, int nz, int cus)
{
    const double cells = (double)nx * ny * nz;
    double best = 0.95 * (16.0 + 3.2e-5 * std::max(0.0, cells - 1e5));
    int pick = -1;
    for (int q = 0; q < (int)(sizeof(kBricks) / sizeof(kBricks[0])); ++q) {
        const double us = kBricks[q].us * std::ceil(brick_count(q, nx, ny, nz) / std::max(1, cus));
        if (us < best) {
            best = us;
            pick = q;
        }
    }
    return pick;
}

// Nodes along y and z that a brick of the shape owns.
void brick_owned(int q, int* rows, int* planes)
{
    *rows = kBricks[q].ry - 4;
    *planes = kBricks[q].rz - 4;
}

// Two steps of one plain board from field copy `par` to the other; `rel`: steps
// past the device counter.
hipError_t launch_brick(int q, const BoardDev& b, int par, int rel, bool wide, bool plane, hipStream_t st)
{
    switch (q) {
        case 0: return launch_t<8, 7>(b, par, rel, wide, plane, st);
        case 1: return launch_t<8, 8>(b, par, rel, wide, plane, st);
        case 2: return launch_t<12, 8>(b, par, rel, wide, plane, st);
        case 3: return launch_t<10, 10>(b, par, rel, wide, plane, st);
        case 4: return launch_t<16, 8>(b, par, rel, wide, plane, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace fdtd
