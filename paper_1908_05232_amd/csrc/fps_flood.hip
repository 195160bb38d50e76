// Flood update of one time step on gfx950: the explicit first-order
// Godunov-type finite-volume scheme of Eq. (2) (sec. 2.2) for the shallow-water
// equations of Eq. (1), with wetting/drying and terrain treatment at every
// face, Manning friction, the inflow hydrograph of sec. 3.1, and the CFL time
// step of sec. 3 reduced on the device for the next step.
//
// Readings of the paper used here (the scheme is deferred to Wang et al. 2011):
//   HLLC face flux (Toro) with dry-bed wave speeds (or, selected per launch,
//   HLL for all three components); non-negative hydrostatic
//   reconstruction z_f = max(zL, zR), h* = h - (z_f - z), h* <= h_dry counts
//   as dry; bed slope as the one-sided pressure correction 1/2 g h*^2; walls by
//   mirrored ghost cells passing no mass; transmissive sides by copied ghosts;
//   splitting point-implicit Manning friction with a no-reversal limiter and
//   roughness n0 (1 + min(Np, cap)) from the evacuee counts (sec. 2.4).
//
// Design: one wave marches up a strip of 64 columns (62 outputs plus a halo
// column each side).  At every row each lane loads one cell (coalesced SoA
// rows), computes the y face above it in registers (the face below is carried
// from the previous row), and the x face to its east from its neighbour lane's
// state (cross-lane shuffle); the west face arrives from the neighbour lane.
// Every face is evaluated once; no LDS staging is needed.  Each wave writes
// partials (FP64 mass / volumes, FP32 max wave speed); a finalize kernel (one
// block per scenario) at the end of the step reduces them in a fixed order,
// advances time and sets the next time step (no cross-block fences inside the
// update).  One launch covers the flood tiles of every scenario of an
// ensemble; each wave finds its scenario and reads its parameters.
#include "fps_device.h"

#include <type_traits>

namespace fps {
namespace {

struct Cell {
    float h, qx, qy, z, u, v;
};

__device__ __forceinline__ float rcp(float x) { return __builtin_amdgcn_rcpf(x); }
// A bed elevation as the faces use it: an infinite one (a block no water passes)
// becomes NaN.  The positive and negative parts of a bed step (one instruction
// each) carry a NaN through, so both sides of such a face are dry: a wall, and
// water that lies on the block stays there.  With fmaxf and fminf, which drop a
// NaN, the step between two such cells was none, and the reconstruction of a dry
// cell beside one left a level bed to flow over.
__device__ __forceinline__ float bed(float z) { return fmaf(z, 0.0f, z); }
__device__ __forceinline__ float step_up(float dz) { return __builtin_elementwise_maximum(dz, 0.0f); }
__device__ __forceinline__ float step_down(float dz) { return __builtin_elementwise_minimum(dz, 0.0f); }
// A value used on a path that few waves take: what is computed from it stays
// on that path (the compiler would otherwise compute it always, and select).
__device__ __forceinline__ float rare(float x)
{
    asm volatile("" : "+v"(x));
    return x;
}
__device__ __forceinline__ float sqrt_fast(float x) { return __builtin_amdgcn_sqrtf(x); }

// Whole-wave DPP shifts (a VALU move, no LDS traffic): lane i receives lane
// i + 1 (wave_shl:1) or lane i - 1 (wave_shr:1); the lane without a source
// receives 0 by the bound control (never used: lanes 0 and 63 are halo
// lanes), so no old value has to be set first.
__device__ __forceinline__ float lane_from_above(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v),
                                                                 0x130, 0xF, 0xF, true));
}
__device__ __forceinline__ float lane_from_below(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v),
                                                                 0x138, 0xF, 0xF, true));
}

// Cell (i, j) with i in [-1, nx], j in [-1, ny]; a ghost mirrors the adjacent
// interior cell (normal discharge negated at a wall).  Indices beyond the
// ghost layer clamp into the grid (their values are never used).  The raw
// load and the derived velocities are split so loads can be issued rows ahead.
struct Src {
    const FPS_GLOBAL float* __restrict__ h;
    const FPS_GLOBAL float* __restrict__ qx;
    const FPS_GLOBAL float* __restrict__ qy;
    const FPS_GLOBAL float* __restrict__ z;
};

// Element idx of a grid array: a 32-bit byte offset from a wave-uniform base
// (grids hold fewer than 2^30 cells), so the access is one global load or
// store with the base in scalar registers and no 64-bit address arithmetic.
template <class T>
__device__ __forceinline__ T ld(const FPS_GLOBAL T* base, uint32_t idx)
{
    return *(const FPS_GLOBAL T*)((const FPS_GLOBAL char*)base + idx * (uint32_t)sizeof(T));
}
template <class T>
__device__ __forceinline__ void st_at(FPS_GLOBAL T* base, uint32_t idx, T v)
{
    *(FPS_GLOBAL T*)((FPS_GLOBAL char*)base + idx * (uint32_t)sizeof(T)) = v;
}

__device__ __forceinline__ Cell load_raw(const Src& src, const FvParams& p, int ii, int j)
{
    const int jj = min(max(j, 0), p.ny - 1);
    const uint32_t k = (uint32_t)jj * (uint32_t)p.nx + (uint32_t)ii;
    Cell c;
    c.h = ld(src.h, k);
    c.qx = ld(src.qx, k);
    c.qy = ld(src.qy, k);
    c.z = ld(src.z, k);
    return c;
}

// One face: reconstruction, then the HLLC flux.  (un, ut) are the normal and
// tangential velocities of each side; F0 mass, F2 tangential momentum; GL / GR
// the normal momentum flux less the pressure 1/2 g h*^2 of the reconstructed
// depth on that side (what the cell on that side receives, with the bed-slope
// correction).  Written without divergent branches: every case is evaluated
// and selected, and every fused multiply-add is written out, so that each
// instantiation rounds alike.  HLL is written from the left flux with the wave
// speeds clamped to either side of zero: the one formula is the left flux
// exactly when sL >= 0, the right flux up to rounding when sR <= 0, and the
// star-region flux between; identical states give F exactly, and still water
// F1 = pL = pR.  What a straightforward form would spend on selections is left
// out:
//  - z_f - z_L and z_f - z_R are the positive and the negative part of the
//    bed step;
//  - a face dry on both sides has zero depths, discharges and pressures, so
//    only its denominator needs a guard, not its fluxes;
//  - the contact speed has the sign of the HLL mass flux, whose numerator is
//    sR hL (uL - sL) - sL hR (uR - sR), so F0 selects the tangential velocity
//    (kHll: the tangential momentum by the HLL average instead).
// kProd: the right side's normal velocity is the product rR * qR, which
// enters the sums with it unrounded.
template <bool kHll, bool kProd>
__device__ __forceinline__ void face_march(const FvParams& p, float hL, float unL, float utL, float zL, float hR,
                                           float unR, float utR, float zR, float rR, float qR, bool wall,
                                           float& F0, float& GL, float& GR, float& F2)
{
#pragma clang fp contract(off)
    const float dz = zR - zL;
    float hl = hL - step_up(dz);
    float hr = hR + step_down(dz);
    const bool wetL = hl > p.eps, wetR = hr > p.eps;
    hl = wetL ? hl : 0.0f;
    hr = wetR ? hr : 0.0f;
    const float pL = p.half_g * hl * hl, pR = p.half_g * hr * hr;
    const float cL = sqrt_fast(p.g * hl), cR = sqrt_fast(p.g * hr);
    const float sum = kProd ? fmaf(rR, qR, unL) : unL + unR;
    const float dif = kProd ? fmaf(-rR, qR, unL) : unL - unR;
    const float us = fmaf(0.5f, sum, cL) - cR;
    const float cs = fmaf(0.25f, dif, 0.5f * (cL + cR));
    const float lo = unL - cL, hi = kProd ? fmaf(rR, qR, cR) : unR + cR;
    // dry-bed wave speeds, then both clamped to either side of zero
    float sL = wetR ? fminf(lo, us - cs) : lo;
    float sR = wetR ? fmaxf(hi, us + cs) : fmaf(2.0f, cL, unL);
    sL = fminf(wetL ? sL : fmaf(-2.0f, cR, unR), 0.0f);
    sR = fmaxf(wetL ? sR : hi, 0.0f);
    const float qL = hl * unL, qr = hr * unR;
    const float ML = fmaf(qL, unL, pL), MR = fmaf(qr, unR, pR);
    const float inv = rcp(fmaxf(sR - sL, 1e-30f));
    const float H0 = fmaf(inv, sL * fmaf(hr - hl, sR, fmaf(-hr, unR, qL)), qL);
    const float F1 = fmaf(inv, sL * fmaf(fmaf(hr, unR, -qL), sR, ML - MR), ML);
    F0 = wall ? 0.0f : H0;
    GL = F1 - pL;
    GR = F1 - pR;
    if (kHll) {
        const float tL = qL * utL;
        const float H2 = fmaf(inv, sL * fmaf(fmaf(utR, hr, -(utL * hl)), sR, fmaf(-utR, qr, tL)), tL);
        F2 = wall ? 0.0f : H2;
    } else {
        F2 = F0 * (F0 >= 0.0f ? utL : utR);
    }
}

// The face of the second-order march in fewer instructions still:
//  - with the Riemann invariants a = uL + 2 cL and b = uR - 2 cR the two-
//    rarefaction wave speeds u* -+ c* are b + (a - b) / 4 and a - (a - b) / 4;
//  - a dry side takes the velocity of the front that the wet side sends into
//    it (a, or b), and the wet formulas then give the dry-bed speeds (its
//    depth, celerity and discharge are zero, so it enters nothing else).
// About 50 instructions against 66; the rounding is another (the first-order
// march keeps the form whose results its runs have always had), no larger: the
// difference of the discharges is rounded once, as there.
template <bool kHll>
__device__ __forceinline__ void face_lean(const FvParams& p, float hL, float unL, float utL, float zL, float hR,
                                          float unR, float utR, float zR, bool wall, float& F0, float& GL,
                                          float& GR, float& F2)
{
#pragma clang fp contract(off)
    const float dz = zR - zL;
    float hl = hL - step_up(dz);
    float hr = hR + step_down(dz);
    const bool wetL = hl > p.eps, wetR = hr > p.eps;
    hl = wetL ? hl : 0.0f;
    hr = wetR ? hr : 0.0f;
    const float pL = p.half_g * hl * hl, pR = p.half_g * hr * hr;
    const float cL = sqrt_fast(p.g * hl), cR = sqrt_fast(p.g * hr);
    const float uL = wetL ? unL : fmaf(-2.0f, cR, unR);
    const float uR = wetR ? unR : fmaf(2.0f, cL, unL);
    const float a = fmaf(2.0f, cL, uL), b = fmaf(-2.0f, cR, uR);
    const float d = a - b;
    const float sL = fminf(fminf(uL - cL, fmaf(0.25f, d, b)), 0.0f);
    const float sR = fmaxf(fmaxf(uR + cR, fmaf(-0.25f, d, a)), 0.0f);
    const float qL = hl * uL, qR = hr * uR;
    const float ML = fmaf(qL, uL, pL), MR = fmaf(qR, uR, pR);
    const float k = sL * rcp(fmaxf(sR - sL, 1e-30f));
    const float dq = fmaf(-hr, uR, qL);
    const float H0 = fmaf(k, fmaf(sR, hr - hl, dq), qL);
    const float F1 = fmaf(k, fmaf(-sR, dq, ML - MR), ML);
    F0 = wall ? 0.0f : H0;
    GL = F1 - pL;
    GR = F1 - pR;
    if (kHll) {
        const float tL = qL * utL;
        const float H2 = fmaf(k, fmaf(sR, fmaf(hr, utR, -(hl * utL)), fmaf(-qR, utR, tL)), tL);
        F2 = wall ? 0.0f : H2;
    } else {
        F2 = F0 * (F0 >= 0.0f ? utL : utR);
    }
}

// g n^2 of a cell with npc evacuees
__device__ __forceinline__ float counted_friction(const FvParams& p, int npc)
{
#pragma clang fp contract(off)
    const float n = fmaf(p.n_base, (float)min(npc, p.np_cap), p.n_base);
    return n * (p.g * n);
}

// Manning friction of a wet cell (kn = g n^2), splitting point-implicit with a
// no-reversal limiter, on the discharges; u, v become the new velocities.
// Still water: the reciprocal of its speed counts as 0, so nothing is taken off
// and no factor overflows, however thin the film (1 / speed bounded by a
// constant overflowed in dt Cf r / speed).
__device__ __forceinline__ void friction(const FvParams& p, float dt, float kn, float hn, float& qx, float& qy,
                                         float& u, float& v)
{
#pragma clang fp contract(off)
    const float r = rcp(hn);
    u = qx * r;
    v = qy * r;
    const float uu = u * u, vv = v * v;
    const float V2 = fmaf(u, u, vv);
    const float speed = sqrt_fast(V2), rspeed = V2 > 0.0f ? rcp(speed) : 0.0f;
    const float Cf = kn * __builtin_amdgcn_exp2f(__builtin_amdgcn_logf(hn) * (-1.0f / 3.0f));
    const float Sx = u * -Cf * speed, Sy = v * -Cf * speed;
    const float a = dt * Cf * r * rspeed;
    const float Dx = fmaf(fmaf(u, u + u, vv), a, 1.0f), Dy = fmaf(fmaf(v, v + v, uu), a, 1.0f);
    float dqx = dt * Sx * rcp(Dx), dqy = dt * Sy * rcp(Dy);
    if (fabsf(dqx) > fabsf(qx)) dqx = -qx;
    if (fabsf(dqy) > fabsf(qy)) dqy = -qy;
    qx += dqx;
    qy += dqy;
    u = qx * r;
    v = qy * r;
}

// Wave reductions by DPP lane moves (VALU only, no LDS round trips): pairs,
// quads (quad permutes), eight and sixteen lanes (half-row and row mirrors)
// leave every lane of a row with the row's total; the row broadcasts of lanes
// 15 and 31 then add the rows, lane 63 ending with the wave's total, which is
// returned to every lane.  Rows a broadcast does not write receive 0; the
// first four moves have a source for every lane, so no old value is set for
// them.  A fixed order, so the result is reproducible.
template <int kCtrl, int kRowMask>
__device__ __forceinline__ int dpp_i32(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, kCtrl, kRowMask, 0xF, kRowMask == 0xF);
}
template <int kCtrl, int kRowMask>
__device__ __forceinline__ double dpp_f64(double v)
{
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)dpp_i32<kCtrl, kRowMask>((int)(unsigned)u);
    const unsigned hi = (unsigned)dpp_i32<kCtrl, kRowMask>((int)(unsigned)(u >> 32));
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
constexpr int kQuadSwap1 = 0xB1, kQuadSwap2 = 0x4E;          // quad_perm [1,0,3,2], [2,3,0,1]
constexpr int kRowHalfMirror = 0x141, kRowMirror = 0x140, kRowBcast15 = 0x142, kRowBcast31 = 0x143;

__device__ __forceinline__ double readlane_f64(double v, int l)
{
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)u, l);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(u >> 32), l);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

__device__ __forceinline__ double wave_sum(double v)
{
    v += dpp_f64<kQuadSwap1, 0xF>(v);
    v += dpp_f64<kQuadSwap2, 0xF>(v);
    v += dpp_f64<kRowHalfMirror, 0xF>(v);
    v += dpp_f64<kRowMirror, 0xF>(v);
    v += dpp_f64<kRowBcast15, 0xA>(v);
    v += dpp_f64<kRowBcast31, 0xC>(v);
    return readlane_f64(v, kWave - 1);
}
// Maximum of non-negative floats (the wave speeds): their bit patterns order
// as the values do, so an unsigned maximum of the bits serves (one
// instruction; a NaN, above every finite pattern, comes through, and every
// later level keeps it in the same way: the end of the step sees it and latches
// the fault).  The rows a broadcast skips receive 0 = +0.0.
__device__ __forceinline__ float wave_max_bits(unsigned u)
{
    u = max(u, (unsigned)dpp_i32<kQuadSwap1, 0xF>((int)u));
    u = max(u, (unsigned)dpp_i32<kQuadSwap2, 0xF>((int)u));
    u = max(u, (unsigned)dpp_i32<kRowHalfMirror, 0xF>((int)u));
    u = max(u, (unsigned)dpp_i32<kRowMirror, 0xF>((int)u));
    u = max(u, (unsigned)dpp_i32<kRowBcast15, 0xA>((int)u));
    u = max(u, (unsigned)dpp_i32<kRowBcast31, 0xC>((int)u));
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane((int)u, kWave - 1));
}
__device__ __forceinline__ float wave_max(float v) { return wave_max_bits(__builtin_bit_cast(unsigned, v)); }
// the bits of a partial's wave speed (partials hold FP32 speeds as doubles)
__device__ __forceinline__ unsigned speed_bits(double s) { return __builtin_bit_cast(unsigned, (float)s); }

// Blocks are handed to the 8 XCDs round-robin by block id; this mapping gives
// each XCD a contiguous run of tiles (a band of rows), so the halo columns and
// rows shared by neighbouring tiles are reused in that XCD's L2.
__device__ __forceinline__ int xcd_tile_block(int b, int nblocks)
{
    const int per = nblocks >> 3;          // nblocks is a multiple of 8
    return (b & 7) * per + (b >> 3);
}

// What bounds it: VALU issue, with HBM close behind.  Counted on 8192^2 wet cells
// at 16 rows a wave: 3,526 vector instructions a wave, 220 a row of 62 cells, one
// every 4.1 cycles a SIMD (a wave's instruction takes four); 427 us, 28 B a cell
// at 4.40 TB/s (a 1 GiB copy on the card: 4.95 TB/s).  The form before took 4,449
// (copies of the rows in flight and of the carried face, volumes that only edge
// cells have) and 499 us; this one takes four rows a turn (no copies), has rare
// work behind uniform branches and the leaner face, with the same bits.  1531 x
// 977: 17.7 -> 16.5 us; 6 x 2048^2 with people: 204 -> 191 us.  Loads run four
// rows ahead, so a wave keeps 16 of them in flight.
// kPeople: some scenario may have evacuee counts (they raise the friction), or
// the caller captures the step and may set some later; else the counts are not
// read (4 of 32 B a cell).  A branch on a word of device memory instead, around
// two marches in one kernel, cost 0.5 to 1 % of a step.
template <bool kOne, bool kHll, bool kPeople>
__global__ __launch_bounds__(kFvBlock) void fv_step_kernel(Batch B)
{
    const int lane = threadIdx.x & (kWave - 1);
    // the wave's flattened tile, its scenario and local tile (wave-uniform)
    const int g = __builtin_amdgcn_readfirstlane(
        xcd_tile_block(blockIdx.x, B.fv_blocks) * (kFvBlock / kWave) + (int)(threadIdx.x >> 6));
    int sc, tile;
    if (kOne) {
        sc = 0;
        tile = g;
    } else if (B.s_only >= 0) {
        sc = B.s_only;
        tile = g;
    } else {
        if (g >= B.total_tiles) return;
        sc = find_scenario(B.tile_off, B.S, g);
        tile = g - B.tile_off[sc];
    }
    // parameters by value: wave-uniform registers, not reloaded after the
    // stores of the march (which the compiler cannot tell apart from them)
    const FvParams p = all_at_once(scn_at<kOne>(B, sc).fv);
    if (tile >= p.ntiles) return;
    const StepState st = step_state(gmem(p.st));
    if (!st.active || st.skipped()) return;
    const int cur = st.cur;
    // selects, not indexing, so that the parameter copy stays in registers
    const Src src{gmem<const float>(cur ? p.h[1] : p.h[0]), gmem<const float>(cur ? p.qx[1] : p.qx[0]),
                  gmem<const float>(cur ? p.qy[1] : p.qy[0]), gmem(p.z)};
    FPS_GLOBAL float* __restrict__ ho = gmem(cur ? p.h[0] : p.h[1]);
    FPS_GLOBAL float* __restrict__ qxo = gmem(cur ? p.qx[0] : p.qx[1]);
    FPS_GLOBAL float* __restrict__ qyo = gmem(cur ? p.qy[0] : p.qy[1]);
    const FPS_GLOBAL int32_t* __restrict__ npp = gmem(p.np);
    // mass, boundary fluxes through the x and y sides, clipped depth
    double m_acc = 0.0, vx_acc = 0.0, vy_acc = 0.0, vclip_acc = 0.0;
    float smax = 0.0f;
    const float dt = st.dt, inc = st.inc;
    const float lx = dt * p.inv_dx, ly = dt * p.inv_dy;

    {
        const int sx = tile % p.nsx, sy = tile / p.nsx;
        if (p.jmask) {
            // judge region: skip waves whose output cells meet no set block
            const int bx0 = sx * kStrip / p.jb, bx1 = min(sx * kStrip + kStrip - 1, p.nx - 1) / p.jb;
            const int by0 = sy * p.H / p.jb, by1 = (min(sy * p.H + p.H, p.ny) - 1) / p.jb;
            int any = 0;
            for (int by = by0; by <= by1 && !any; ++by)
                for (int bx = bx0; bx <= bx1; ++bx) any |= p.jmask[by * p.jbx + bx];
            if (!any) {
                if (lane == 0) {
                    FPS_GLOBAL double* dst = gmem(&p.partials[4 * tile]);
                    dst[0] = 0.0;
                    dst[1] = 0.0;
                    dst[2] = 0.0;
                    dst[3] = 0.0;
                }
                return;
            }
        }
        const int i = sx * kStrip - 1 + lane;
        const int ii = min(max(i, 0), p.nx - 1);
        const int j0 = sy * p.H, j1 = min(j0 + p.H, p.ny);
        const bool out_lane = lane >= 1 && lane <= kStrip && i < p.nx;
        // what only the strips on the west and east sides do (wave-uniform)
        const bool first_strip = sx == 0, last_strip = sx == p.nsx - 1;
        const bool side_strip = first_strip || last_strip;
        const bool mirror_x = (i < 0 && p.bc[0] == FPS_BC_WALL) || (i >= p.nx && p.bc[1] == FPS_BC_WALL);
        const bool xwall = (i == -1 && p.bc[0] == FPS_BC_WALL) ||
                           (i + 1 == p.nx && p.bc[1] == FPS_BC_WALL);
        const bool inflow_x = (p.inflow_side == FPS_SIDE_W && first_strip) || (p.inflow_side == FPS_SIDE_E && last_strip);
        const int in_row = p.inflow_side == FPS_SIDE_S ? 0 : p.inflow_side == FPS_SIDE_N ? p.ny - 1 : -1;
        const int in_col = p.inflow_side == FPS_SIDE_W ? 0 : p.nx - 1;
        const bool out_w = first_strip && p.bc[0] == FPS_BC_TRANSMISSIVE, out_e = last_strip && p.bc[1] == FPS_BC_TRANSMISSIVE;
        const int out_s = p.bc[2] == FPS_BC_TRANSMISSIVE ? 0 : -1, out_n = p.bc[3] == FPS_BC_TRANSMISSIVE ? p.ny - 1 : -1;
        const float kn0 = p.n_base * (p.g * p.n_base);        // g n^2 of a cell with no evacuees
        // largest |u| + c and |v| + c of the lane's cells, as bits (they order
        // as the non-negative values do, and a NaN comes through)
        unsigned umax = 0, vmax = 0;

        // the derived velocities of a raw row (ghost rows and columns mirrored at
        // walls) and the reciprocal depth
        auto prim = [&](const Cell& raw, int j, float& r) {
            Cell c = raw;
            c.z = bed(raw.z);
            r = c.h > p.eps ? rcp(c.h) : 0.0f;
            if (side_strip && mirror_x) c.qx = -c.qx;
            if ((j < 0 && p.bc[2] == FPS_BC_WALL) || (j >= p.ny && p.bc[3] == FPS_BC_WALL)) c.qy = -c.qy;
            c.u = c.qx * r;
            c.v = c.qy * r;
            return c;
        };
        struct Flux {
            float F0, G, F2;       // mass, normal momentum less the upper cell's pressure, tangential momentum
        };
        // row j with its cells c, the face below it s and the raw row above it
        // (held in ring, which then takes the row four further up): the face
        // above goes to n, the cells above to nb
        auto row = [&](const Cell& c, Cell& nb, Cell& ring, int j, const Flux& s, Flux& n, auto fetch) {
            const uint32_t k = (uint32_t)j * (uint32_t)p.nx + (uint32_t)ii;     // ii: in the grid on every lane
            int npc = 0;
            if (kPeople) npc = ld(npp, k);
            float rn;
            nb = prim(ring, j + 1, rn);
            // a row past the tile's last need is replaced by that row (cached):
            // a load under a condition would make the compiler copy the ring,
            // and so wait for its loads, at every row
            if constexpr (decltype(fetch)::value) ring = load_raw(src, p, ii, min(j + 5, j1));
            // north face (y normal: v normal, u tangential)
            float Gn;
            face_march<kHll, true>(p, c.h, c.v, c.u, c.z, nb.h, nb.v, nb.u, nb.z, rn, nb.qy,
                                   j + 1 == p.ny && p.bc[3] == FPS_BC_WALL, n.F0, Gn, n.G, n.F2);
            // east face with the neighbour lane's cell; the west face is the east face of the lane below
            const float eh = lane_from_above(c.h), eu = lane_from_above(c.u);
            const float ev = lane_from_above(c.v), ez = lane_from_above(c.z);
            float Fe0, Ge, Gw_next, Fe2;
            face_march<kHll, false>(p, c.h, c.u, c.v, c.z, eh, eu, ev, ez, 0.0f, 0.0f, xwall, Fe0, Ge, Gw_next, Fe2);
            const float Fw0 = lane_from_below(Fe0), Gw = lane_from_below(Gw_next), Fw2 = lane_from_below(Fe2);
            if (out_lane) {
#pragma clang fp contract(off)
                float hn = c.h - fmaf(ly, n.F0 - s.F0, lx * (Fe0 - Fw0));
                float qxn = c.qx - fmaf(ly, n.F2 - s.F2, lx * (Ge - Gw));
                float qyn = c.qy - fmaf(ly, Gn - s.G, lx * (Fe2 - Fw2));
                // inflow line source (sec. 3.1)
                if (j == in_row) {
                    if (i >= p.c0 && i < p.c1) hn += inc;
                } else if (inflow_x && j >= p.c0 && j < p.c1) {
                    if (i == in_col) hn += inc;
                }
                // non-negative depth, no discharge on dry cells
                if (hn < 0.0f) {
                    vclip_acc -= (double)rare(hn);
                    hn = 0.0f;
                }
                if (hn > p.eps) {
                    float u, v;
                    friction(p, dt, kPeople ? counted_friction(p, npc) : kn0, hn, qxn, qyn, u, v);
                    const float cel = sqrt_fast(p.g * hn);
                    umax = max(umax, __builtin_bit_cast(unsigned, fabsf(u) + cel));
                    vmax = max(vmax, __builtin_bit_cast(unsigned, fabsf(v) + cel));
                } else {
                    qxn = 0.0f;
                    qyn = 0.0f;
                }
                m_acc += (double)hn;
                // outflow through transmissive sides
                if (out_w || out_e || j == out_s || j == out_n) {
                    if (out_w && i == 0) vx_acc -= (double)rare(Fw0);
                    if (out_e && i == p.nx - 1) vx_acc += (double)rare(Fe0);
                    if (j == out_s) vy_acc -= (double)rare(s.F0);
                    if (j == out_n) vy_acc += (double)rare(n.F0);
                }
                st_at(ho, k, hn);
                st_at(qxo, k, qxn);
                st_at(qyo, k, qyn);
            }
        };

        // The rows j0 - 1 and j0 form the face below the tile; then the march,
        // four rows a turn, so that the cells, the carried face and the four
        // rows in flight stay where they are instead of being moved along.
        // Every row runs the same code (same rounding) whatever the tile height.
        Cell A = load_raw(src, p, ii, j0 - 1);
        Cell R0 = load_raw(src, p, ii, j0), R1 = {}, R2 = {}, R3 = {}, Bc;
        if (j0 + 1 <= j1) R1 = load_raw(src, p, ii, j0 + 1);
        if (j0 + 2 <= j1) R2 = load_raw(src, p, ii, j0 + 2);
        if (j0 + 3 <= j1) R3 = load_raw(src, p, ii, j0 + 3);
        Flux Fa, Fb;
        {
            float ra, rb, unused;
            A = prim(A, j0 - 1, ra);
            Bc = prim(R0, j0, rb);
            if (j0 + 4 <= j1) R0 = load_raw(src, p, ii, j0 + 4);
            face_march<kHll, true>(p, A.h, A.v, A.u, A.z, Bc.h, Bc.v, Bc.u, Bc.z, rb, Bc.qy,
                                   j0 == 0 && p.bc[2] == FPS_BC_WALL, Fa.F0, unused, Fa.G, Fa.F2);
        }
        const std::true_type fetch{};
        const std::false_type last{};
        int j = j0;
        for (; j + 4 <= j1; j += 4) {
            row(Bc, A, R1, j, Fa, Fb, fetch);
            row(A, Bc, R2, j + 1, Fb, Fa, fetch);
            row(Bc, A, R3, j + 2, Fa, Fb, fetch);
            row(A, Bc, R0, j + 3, Fb, Fa, fetch);
        }
        if (j < j1) {
            row(Bc, A, R1, j, Fa, Fb, last);
            if (j + 1 < j1) row(A, Bc, R2, j + 1, Fb, Fa, last);
            if (j + 2 < j1) row(Bc, A, R3, j + 2, Fa, Fb, last);
        }
        const float su = __builtin_bit_cast(float, umax) * p.inv_dx, sv = __builtin_bit_cast(float, vmax) * p.inv_dy;
        smax = __builtin_bit_cast(float, max(__builtin_bit_cast(unsigned, su), __builtin_bit_cast(unsigned, sv)));
    }
    // wave partials, fixed reduction order; reduced by the finalize kernel.
    // Outflow and clipped volumes are zero in almost every wave (outflow only
    // on transmissive sides, clipping only where a depth went negative): their
    // sums are skipped when no lane holds a non-zero value.
    m_acc = wave_sum(m_acc);
    double vout_acc = (double)dt * (vx_acc * p.dy + vy_acc * p.dx);
    if (__ballot(vout_acc != 0.0)) vout_acc = wave_sum(vout_acc);
    else vout_acc = 0.0;
    if (__ballot(vclip_acc != 0.0)) vclip_acc = wave_sum(vclip_acc);
    else vclip_acc = 0.0;
    smax = wave_max(smax);
    if (lane == 0) {
        FPS_GLOBAL double* dst = gmem(&p.partials[4 * tile]);
        dst[0] = m_acc;
        dst[1] = vout_acc;
        dst[2] = vclip_acc;
        dst[3] = (double)smax;
        // one flag per group of blocks; every wet wave of the group stores the
        // same 1 with a plain store (no read-modify-write, nothing to wait for:
        // the wave ends as soon as its stores are issued)
        if (!(smax <= 0.0f)) st_at(gmem(p.wet), (uint32_t)(kWetStride * (blockIdx.x & (kWetSlots - 1))), 1);
    }
}

// ---------------------------------------------------------------------------
// Second-order variant (the scheme the paper reduced to first order, sec.
// 2.2): MUSCL reconstruction of (h, eta = h + z, u, v) per direction with
// the minmod limiter (zero slope where the cell or a neighbour in that
// direction is dry, and in ghost cells), the hydrostatic reconstruction and
// the HLLC / HLL flux of the first-order scheme at each face on the
// reconstructed states, the second-order bed-slope form of Audusse et al.
// (2004) (each face adds g/2 (h_f^2 - h*_f^2) to its side's normal momentum,
// each cell the centred -g/2 (h_w + h_e)(z_e - z_w)), and Heun's two-stage
// Runge-Kutta step: U1 = U + dt L(U), U' = (U + U1 + dt L(U1)) / 2, with the
// depth cleanup after each stage and the inflow and friction once after both.
//
// The march of the first-order update widened to the stencil of radius 2: a
// wave holds 64 adjacent columns and owns the middle kStrip2 (two halo lanes
// a side), marching down its rows with a window of three rows in registers.
// Each row is reconstructed once per direction: in x from the neighbour
// lanes' cells (DPP moves), in y from the window.  Each face is evaluated
// once: a lane forms its west face (the east state of the lane below against
// its own west state) and takes its east face from the lane above; the face
// below row r is formed when row r is reconstructed and, carried, is the
// face above row r - 1, which is then complete and updated (one row behind).
// ---------------------------------------------------------------------------
constexpr int kStrip2 = kWave - 4;      // output columns of one wave in the second-order march

struct V4 {
    float h, eta, u, v;     // depth, surface elevation, velocities (0 where h <= h_dry)
};

// minmod: the median of the two differences and zero
__device__ __forceinline__ float minmod(float a, float b) { return __builtin_amdgcn_fmed3f(a, b, 0.0f); }

__device__ __forceinline__ V4 operator-(const V4& a, const V4& b)
{
    return V4{a.h - b.h, a.eta - b.eta, a.u - b.u, a.v - b.v};
}

// cell c reconstructed at its two faces in one direction from the differences
// f (to the next cell) and g (from the cell before); half: 1/2, or 0 for a
// ghost or next to a dry cell (no slope).  Returns the change of the surface
// across the cell, between the face values as rounded.  A face value lies between the cell's and its mean with a
// neighbour, so a face is dry only where the cell is, and its velocity is then 0.
__device__ __forceinline__ float recon(const V4& c, const V4& f, const V4& g, float half, V4& lo, V4& hi)
{
    const V4 m{minmod(f.h, g.h), minmod(f.eta, g.eta), minmod(f.u, g.u), minmod(f.v, g.v)};
    lo = V4{fmaf(-half, m.h, c.h), fmaf(-half, m.eta, c.eta), fmaf(-half, m.u, c.u), fmaf(-half, m.v, c.v)};
    hi = V4{fmaf(half, m.h, c.h), fmaf(half, m.eta, c.eta), fmaf(half, m.u, c.u), fmaf(half, m.v, c.v)};
    return hi.eta - lo.eta;
}

// One Runge-Kutta stage of the second-order variant over one tile (kStage 1:
// U1 = U + dt L(U) into the stage buffer; kStage 2: U' = (U + U1 + dt L(U1))
// / 2 into the other ping-pong buffer, then inflow, friction, volumes and the
// wave speed).  The outflow and clipped volumes of stage 1 are left in the
// tile's partial slots for stage 2 to add to (each stage counts half).
//
// The bed slope: a face gives its cell G + 1/2 g h_f^2 (G the momentum flux
// less 1/2 g h*^2), the centred term 1/2 g (h_w + h_e)(z_e - z_w); the squares
// and that term are together 1/2 g (h_w + h_e)(eta_e - eta_w), and h_w + h_e is
// twice the cell's depth, so a cell receives G_e - G_w + g h (eta_e - eta_w):
// one multiply-add, and nothing where the surface is level.  eta_e - eta_w is
// taken from the face values as rounded, which the faces used too: the slope
// itself, unrounded, leaves 3 % more rounding error in the discharges after
// eight steps (rms on long waves 1.10e-8 m^2/s; 1.06e-8 so, and 1.07e-8 with the
// terms as squares).
//
// What bounds it: VALU issue up to a few million cells (counted at 2048^2 and 8
// rows a wave: 223 and 289 vector instructions a row, one every 4.3 cycles a SIMD
// while waves run), HBM (72 B a cell over the two stages) beyond.  Before this
// form (general faces and limiter, window and carried faces moved along every
// row, one row of U^n loaded where it is used) both stages took 122 us at 2048^2
// and 16 rows a wave; now 70 us at 8 rows, and 972 us at 8192^2 (4.97 TB/s).  It
// holds 98 VGPRs in stage 1 and 116 in stage 2 (four waves a SIMD; stage 1 at 96
// and five took as long); the scheduling barriers keep the two faces of a row
// from being interleaved, which would take 123.
template <bool kOne, bool kHll, bool kPeople, int kStage>
__global__ __launch_bounds__(kFvBlock) void fv2_stage_kernel(Batch B)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int g = __builtin_amdgcn_readfirstlane(
        xcd_tile_block(blockIdx.x, B.fv_blocks) * (kFvBlock / kWave) + (int)(threadIdx.x >> 6));
    int sc, tile;
    if (kOne) {
        sc = 0;
        tile = g;
    } else if (B.s_only >= 0) {
        sc = B.s_only;
        tile = g;
    } else {
        if (g >= B.total_tiles) return;
        sc = find_scenario(B.tile_off, B.S, g);
        tile = g - B.tile_off[sc];
    }
    const FvParams p = all_at_once(scn_at<kOne>(B, sc).fv);
    if (tile >= p.ntiles) return;
    const StepState st = step_state(gmem(p.st));
    if (!st.active || st.skipped()) return;
    const int cur = st.cur;
    const Src s0{gmem<const float>(cur ? p.h[1] : p.h[0]), gmem<const float>(cur ? p.qx[1] : p.qx[0]),
                 gmem<const float>(cur ? p.qy[1] : p.qy[0]), gmem(p.z)};
    const Src s1{gmem<const float>(p.h1), gmem<const float>(p.qx1), gmem<const float>(p.qy1), gmem(p.z)};
    const Src& src = kStage == 1 ? s0 : s1;        // the state the residual is taken of
    FPS_GLOBAL float* __restrict__ ho = gmem(kStage == 1 ? p.h1 : cur ? p.h[0] : p.h[1]);
    FPS_GLOBAL float* __restrict__ qxo = gmem(kStage == 1 ? p.qx1 : cur ? p.qx[0] : p.qx[1]);
    FPS_GLOBAL float* __restrict__ qyo = gmem(kStage == 1 ? p.qy1 : cur ? p.qy[0] : p.qy[1]);
    const FPS_GLOBAL int32_t* __restrict__ npp = gmem(p.np);
    const float dt = st.dt, inc = st.inc;
    const float lx = dt * p.inv_dx, ly = dt * p.inv_dy;
    const int sx = tile % p.nsx, sy = tile / p.nsx;
    const int i = sx * kStrip2 - 2 + lane;
    const int ii = min(max(i, 0), p.nx - 1);
    const int j0 = sy * p.H, j1 = min(j0 + p.H, p.ny);
    const bool out_lane = lane >= 2 && lane < 2 + kStrip2 && i < p.nx;
    const bool gx = i < 0 || i >= p.nx;       // ghost column (no x slope)
    const bool mirror_x = (i < 0 && p.bc[0] == FPS_BC_WALL) || (i >= p.nx && p.bc[1] == FPS_BC_WALL);
    // the west face of this lane's column is a wall face
    const bool xwall = (i == 0 && p.bc[0] == FPS_BC_WALL) || (i == p.nx && p.bc[1] == FPS_BC_WALL);
    // what only the strips on the west and east sides do (wave-uniform)
    const bool first_strip = sx == 0, last_strip = sx == p.nsx - 1;
    const bool out_w = first_strip && p.bc[0] == FPS_BC_TRANSMISSIVE, out_e = last_strip && p.bc[1] == FPS_BC_TRANSMISSIVE;
    const int out_s = p.bc[2] == FPS_BC_TRANSMISSIVE ? 0 : -1, out_n = p.bc[3] == FPS_BC_TRANSMISSIVE ? p.ny - 1 : -1;
    const bool inflow_x = (p.inflow_side == FPS_SIDE_W && first_strip) || (p.inflow_side == FPS_SIDE_E && last_strip);
    const int in_row = p.inflow_side == FPS_SIDE_S ? 0 : p.inflow_side == FPS_SIDE_N ? p.ny - 1 : -1;
    const int in_col = p.inflow_side == FPS_SIDE_W ? 0 : p.nx - 1;
    const float kn0 = p.n_base * (p.g * p.n_base);
    // mass, boundary fluxes through the x and y sides, clipped depth
    double m_acc = 0.0, vx_acc = 0.0, vy_acc = 0.0, vclip_acc = 0.0;
    unsigned umax = 0, vmax = 0;     // largest |u| + c and |v| + c of the lane's cells, as bits
    FPS_GLOBAL double* part = gmem(&p.partials[4 * tile]);

    // a row of cells: surface and velocities, the raw discharges, and which lanes are wet
    struct Row {
        V4 v;
        float qx, qy;
        unsigned long long wet;
    };
    auto derive = [&](const Cell& raw, int j) {
        Row c;
        const bool wet = raw.h > p.eps;
        const float r = wet ? rcp(raw.h) : 0.0f;
        c.qx = raw.qx;
        c.qy = raw.qy;
        c.v.h = raw.h;
        c.v.eta = raw.h + bed(raw.z);
        c.v.u = raw.qx * r;
        c.v.v = raw.qy * r;
        if (mirror_x) c.v.u = -c.v.u;
        if ((j < 0 && p.bc[2] == FPS_BC_WALL) || (j >= p.ny && p.bc[3] == FPS_BC_WALL)) c.v.v = -c.v.v;
        c.wet = __ballot(wet);
        return c;
    };
    // what a row hands to the one above: its north face state, and its cells'
    // change but the north face's part with the values it applies to
    struct Up {
        V4 n;
        float ih, iqx, iqy, h, qx, qy;
        float bh, bqx, bqy;      // stage 2: the state at the start of the step
    };

    // Row r (c; the row above it nb), the differences gy from the row below
    // and its wetness wb; lower: what row r - 1 hands up.  Forms the face below
    // row r (first: none below the tile's halo row), completes row r - 1
    // (done) and starts row r (start), leaving up and the differences fy.
    auto row = [&](const Row& c, const Row& nb, const V4& gy, unsigned long long wb, int r, const Up& lower, Up& up,
                   V4& fy, auto face_, auto done_, auto start_) {
#pragma clang fp contract(off)
        constexpr bool face = decltype(face_)::value, done = decltype(done_)::value, start = decltype(start_)::value;
        fy = nb.v - c.v;
        const bool inside = r >= 0 && r < p.ny;      // a ghost row has no slope
        const unsigned long long wy = inside ? wb & c.wet & nb.wet : 0ull;
        V4 sr;
        const float ey = recon(c.v, fy, gy, __builtin_amdgcn_inverse_ballot_w64(wy) ? 0.5f : 0.0f, sr, up.n);
        float F0 = 0.0f, GL = 0.0f, GR = 0.0f, F2 = 0.0f;
        if (face)
            face_lean<kHll>(p, lower.n.h, lower.n.v, lower.n.u, lower.n.eta - lower.n.h, sr.h, sr.v, sr.u,
                            sr.eta - sr.h, (r == 0 && p.bc[2] == FPS_BC_WALL) || (r == p.ny && p.bc[3] == FPS_BC_WALL),
                            F0, GL, GR, F2);
        __builtin_amdgcn_sched_barrier(0);
        if (done) {
            // row r - 1 is complete: its north face is this one
            const int jr = r - 1;
            if (out_lane) {
                const uint32_t k = (uint32_t)jr * (uint32_t)p.nx + (uint32_t)i;
                if (jr == out_n) vy_acc += (double)rare(F0);
                float h = lower.h - fmaf(ly, F0, lower.ih), qx = lower.qx - fmaf(ly, F2, lower.iqx),
                      qy = lower.qy - fmaf(ly, GL, lower.iqy);
                if (h < 0.0f) {
                    vclip_acc -= (double)rare(h);
                    h = 0.0f;
                }
                if (!(h > p.eps)) {
                    qx = 0.0f;
                    qy = 0.0f;
                }
                if (kStage == 2) {
                    h = 0.5f * (lower.bh + h);
                    qx = 0.5f * (lower.bqx + qx);
                    qy = 0.5f * (lower.bqy + qy);
                    if (jr == in_row) {
                        if (i >= p.c0 && i < p.c1) h += inc;
                    } else if (inflow_x && jr >= p.c0 && jr < p.c1) {
                        if (i == in_col) h += inc;
                    }
                    if (h > p.eps) {
                        float u, v;
                        friction(p, dt, kPeople ? counted_friction(p, ld(npp, k)) : kn0, h, qx, qy, u, v);
                        const float cel = sqrt_fast(p.g * h);
                        umax = max(umax, __builtin_bit_cast(unsigned, fabsf(u) + cel));
                        vmax = max(vmax, __builtin_bit_cast(unsigned, fabsf(v) + cel));
                    } else {
                        qx = 0.0f;
                        qy = 0.0f;
                    }
                    m_acc += (double)h;
                }
                st_at(ho, k, h);
                st_at(qxo, k, qx);
                st_at(qyo, k, qy);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        if (start) {
            if (kStage == 2) {
                // the state at the start of the step, used when the row is complete
                const uint32_t k = (uint32_t)r * (uint32_t)p.nx + (uint32_t)ii;
                up.bh = ld(s0.h, k);
                up.bqx = ld(s0.qx, k);
                up.bqy = ld(s0.qy, k);
            }
            // x reconstruction from the neighbour lanes, the west face, and the
            // east face from the lane above
            const V4 fx{lane_from_above(c.v.h) - c.v.h, lane_from_above(c.v.eta) - c.v.eta,
                        lane_from_above(c.v.u) - c.v.u, lane_from_above(c.v.v) - c.v.v};
            const V4 gw{lane_from_below(fx.h), lane_from_below(fx.eta), lane_from_below(fx.u), lane_from_below(fx.v)};
            const unsigned long long wx = c.wet & (c.wet >> 1) & (c.wet << 1);
            V4 wr, er;
            const float ex = recon(c.v, fx, gw, __builtin_amdgcn_inverse_ballot_w64(wx) && !gx ? 0.5f : 0.0f, wr, er);
            const V4 el{lane_from_below(er.h), lane_from_below(er.eta), lane_from_below(er.u), lane_from_below(er.v)};
            float Fw0, GwL, GwR, Fw2;
            face_lean<kHll>(p, el.h, el.u, el.v, el.eta - el.h, wr.h, wr.u, wr.v, wr.eta - wr.h, xwall, Fw0, GwL, GwR,
                            Fw2);
            const float Fe0 = lane_from_above(Fw0), Ge = lane_from_above(GwL), Fe2 = lane_from_above(Fw2);
            const float gh = p.g * c.v.h;
            up.ih = fmaf(-ly, F0, lx * (Fe0 - Fw0));
            up.iqx = fmaf(-ly, F2, lx * fmaf(gh, ex, Ge - GwR));
            up.iqy = fmaf(ly, fmaf(gh, ey, -GR), lx * (Fe2 - Fw2));
            up.h = c.v.h;
            up.qx = c.qx;
            up.qy = c.qy;
            // outflow of the row through the west, east and south sides
            if (out_lane) {
                if (r == out_s) vy_acc -= (double)rare(F0);
                if (out_w && i == 0) vx_acc -= (double)rare(Fw0);
                if (out_e && i == p.nx - 1) vx_acc += (double)rare(Fe0);
            }
        }
    };
    const std::true_type yes{};
    const std::false_type no{};

    // Rows j0 - 1 to j1 + 1 with a ring of rows in flight (rows past the last
    // one needed are replaced by it); two rows a turn, so that the window stays
    // where it is.
    auto fetch = [&](int j) { return load_raw(src, p, ii, min(j, j1 + 1)); };
    Row A, Bc;
    Up Ua, Ub;
    V4 fa, fb;
    unsigned long long wl;
    {
        const Cell r0 = load_raw(src, p, ii, j0 - 2), r1 = load_raw(src, p, ii, j0 - 1), r2 = load_raw(src, p, ii, j0);
        A = derive(r0, j0 - 2);
        Bc = derive(r1, j0 - 1);
        fb = Bc.v - A.v;
        wl = A.wet;
        A = derive(r2, j0);
    }
    Cell R0 = fetch(j0 + 1), R1 = fetch(j0 + 2);
    // row j0 - 1: its north state only
    row(Bc, A, fb, wl, j0 - 1, Ub, Ua, fa, no, no, no);
    wl = Bc.wet;
    Bc = derive(R0, j0 + 1);
    R0 = fetch(j0 + 3);
    // row j0: its faces, no row below to complete
    row(A, Bc, fa, wl, j0, Ua, Ub, fb, yes, no, yes);
    wl = A.wet;
    A = derive(R1, j0 + 2);
    R1 = fetch(j0 + 4);
    int r = j0 + 1;
    for (; r + 2 <= j1; r += 2) {
        row(Bc, A, fb, wl, r, Ub, Ua, fa, yes, yes, yes);
        wl = Bc.wet;
        Bc = derive(R0, r + 2);
        R0 = fetch(r + 4);
        row(A, Bc, fa, wl, r + 1, Ua, Ub, fb, yes, yes, yes);
        wl = A.wet;
        A = derive(R1, r + 3);
        R1 = fetch(r + 5);
    }
    if (r < j1) {
        row(Bc, A, fb, wl, r, Ub, Ua, fa, yes, yes, yes);
        wl = Bc.wet;
        Bc = derive(R0, r + 2);
        row(A, Bc, fa, wl, r + 1, Ua, Ub, fb, yes, yes, no);
    } else {
        row(Bc, A, fb, wl, r, Ub, Ua, fa, yes, yes, no);
    }
    // the two stages' volumes in the tile's partials, each stage for half
    // (stage 1 leaves its outflow and clipped volumes there for stage 2)
    double vout_acc = 0.5 * (double)dt * (vx_acc * p.dy + vy_acc * p.dx);
    vclip_acc *= 0.5;
    if (__ballot(vout_acc != 0.0)) vout_acc = wave_sum(vout_acc);
    else vout_acc = 0.0;
    if (__ballot(vclip_acc != 0.0)) vclip_acc = wave_sum(vclip_acc);
    else vclip_acc = 0.0;
    if (kStage == 1) {
        if (lane == 0) {
            part[1] = vout_acc;
            part[2] = vclip_acc;
        }
        return;
    }
    m_acc = wave_sum(m_acc);
    const float su = __builtin_bit_cast(float, umax) * p.inv_dx, sv = __builtin_bit_cast(float, vmax) * p.inv_dy;
    const float smax = wave_max(__builtin_bit_cast(
        float, max(__builtin_bit_cast(unsigned, su), __builtin_bit_cast(unsigned, sv))));
    if (lane == 0) {
        const double vo1 = part[1], vc1 = part[2];
        part[0] = m_acc;
        part[1] = vo1 + vout_acc;
        part[2] = vc1 + vclip_acc;
        part[3] = (double)smax;
        if (!(smax <= 0.0f)) st_at(gmem(p.wet), (uint32_t)(kWetStride * (blockIdx.x & (kWetSlots - 1))), 1);
    }
}

// Scan of the current state only: mass, wetness and the time step that the
// next update will use (no time advance).  One scenario; one partial per block.
__global__ __launch_bounds__(kFvBlock) void fv_scan_kernel(Batch B, int sc)
{
    const FvParams& p = B.scn[sc].fv;
    const int cur = p.st->cur;
    const float* __restrict__ hh = p.h[cur];
    const float* __restrict__ qxx = p.qx[cur];
    const float* __restrict__ qyy = p.qy[cur];
    double m_acc = 0.0;
    float smax = 0.0f;
    const int64_t nc = (int64_t)p.nx * p.ny;
    for (int64_t k = (int64_t)blockIdx.x * kFvBlock + threadIdx.x; k < nc;
         k += (int64_t)gridDim.x * kFvBlock) {
        float h = hh[k];
        m_acc += (double)h;
        if (h > p.eps) {
            float r = rcp(h);
            float u = qxx[k] * r, v = qyy[k] * r;
            float cel = sqrt_fast(p.g * h);
            smax = fmaxf(smax, fmaxf((fabsf(u) + cel) * p.inv_dx, (fabsf(v) + cel) * p.inv_dy));
        }
    }
    __shared__ double wred[kFvBlock / kWave][2];
    m_acc = wave_sum(m_acc);
    smax = wave_max(smax);
    if ((threadIdx.x & (kWave - 1)) == 0) {
        wred[threadIdx.x >> 6][0] = m_acc;
        wred[threadIdx.x >> 6][1] = (double)smax;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double s0 = 0, s3 = 0;
        for (int w = 0; w < kFvBlock / kWave; ++w) {
            s0 += wred[w][0];
            s3 = fmax(s3, wred[w][1]);
        }
        double* dst = &p.partials[4 * blockIdx.x];
        dst[0] = s0;
        dst[1] = 0.0;
        dst[2] = 0.0;
        dst[3] = s3;
    }
}

// First level of the reduction of a large grid's partials (more than
// kRedMin tiles): block c adds the partials of tiles [c kRedTiles, (c + 1)
// kRedTiles) in a fixed order into the first of them, which the end-of-step
// block then reads.  One block reading them all is a chain of dependent loads
// (8192^2 at 16 rows a wave: 68,096 partials).
__global__ __launch_bounds__(kFvBlock) void fv_reduce_kernel(Batch B, int s_first)
{
    const FvParams& p = B.scn[s_first + blockIdx.y].fv;
    const int ntiles = p.ntiles, t0 = blockIdx.x * kRedTiles;
    if (ntiles <= kRedMin || t0 >= ntiles) return;
    constexpr int kPer = kRedTiles / kFvBlock;
    double2* P2 = reinterpret_cast<double2*>(p.partials);
    double2 a[kPer], c[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int b = min(t0 + (int)threadIdx.x + u * kFvBlock, ntiles - 1);
        a[u] = P2[2 * b];
        c[u] = P2[2 * b + 1];
    }
    double m = 0.0, vo = 0.0, vc = 0.0;
    unsigned sm = 0;
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        if (t0 + (int)threadIdx.x + u * kFvBlock < ntiles) {
            m += a[u].x;
            vo += a[u].y;
            vc += c[u].x;
            sm = max(sm, speed_bits(c[u].y));
        }
    }
    __shared__ double red[kFvBlock / kWave][3];
    __shared__ unsigned redsm[kFvBlock / kWave];
    m = wave_sum(m);
    vo = wave_sum(vo);
    vc = wave_sum(vc);
    sm = __builtin_bit_cast(unsigned, wave_max_bits(sm));
    if ((threadIdx.x & (kWave - 1)) == 0) {
        const int w = threadIdx.x >> 6;
        red[w][0] = m;
        red[w][1] = vo;
        red[w][2] = vc;
        redsm[w] = sm;
    }
    __syncthreads();      // every partial of the block has been read
    if (threadIdx.x == 0) {
        for (int w = 1; w < kFvBlock / kWave; ++w) {
            m += red[w][0];
            vo += red[w][1];
            vc += red[w][2];
            sm = max(sm, redsm[w]);
        }
        P2[2 * t0] = make_double2(m, vo);
        P2[2 * t0 + 1] = make_double2(vc, (double)__builtin_bit_cast(float, sm));
    }
}

// Exact integral over [a, b] of the piecewise-linear hydrograph (sec. 3.1),
// on one wave whose lane k holds knot k (tk, qk) for k < nh: lane k takes the
// part of [a, b] in [t_k, t_k+1] by the trapezoid rule (exact on a linear
// piece), lane 0 the constant part before the first knot, lane nh - 1 the
// constant part after the last; the pieces are added in time order.  Every
// lane returns the total.
__device__ double wave_hydro_integral(int nh, double tk, double qk, double a, double b)
{
    const int lane = threadIdx.x & (kWave - 1);
    // the next knot from the lane above (a whole-wave DPP shift; lane 63,
    // which gets 0, has no next knot: nh <= 64)
    const double tn = dpp_f64<0x130, 0xF>(tk), qn = dpp_f64<0x130, 0xF>(qk);
    if (nh <= 0 || !(b > a)) return 0.0;
    double piece = 0.0, before = 0.0, after = 0.0;
    if (lane + 1 < nh) {
        const double lo = fmax(a, tk), hi = fmin(b, tn);
        if (hi > lo) {
            const double ql = qk + ((lo - tk) / (tn - tk)) * (qn - qk);
            const double qh = qk + ((hi - tk) / (tn - tk)) * (qn - qk);
            piece = 0.5 * (ql + qh) * (hi - lo);
        }
    }
    if (lane == 0 && a < tk) before = qk * (fmin(b, tk) - a);
    if (lane == nh - 1 && b > tk) after = qk * (b - fmax(a, tk));
    double total = readlane_f64(before, 0);
    for (unsigned long long m = __ballot(piece != 0.0); m; m &= m - 1)
        total += readlane_f64(piece, __builtin_ctzll(m));
    return total + readlane_f64(after, nh - 1);
}

// End of a step: a row of blocks, one per scenario, updates the states; beside
// them, the next rows rebuild the neighbour bins of scenarios binned in LDS, and
// further rows count the chunks of the others (they share no data).  The state update
// reduces the flood partials in a fixed order, advances time, sets the next CFL
// time step (sec. 3) and inflow depth, and applies the sandbag drops of the step
// to the barrier line (sec. 2.4).  Mode 1 only recomputes the time step and mass
// of the current state, of the scenarios from s_first.
template <bool kOne>
__global__ __launch_bounds__(kScanThreads) void finalize_kernel(Batch B, int mode, int s_first)
{
    if (blockIdx.y > 0) {
        const int r = (int)blockIdx.y - 1, tiles = B.fin_tiles;
        if (r < tiles) {
            if (blockIdx.z > 0) return;
            const Scn& S = scn_at<kOne>(B, s_first + blockIdx.x);
            if (S.lds_bins && r * kLdsTile < S.bins.nbins) lds_bins_build(S.bins, r);
            return;
        }
        const int64_t row = (int64_t)blockIdx.z * ((int)gridDim.y - 1 - tiles) + r - tiles;
        const int64_t at = (row * (int)gridDim.x + (int)blockIdx.x) * kChunkWaves + (int)(threadIdx.x >> 6);
        if (at >= B.total_chunks) return;
        const int g = __builtin_amdgcn_readfirstlane((int)at);
        const int sc = kOne ? 0 : find_scenario(B.chunk_off, B.S, g);
        wave_chunk_sum(scn_at<kOne>(B, sc).bins, g - (kOne ? 0 : B.chunk_off[sc]));
        return;
    }
    if (blockIdx.z > 0) return;
    const int sc = s_first + blockIdx.x;
    const Scn& S = scn_at<kOne>(B, sc);
    // the parameters used, in registers: loaded in the first round, not
    // reloaded after the stores below
    const FvParams& p = S.fv;
    FPS_GLOBAL DevState* gst = gmem(p.st);
    const FPS_GLOBAL double* partials = gmem(p.partials);
    FPS_GLOBAL int32_t* wet = gmem(p.wet);
    // partials of a large grid were added by chunks into every kRedTiles-th one
    const int every = p.ntiles > kRedMin ? kRedTiles : 1;
    const int ntiles = (p.ntiles + every - 1) / every, n_inflow = p.n_inflow, inflow_side = p.inflow_side;
    const double dxdy = p.dxdy;
    const float cfl = p.cfl, dt_max = p.dt_max, dn = inflow_side <= 1 ? p.dx : p.dy;
    const bool jmask = p.jmask != nullptr;
    const int na = S.na, nline = S.bar.nline, nchunk = S.bins.nchunk;
    FPS_GLOBAL int32_t* stepped = gmem(S.bins.csum.p);
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x >> 6;
    // The scenario's state words go through LDS: one cooperative load, the
    // serial end-of-step logic on the copy, one cooperative store.  Nothing
    // else touches them while this block runs.  The hydrograph knots stay out
    // of the copy (they do not change): they are loaded into registers, one
    // knot per lane, and the first wave uses them.
    __shared__ DevState sst;
    constexpr int kWords = (int)(sizeof(DevState) / sizeof(uint32_t));
    constexpr int kHyd0 = (int)(offsetof(DevState, hyd_t) / sizeof(uint32_t));
    constexpr int kHyd1 = (int)(offsetof(DevState, step) / sizeof(uint32_t));
    constexpr int kCopy = kHyd0 + kWords - kHyd1;
    static_assert(sizeof(DevState) % sizeof(uint32_t) == 0, "DevState is copied as words");
    static_assert(offsetof(DevState, hyd_q) == offsetof(DevState, hyd_t) + sizeof(double) * kMaxHydro &&
                  offsetof(DevState, step) == offsetof(DevState, hyd_q) + sizeof(double) * kMaxHydro,
                  "the hydrograph knots are one run of words");
    static_assert(kCopy <= kScanThreads && kMaxHydro <= kWave, "one word per thread, one knot per lane");
    // Every load of the block goes out before the first wait: the state words
    // and the hydrograph knots into registers (written to LDS afterwards), and
    // eight flood partials per thread.  The loads are unconditional, at
    // clamped indices, and the values past the end are dropped when summed: a
    // load under a condition makes the compiler wait for it before the
    // lanes that skip it may touch its register.
    const int cw = threadIdx.x < kHyd0 ? (int)threadIdx.x : (int)threadIdx.x - kHyd0 + kHyd1;
    const uint32_t word = ((const FPS_GLOBAL uint32_t*)gst)[threadIdx.x < kCopy ? cw : 0];
    const double hk_t = gst->hyd_t[lane], hk_q = gst->hyd_q[lane];
    // the flood partials summed in tile order
    double m = 0.0, vo = 0.0, vc = 0.0;
    unsigned sm = 0;      // the largest wave speed, as bits
    {
        constexpr int kPU = 8;
        const FPS_GLOBAL Double2* P2 = (const FPS_GLOBAL Double2*)partials;
        Double2 a[kPU], c[kPU];
#pragma unroll
        for (int u = 0; u < kPU; ++u) {
            const int b = threadIdx.x + u * kScanThreads, bc = (b < ntiles ? b : 0) * every;
            a[u] = P2[2 * bc];
            c[u] = P2[2 * bc + 1];
        }
        if (threadIdx.x < kCopy) reinterpret_cast<uint32_t*>(&sst)[cw] = word;
#pragma unroll
        for (int u = 0; u < kPU; ++u) {
            if (threadIdx.x + u * kScanThreads < ntiles) {
                m += a[u].x;
                vo += a[u].y;
                vc += c[u].x;
                sm = max(sm, speed_bits(c[u].y));
            }
        }
        for (int b = threadIdx.x + kPU * kScanThreads; b < ntiles; b += kScanThreads) {
            const FPS_GLOBAL double* q = partials + 4 * (size_t)b * every;
            m += q[0];
            vo += q[1];
            vc += q[2];
            sm = max(sm, speed_bits(q[3]));
        }
    }
    __syncthreads();
    DevState* st = &sst;
    // the chunk scan that follows asks whether this step was one of the scenario
    if (mode == 0 && nchunk > 0 && threadIdx.x == 0) stepped[nchunk] = st->active;
    if (mode == 0 && !st->active) return;     // the whole block: one LDS word
    const bool skipped = mode == 0 && flood_skipped(st);
    if (skipped) {
        m = 0.0;
        vo = 0.0;
        vc = 0.0;
        sm = 0;
    }
    // the pedestrians of this step have read the wetness flags: clear them
    if (threadIdx.x < kWetSlots) wet[kWetStride * threadIdx.x] = 0;
    __shared__ double red[kScanThreads / kWave][3];
    __shared__ unsigned redsm[kScanThreads / kWave];
    m = wave_sum(m);
    vo = wave_sum(vo);
    vc = wave_sum(vc);
    sm = __builtin_bit_cast(unsigned, wave_max_bits(sm));
    if (lane == 0) {
        red[wid][0] = m;
        red[wid][1] = vo;
        red[wid][2] = vc;
        redsm[wid] = sm;
    }
    __syncthreads();
    if (wid == 0) {
        // the serial end of the step, on every lane of the first wave (same
        // values); lane 0 stores
        // lanes 0-2 add one quantity each over the waves, in wave order
        double acc = 0.0;
        if (lane < 3) {
            acc = red[0][lane];
            for (int w = 1; w < kScanThreads / kWave; ++w) acc += red[w][lane];
        }
        const double M = readlane_f64(acc, 0), VO = readlane_f64(acc, 1), VC = readlane_f64(acc, 2);
        const float smax = wave_max_bits(redsm[lane & (kScanThreads / kWave - 1)]);
        double t = st->t, v_out = st->v_out, v_clip = st->v_clip, v_in = st->v_in, mass = st->mass;
        int64_t step = st->step;
        float dt = st->dt, dt_prev = st->dt_prev;
        int cur = st->cur, flood_steps = st->flood_steps, settled = st->settled, any_wet = st->any_wet;
        int status = st->status;
        if (mode == 0) {
            t += (double)dt;
            step += 1;
            dt_prev = dt;
            if (!skipped) {
                v_out += VO;
                v_clip += VC * dxdy;
                v_in += (double)st->inc * (double)n_inflow * dxdy;
                cur ^= 1;
                flood_steps += 1;
                settled = 1;
            }
        }
        if (!skipped) {
            mass = M * dxdy;
            any_wet = !(smax <= 0.0f);
            dt = any_wet && !jmask ? fminf(cfl / smax, dt_max) : dt_max;
        }
        float inc = 0.0f;
        if (inflow_side >= 0)
            inc = (float)(wave_hydro_integral(st->nh, hk_t, hk_q, t, t + (double)dt) / (double)dn);
        if (!isfinite(mass) || !(dt > 0.0f) || !isfinite(dt) || !(smax == smax)) status = FPS_E_NUMERIC;
        if (lane == 0) {
            st->t = t;
            st->step = step;
            st->dt_prev = dt_prev;
            st->v_out = v_out;
            st->v_clip = v_clip;
            st->v_in = v_in;
            st->cur = cur;
            st->flood_steps = flood_steps;
            st->settled = settled;
            st->mass = mass;
            st->any_wet = any_wet;
            st->dt = dt;
            st->inc = inc;
            st->status = status;
            // sandbag write-back: drops of this step applied to the barrier line in order
            if (mode == 0 && na > 0) {
                const int D = st->drops;
                st->drops = 0;
                st->drops_total += D;
                if (!st->done && nline > 0) {
                    const BarrierParams Bb = S.bar;      // by value, read only while a barrier is built
                    int bags = st->bags + D;
                    int cell = st->active_cell, layers = st->layers_done, fin = 0;
                    while (!fin && bags >= Bb.bags_per) {
                        bags -= Bb.bags_per;
                        const float th = layers == Bb.n_layers - 1 ? Bb.t_last : Bb.t_bag;
                        Bb.z[Bb.line[cell]] += th;
                        cell += 1;
                        if (cell == Bb.nline) {
                            cell = 0;
                            layers += 1;
                            if (layers >= Bb.n_layers) fin = 1;
                        }
                    }
                    st->bags = bags;
                    st->active_cell = cell;
                    st->layers_done = layers;
                    st->done = fin;
                }
            }
            if (mode == 0) st->active = !(st->t_end > 0.0) || t < st->t_end;
        }
    }
    __syncthreads();
    if (threadIdx.x < kCopy)
        ((FPS_GLOBAL uint32_t*)gst)[cw] = reinterpret_cast<const uint32_t*>(&sst)[cw];
}

// After the last step of a call: scenarios whose state sits in the scratch
// buffer copy it back to the caller's buffers (grid: blocks x scenarios), and
// the state is in the caller's buffer again.  kCount: the last block of a
// scenario to be done says so (every block has read `cur` before it counts
// itself in, and the count ends at 0), which saves a call of one step a launch
// of 2 us; its grid is small, since the blocks count on one word.  Otherwise a
// launch of its own follows.
template <bool kCount>
__global__ void sync_back_kernel(Batch B)
{
    const FvParams& p = B.scn[blockIdx.y].fv;
    FPS_GLOBAL DevState* st = gmem(p.st);
    if (st->cur == 0) return;
    const int64_t nc = (int64_t)p.nx * p.ny;
    const FPS_GLOBAL float *h = gmem(p.h[1]), *qx = gmem(p.qx[1]), *qy = gmem(p.qy[1]);
    FPS_GLOBAL float *ho = gmem(p.h[0]), *qxo = gmem(p.qx[0]), *qyo = gmem(p.qy[0]);
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < nc;
         k += (int64_t)gridDim.x * blockDim.x) {
        const float a = h[k], b = qx[k], c = qy[k];
        ho[k] = a;
        qxo[k] = b;
        qyo[k] = c;
    }
    if constexpr (kCount) {
        __syncthreads();
        int32_t* count = p.wet + 1;       // between two wetness flags
        if (threadIdx.x == 0 && atomicAdd(count, 1) == (int)gridDim.x - 1) {
            *count = 0;
            st->cur = 0;
        }
    }
}
__global__ void reset_cur_kernel(Batch B)
{
    for (int s = threadIdx.x; s < B.S; s += blockDim.x) B.scn[s].fv.st->cur = 0;
}

// Streaming probe: n_in arrays read and n_out arrays written, 16 bytes a
// lane, grid-stride; out_k = sum of the inputs + k, so every input byte is
// used.  A bandwidth ceiling for kernels that stream SoA fields.
template <int NIN, int NOUT>
__global__ __launch_bounds__(256) void stream_probe_kernel(float* __restrict__ buf, int64_t n4, int64_t stride4)
{
    const float4* in = reinterpret_cast<const float4*>(buf);
    float4* out = reinterpret_cast<float4*>(buf) + NIN * stride4;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4; i += (int64_t)gridDim.x * blockDim.x) {
        float4 a[NIN];
#pragma unroll
        for (int k = 0; k < NIN; ++k) a[k] = in[k * stride4 + i];
        float4 t = a[0];
#pragma unroll
        for (int k = 1; k < NIN; ++k) t = make_float4(t.x + a[k].x, t.y + a[k].y, t.z + a[k].z, t.w + a[k].w);
#pragma unroll
        for (int k = 0; k < NOUT; ++k)
            out[k * stride4 + i] = make_float4(t.x + (float)k, t.y + (float)k, t.z + (float)k, t.w + (float)k);
    }
}

}  // namespace

hipError_t launch_stream_probe(float* buf, int64_t n, int64_t stride, int n_in, int n_out, int blocks, hipStream_t s)
{
    const int64_t n4 = n / 4, s4 = stride / 4;
    const dim3 grid(blocks), block(256);
    if (n_in == 1 && n_out == 1) hipLaunchKernelGGL((stream_probe_kernel<1, 1>), grid, block, 0, s, buf, n4, s4);
    else if (n_in == 5 && n_out == 3) hipLaunchKernelGGL((stream_probe_kernel<5, 3>), grid, block, 0, s, buf, n4, s4);
    else if (n_in == 4 && n_out == 3) hipLaunchKernelGGL((stream_probe_kernel<4, 3>), grid, block, 0, s, buf, n4, s4);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

int fv_tiles2(int nx, int ny, int H)
{
    const int64_t nsx = (nx + kStrip2 - 1) / kStrip2;
    return (int)(nsx * ((ny + H - 1) / H));
}

int fv_strip(bool order2) { return order2 ? kStrip2 : kStrip; }

int fv_tiles(int nx, int ny, int H)
{
    const int64_t nsx = (nx + kStrip - 1) / kStrip;
    return (int)(nsx * ((ny + H - 1) / H));
}

int fv_blocks_for_tiles(int64_t tiles)
{
    const int64_t blocks = (tiles + kFvBlock / kWave - 1) / (kFvBlock / kWave);
    return (int)((blocks + 7) / 8 * 8);    // a multiple of the 8 XCDs
}

hipError_t launch_fv(const Batch& b, hipStream_t s)
{
    if (b.fv_blocks > 0 && b.order2) {
        const dim3 grid(b.fv_blocks), block(kFvBlock);
        const auto go = [&](auto one, auto hll) {
            constexpr bool kOne = decltype(one)::value, kHll = decltype(hll)::value;
            hipLaunchKernelGGL((fv2_stage_kernel<kOne, kHll, false, 1>), grid, block, 0, s, b);
            if (b.people) hipLaunchKernelGGL((fv2_stage_kernel<kOne, kHll, true, 2>), grid, block, 0, s, b);
            else hipLaunchKernelGGL((fv2_stage_kernel<kOne, kHll, false, 2>), grid, block, 0, s, b);
        };
        if (b.S == 1) {
            if (b.hll) go(std::true_type{}, std::true_type{});
            else go(std::true_type{}, std::false_type{});
        } else {
            if (b.hll) go(std::false_type{}, std::true_type{});
            else go(std::false_type{}, std::false_type{});
        }
        return hipGetLastError();
    }
    if (b.fv_blocks > 0) {
        const dim3 grid(b.fv_blocks), block(kFvBlock);
        const auto go = [&](auto one, auto hll, auto people) {
            hipLaunchKernelGGL((fv_step_kernel<decltype(one)::value, decltype(hll)::value, decltype(people)::value>),
                               grid, block, 0, s, b);
        };
        const auto with_people = [&](auto one, auto hll) {
            if (b.people) go(one, hll, std::true_type{});
            else go(one, hll, std::false_type{});
        };
        if (b.S == 1) {
            if (b.hll) with_people(std::true_type{}, std::true_type{});
            else with_people(std::true_type{}, std::false_type{});
        } else {
            if (b.hll) with_people(std::false_type{}, std::true_type{});
            else with_people(std::false_type{}, std::false_type{});
        }
    }
    return hipGetLastError();
}

hipError_t launch_fv_scan(const Batch& b, int scenario, int ntiles, hipStream_t s)
{
    hipLaunchKernelGGL(fv_scan_kernel, dim3(ntiles), dim3(kFvBlock), 0, s, b, scenario);
    return hipGetLastError();
}

hipError_t launch_fv_reduce(const Batch& b, int s_first, int count, hipStream_t s)
{
    if (b.red_chunks > 0)
        hipLaunchKernelGGL(fv_reduce_kernel, dim3(b.red_chunks, count), dim3(kFvBlock), 0, s, b, s_first);
    return hipGetLastError();
}

// Rows per wave before any tuning: the longest march (fewest halo rows and
// partials) that still leaves enough waves to fill the chip and hide its loads;
// the fewer rows, the more a halving costs, so the fewer waves will do.
// Measured, a whole step (us) at 1, 2, 4, 8, 16 rows, and the waves the rule asks
// of a height, between the sizes on either side of the line:
//   400^2        11.9  12.5  13.1  15.6  20.6      1 (1,400 waves at 2)
//   440^2        13.0  12.7  13.1  15.7  20.6      2 (1,760)                   2 rows: 1,600
//   480^2        13.1  12.7  13.0  15.7  20.7      2
//   512^2        13.3  13.2  14.2  15.5  20.6      2
//   620^2        15.1  14.2  14.3  15.6  20.8      2 (1,550 at 4)
//   768^2        20.6  15.5  15.9  17.6  20.9      2 (2,496)
//   1811 x 364   23.0  18.3  17.7  19.7  22.7      4 (2,730)                   4 rows: 2,560
//   860^2        22.0  16.8  16.1  17.9  20.9      4 (3,010)
//   1024^2       25.3  23.0  19.6  21.2  24.9      4 (2,176 at 8)
//   1200^2       29.3  26.1  22.3  22.0  25.6      4 (3,000)
//   1400^2       33.8  29.5  26.0  25.8  26.2      4 (4,025)                   8 rows: 4,096
//   1600^2       39.2  33.9  33.5  31.6  31.7      8 (5,200; 2,600 at 16)
//   2048^2       54.6  45.2  42.6  43.7  42.7      8 (4,352; second order 84.7, 80.6, 81.8)
//   2400^2       68.4  55.2  51.6  52.2  48.7     16 (5,850)                  16 rows: 5,000
//   3000^2      102.6  80.4  75.2  72.2  70.3     16 (9,212)
// and the flood launch of 6 x 2048^2: 365, 273, 223, 200, 193 (201 at 32).  Beyond
// 8,192 waves of one grid the partials take a launch more (fv_reduce_kernel).
// The waves of all members of a launch count, and all get one height: a mix of
// heights gives the XCDs, each with a run of as many waves, unequal work (four
// grids each of 1024, 512, 256 and 716 a side 64.6 us a step at 16 rows, 71.0 with
// at least 1,024 waves a member).  But members stop, or are dry, and the others
// then march alone: an average member must keep 512 waves, half a wave a SIMD,
// beyond four rows.  That mix gets 8 rows (65.5 us), and its members left alone take
// 60.0, 29.8, 21.0 and 41.4 us, where 16 rows took 59.2, 33.2, 22.2 and 47.8; 32 x
// 256^2 gets 4: 31.8 us, alone 16.9 (32.1 and 19.1 at 8).
int fv_rows_per_wave(const fps_grid_desc* d, int S)
{
    for (int H = 16; H > 1; H >>= 1) {
        const int64_t enough = H >= 16 ? 5000 : H >= 8 ? 4096 : H >= 4 ? 2560 : 1600;
        int64_t tiles = 0;
        for (int k = 0; k < S; ++k) tiles += fv_tiles(d[k].nx, d[k].ny, H);
        if (tiles >= enough && (H <= 4 || tiles >= (int64_t)512 * S)) return H;
    }
    return 1;
}

hipError_t prepare_finalize(int lds_bytes)
{
    static int granted = 0;     // the attribute is per kernel: raise it once to the largest size
    if (lds_bytes <= granted) return hipSuccess;
    hipError_t e = hipFuncSetAttribute((const void*)finalize_kernel<true>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
    if (e == hipSuccess)
        e = hipFuncSetAttribute((const void*)finalize_kernel<false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                lds_bytes);
    if (e == hipSuccess) granted = lds_bytes;
    return e;
}

hipError_t launch_finalize(const Batch& b, int mode, int s_first, int count, hipStream_t s)
{
    // rows of blocks: the states; after a step, where there are such, the LDS
    // binnings and then the chunks (the kind by the row: a bound from the
    // arguments, read first, cost the state update 0.3 us)
    const int blocks = mode == 0 ? (b.total_chunks + kChunkWaves - 1) / kChunkWaves : 0;
    const int chunks = (blocks + count - 1) / count;
    const int tiles = mode == 0 ? b.fin_tiles : 0;
    constexpr int kRows = 32768;      // rows of chunks a layer (a grid has at most 65,535)
    const dim3 grid(count, 1 + tiles + std::min(chunks, kRows), std::max((chunks + kRows - 1) / kRows, 1));
    const int lds = mode == 0 ? b.fin_lds_bytes : 0;
    if (b.S == 1) hipLaunchKernelGGL(finalize_kernel<true>, grid, dim3(kScanThreads), lds, s, b, mode, s_first);
    else hipLaunchKernelGGL(finalize_kernel<false>, grid, dim3(kScanThreads), lds, s, b, mode, s_first);
    return hipGetLastError();
}

hipError_t launch_sync_back(const Batch& b, int64_t max_cells, hipStream_t s)
{
    const int64_t need = std::max<int64_t>((max_cells + 255) / 256, 1);
    if (need <= kSyncCount) {
        hipLaunchKernelGGL(sync_back_kernel<true>, dim3((unsigned)need, b.S), dim3(256), 0, s, b);
    } else {
        hipLaunchKernelGGL(sync_back_kernel<false>, dim3((unsigned)std::min<int64_t>(need, 2048), b.S), dim3(256), 0, s, b);
        hipLaunchKernelGGL(reset_cur_kernel, dim3(1), dim3(256), 0, s, b);
    }
    return hipGetLastError();
}

}  // namespace fps
