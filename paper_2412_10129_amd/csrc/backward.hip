// Matched backprojectors: the exact transposes A^T of the Siddon and the
// interpolated forward projectors (needed by the Krylov methods of section
// 2.2.1, and as the gradient of the autograd operator).
//
// Voxel-driven by bricks: a workgroup owns one brick of 16 x 16 x BZ output
// voxels and accumulates it over every view of the call; each voxel has one writer
// in global memory and no global atomics are used.  Views are taken in groups
// of GV.  For each view the brick's detector footprint (bounding box of its
// projected corners) is cut into batches of 64 pixels, and the workgroup's
// waves take the group's batches in turn: every lane re-traces one pixel's ray
// through the brick with the forward kernel's FP32 arithmetic (shared helpers
// in ctmi_internal.h), keeps it in registers and walks it to its end.  A
// batch belongs to one view, so the view's geometry sits in scalar registers,
// and between a group's scale (below) and its flush the waves run free of
// barriers.
//
// Accumulation is in fixed point in LDS: FP32 LDS atomics are serialised
// on gfx950 (192 clocks per wave instruction measured) while integer LDS
// atomics on scattered addresses take 7.5 (32-bit) or 12.5 (64-bit) clocks.
// The scale is chosen per group of views so that everything the group can add
// to one cell fits an int32 (group_scale); integer addition is associative,
// so the result is bit-reproducible whatever the order of the atomics.  A
// group ends with a flush: the cells' exact integer sums go, scaled by a power
// of two, into per-thread FP32 registers in a fixed order.
//
// LDS atomics bound the interpolated adjoint and weigh on the Siddon one, so
// the order of a footprint's pixels over the lanes is chosen for them: of 16
// lanes (the atomic unit's step) no two should meet in a bank, while a wave's
// rays should be of similar length.  Footprint columns are taken in narrow
// groups and, inside a group, rows in strides of about one voxel (pixel_order).
//
// Measured against the form this replaced (rounds of 256 or 512 rays recorded
// in an LDS table, cut into items and numbered by block scans, with a scale and
// a flush per round; the interpolated one with eight 32-bit atomics per
// sample): interpolated, 512^3 x 120 views of 1024 x 768: 152 -> 100 ms (83 -> 55
// clocks of a CU per 64 samples; at 720 views LDS is at work 78 % of the time, with 1.36
// vector instructions per clock of the 1 to 1.6 that its mix allows); Siddon, 256^3 x
// 90 views of 512 x 512: 13.1 -> 7.6 ms (512^3 x 720: 1.31 vector instructions per
// clock, LDS at work 38 %).
#include "adjoint_bricks.h"

namespace ctmi {

namespace {

typedef unsigned long long u64;

// A brick's detector footprint in one view, and what bounds its sums.
//
// Footprint: foot_pixels of the box [lo, hi] (voxel-centre coordinates, x, y, z).
//
// su, sv: bound on the pixels that the projection of a point moves by when
// the point moves by at most one voxel along every axis, anywhere in the
// box: with U, V, W the projection's numerators and denominator,
// u(p) - u(c) = (U(p - c) - u(c) W(p - c)) / W(p), the offset's terms without
// their constants, so |du| <= sum_a (|MU_a - um MW_a| + hu |MW_a|) / Wmin for
// u(c) within hu of um.
//
// along: the largest |d| / |d_a| over the points of the box, in mm per voxel
// of the best axis a (d the direction from the source): a ray spends at most
// `along` mm between two planes of that axis one voxel apart.  Infinite when
// every axis has the source between its faces.
struct Foot {
    int u0, u1, v0, v1;
    float su, sv, along;
};

__device__ __forceinline__ Foot footprint(const ViewGeo& g, const float lo[3], const float hi[3], const DetDims& det,
                                          const VolDims& v)
{
    float umin = CTMI_INF, umax = -CTMI_INF, vmin = CTMI_INF, vmax = -CTMI_INF;
    float xmin = CTMI_INF, xmax = -CTMI_INF, ymin = CTMI_INF, ymax = -CTMI_INF, wmin = CTMI_INF, lmax = 0.0f;
    // the sources's position in voxel-centre coordinates (the table's are voxel-cell)
    const float S[3] = {g.S[0] - 0.5f, g.S[1] - 0.5f, g.S[2] - 0.5f};
    const float h[3] = {v.hx, v.hy, v.hz};
    auto project = [&](const float c[3], float& u, float& w, float& W) {
        W = __builtin_fmaf(g.MW[0], c[0], __builtin_fmaf(g.MW[1], c[1], __builtin_fmaf(g.MW[2], c[2], g.MW[3])));
        const float U = __builtin_fmaf(g.MU[0], c[0], __builtin_fmaf(g.MU[1], c[1], __builtin_fmaf(g.MU[2], c[2], g.MU[3])));
        const float V = __builtin_fmaf(g.MV[0], c[0], __builtin_fmaf(g.MV[1], c[1], __builtin_fmaf(g.MV[2], c[2], g.MV[3])));
        const float rw = 1.0f / W;
        u = U * rw;
        w = V * rw;
    };
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const float c[3] = {(q & 1) ? hi[0] : lo[0], (q & 2) ? hi[1] : lo[1], (q & 4) ? hi[2] : lo[2]};
        float pu, pv, W;
        project(c, pu, pv, W);
        umin = fminf(umin, pu);
        umax = fmaxf(umax, pu);
        vmin = fminf(vmin, pv);
        vmax = fmaxf(vmax, pv);
        // the box grown by one voxel, for the bounds: any point that adds to
        // one of the brick's cells lies in it
        const float e[3] = {c[0] + ((q & 1) ? 1.0f : -1.0f), c[1] + ((q & 2) ? 1.0f : -1.0f),
                            c[2] + ((q & 4) ? 1.0f : -1.0f)};
        project(e, pu, pv, W);
        xmin = fminf(xmin, pu);
        xmax = fmaxf(xmax, pu);
        ymin = fminf(ymin, pv);
        ymax = fmaxf(ymax, pv);
        wmin = fminf(wmin, W);
        float l2 = 0.0f;
#pragma unroll
        for (int a = 0; a < 3; ++a) l2 = __builtin_fmaf((e[a] - S[a]) * h[a], (e[a] - S[a]) * h[a], l2);
        lmax = fmaxf(lmax, l2);
    }
    Foot f;
    const float um = 0.5f * (xmin + xmax), hu = 0.5f * (xmax - xmin), ym = 0.5f * (ymin + ymax), hv = 0.5f * (ymax - ymin);
    f.su = f.sv = 0.0f;
    float da = 0.0f;   // the best axis's smallest voxels of travel per voxel-sized unit, d_a in voxels
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        f.su += fabsf(__builtin_fmaf(-um, g.MW[a], g.MU[a])) + hu * fabsf(g.MW[a]);
        f.sv += fabsf(__builtin_fmaf(-ym, g.MW[a], g.MV[a])) + hv * fabsf(g.MW[a]);
        // distance from the source to the grown box along axis a (0 when between its faces)
        da = fmaxf(da, fmaxf(lo[a] - 1.0f - S[a], S[a] - hi[a] - 1.0f));
    }
    const float rw = 1.0f / wmin;
    f.su = wmin > 0.0f ? f.su * rw * 1.001f : CTMI_INF;
    f.sv = wmin > 0.0f ? f.sv * rw * 1.001f : CTMI_INF;
    f.along = da > 0.0f ? __builtin_sqrtf(lmax) / da * 1.001f : CTMI_INF;
    foot_pixels(umin, umax, vmin, vmax, det, f.u0, f.u1, f.v0, f.v1);
    return f;
}

// A group of views: the footprints, the batches of each view's pixels
// (prefix sums in pre) and the order of the pixels over the lanes.
template <int GV>
struct GroupLds {
    int u0[GV], v0[GV], w[GV], h[GV];
    int ku[GV], kv[GV], rk[GV], hp[GV], wide[GV], pre[GV + 1];
    float rcol[GV], rrow[GV];   // reciprocals of ku kv hp (pixels per column group) and hp
    float most[GV], f[GV];      // rays on one cell times the most each adds per unit y; the latter
    float red[2][16];           // per wave: largest |y|, sum of |y|
};

// Order of a view's footprint pixels: columns in groups of ku, rows padded to
// a multiple of kv; inside a group the pixel's index runs over (row class
// a < kv, column b < ku, row): pixel (u, v) = (group ku + b, a + kv r).  ku and
// kv are the pixels per voxel (rounded up past 0.1), so consecutive lanes hold
// rays of one column about one voxel apart: rays closer than that meet in one
// cell, whose atomics serialise, and rays of one column have paths of similar
// length.  A bank model of the atomics (16 lanes per step, 64 banks) gives 44
// clocks per 64 samples at 1.5 pixels per voxel, 69 for plain column order, 68
// for row order, with 79 % of the lanes at work (76 % for groups of 2 ku).
// Where a column's rows end within 16 lanes, a step of the interpolated adjoint's
// atomics takes in the next column too, whose rays share its cells: there a group
// is 2 ku columns in the order 0, ku, 1, ku + 1, ... (`wide`; 245x112x112 x 46
// views 2.21 -> 2.06 ms, 201x84x178 x 46 0.80 -> 0.73, 512^3 x 120 102.0 -> 100.0).
// Not for three row classes and more, whose ku columns fill a wave already
// (117x203x181 x 37: 2.73 -> 2.76 ms), nor for Siddon, whose walks leave a cell
// at every step (259x78x51 x 46: 612 -> 635 us).
// Where no more than five rows follow each other it is 4 ku columns (0, ku, 2 ku, 3 ku,
// 1, ...), so that a step's columns are a voxel apart again: 128^3 x 36 views on pixels of
// 4 x 0.5 voxels 607 -> 500 us, 3 x 0.7 487 -> 452.
constexpr float KMAX = 32.0f;   // most columns and row classes (of 8, rays meet in cells beyond: 96^3 on 8 pixels per voxel 35.1 -> 26.4 ms)
template <bool SIDDON, bool PACK, int GV>
__device__ __forceinline__ void pixel_order(GroupLds<GV>& G, int g, float pu, float pv)
{
    const int w = G.w[g], h = G.h[g];
    const int ku = max((int)__builtin_ceilf(fminf(pu, KMAX) - 0.1f), 1);
    const int kv = max((int)__builtin_ceilf(fminf(pv, KMAX) - 0.1f), 1);
    const int hp = (h + kv - 1) / kv, wide = !SIDDON && kv <= 2 && hp <= 16 ? (hp <= 5 ? 4 : 2) : 1;
    const int per = wide * ku * kv * hp;
    G.ku[g] = ku;
    G.wide[g] = wide;
    G.kv[g] = kv;
    G.rk[g] = (65536 + wide * ku - 1) / (wide * ku);   // ceil(2^16 / n): i / n for i (n - 1) < 2^16 (i < 1024, n <= 32, or i < 256, n <= 128)
    G.hp[g] = hp;
    G.rcol[g] = 1.0f / (float)per;
    G.rrow[g] = 1.0f / (float)hp;
    const int n = (w + wide * ku - 1) / (wide * ku) * per;
    G.pre[g + 1] = PACK ? n : (n + 63) / 64;
}

// Lane `lane` of batch bt: its view g of the group and its pixel; false when it falls on
// padding.  Batches come in order (g starts at 0 and is kept by the caller); with
// PACK a batch runs over the views' ends.  The quotients come from FP32 reciprocals:
// floor((i + 1/2) r), r = fl(1/n), is i div n for every i < 2^22.  (In a footprint of
// more pixels than that, of a voxel that covers thousands, both are corrected by an
// exact remainder step.)
template <bool SIDDON, bool PACK, int GV>
__device__ __forceinline__ bool group_pixel(const GroupLds<GV>& G, int bt, int lane, int& g, int& iu, int& iv)
{
    // without PACK the view and its layout are the same in every lane: scalar registers
    auto get = [&](int v) { return PACK ? v : __builtin_amdgcn_readfirstlane(v); };
    int p;
    bool in = true;
    if (PACK) {
        p = 64 * bt + lane;
        in = p < G.pre[GV];
        g = 0;
#pragma unroll
        for (int st = GV / 2; st > 0; st >>= 1) g += p >= G.pre[g + st] ? st : 0;
        p -= G.pre[g];
    } else {
        while (bt >= get(G.pre[g + 1])) ++g;
        p = 64 * (bt - get(G.pre[g])) + lane;
    }
    const int ku = get(G.ku[g]), kv = get(G.kv[g]), wide = SIDDON ? 1 : get(G.wide[g]), hp = get(G.hp[g]);
    const int per = wide * ku * kv * hp;
    const bool large = G.pre[g + 1] - G.pre[g] > (PACK ? 1 << 22 : 1 << 16);
    int cg = (int)(((float)p + 0.5f) * G.rcol[g]);
    if (large) {
        const int rem = p - cg * per;
        cg += rem >= per ? 1 : (rem < 0 ? -1 : 0);
    }
    int r = p - cg * per;
    int ab = (int)(((float)r + 0.5f) * G.rrow[g]);
    if (large) {
        const int rem = r - ab * hp;
        ab += rem >= hp ? 1 : (rem < 0 ? -1 : 0);
    }
    r -= ab * hp;
    const int a = (ab * G.rk[g]) >> 16;
    const int b = ab - a * wide * ku;
    const int lw = wide >> 1;   // log2(wide)
    const int du = cg * wide * ku + (b >> lw) + (b & (wide - 1)) * ku, dv = a + kv * r;
    iu = G.u0[g] + du;
    iv = G.v0[g] + dv;
    return in && du < G.w[g] && dv < G.h[g];
}

// Prepares the group of views [k, k + n): footprints of the box [lo, hi],
// batches, and the group's fixed-point exponents.  Returns the number of
// batches, 0 when the group adds nothing.
//
// Values far above the rest (more than 8 times the footprints' mean |y|: the
// weighted residuals of rays that graze the volume, hot pixels) form a second
// class that the group adds in a second pass at a unit of its own, so that they
// do not coarsen the unit of all others: ex[0] is the exponent of |y| <= cut,
// ex[1] that of |y| > cut; without such values cut is infinite and one pass
// does.
//
// One cell's sum over the group is at most F sum |y| (F the most one ray adds
// to one cell per unit y, over the group's views) and at most max |y| times
// the sum over views of the rays that can reach one cell times that view's
// f; the smaller of the two is scaled to 2^30.  A ray reaches a cell when its
// pixel centre lies in the projection of the cell's support, a box of half
// width `reach` voxels (1/2 for a Siddon cell, 1 for a trilinear tent): at
// most floor(2 reach su) + 1 columns by floor(2 reach sv) + 1 rows, and no
// more than the footprint holds.  It adds at most one chord (Siddon), or the
// samples' tent weights along its best axis, whose positions are delta =
// ds / along voxels apart: sum tent <= 1 / delta + delta / 4 for delta <= 1,
// and never more than fmax (the plan's bound for any direction).  While a cell
// has no more than some thousand rays (N below 2^12 F), that second bound is
// scaled to 2^31 less 1 %: 2.1e7 units are then left for the roundings of its
// terms, half a unit each.
template <bool SIDDON, bool PACK, int NW, int GV>
__device__ __forceinline__ int group_scale(GroupLds<GV>& G, const ViewGeo* __restrict__ tab,
                                           const float* __restrict__ proj, int view0, int k, int n, const float lo[3],
                                           const float hi[3], const DetDims& det, const VolDims& v, float ds,
                                           float fmax_, int (&ex)[2], float& cut)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid < GV) {
        const int g = tid;
        G.w[g] = G.h[g] = 0;
        G.pre[g + 1] = 0;
        G.most[g] = G.f[g] = 0.0f;
        if (g < n) {
            const Foot f = footprint(tab[view0 + k + g], lo, hi, det, v);
            if (f.u0 <= f.u1 && f.v0 <= f.v1) {
                G.u0[g] = f.u0;
                G.v0[g] = f.v0;
                G.w[g] = f.u1 - f.u0 + 1;
                G.h[g] = f.v1 - f.v0 + 1;
                const float reach = SIDDON ? 1.0f : 2.0f;   // twice the support's half width
                const float cu = fminf(__builtin_floorf(reach * f.su + 0.02f) + 1.0f, (float)G.w[g]);
                const float cv = fminf(__builtin_floorf(reach * f.sv + 0.02f) + 1.0f, (float)G.h[g]);
                float one = fmax_;
                if (SIDDON) {
                    one = fminf(one, f.along);
                } else {
                    const float rd = f.along / ds;   // 1 / delta
                    if (rd >= 1.0f) one = fminf(one, ds * (rd + 0.25f) * 1.001f);
                }
                G.f[g] = one;
                G.most[g] = cu * cv * one;
                pixel_order<SIDDON, PACK>(G, g, f.su, f.sv);
            }
        }
    }
    __syncthreads();
    // largest |y| and sum of |y| over the footprints (a row at a time; two
    // rows where a row fills half a wave or less)
    float ym = 0.0f, ys = 0.0f;
    for (int g = 0; g < n; ++g) {
        const int w = G.w[g], h = G.h[g];
        const float* pk = proj + ((int64_t)(k + g) * det.nv + G.v0[g]) * det.nu + G.u0[g];
        const int two = w <= 32 ? 1 : 0;
        const int r0 = two ? 2 * wave + (lane >> 5) : wave, l = two ? (lane & 31) : lane;
        for (int r = r0; r < h; r += NW << two)
            for (int u = l; u < w; u += 64) {
                const float y = fabsf(finite_or_zero(pk[(int64_t)r * det.nu + u]));
                ym = fmaxf(ym, y);
                ys += y;
            }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        ym = fmaxf(ym, __shfl_xor(ym, o, 64));
        ys += __shfl_xor(ys, o, 64);
    }
    if (lane == 0) {
        G.red[0][wave] = ym;
        G.red[1][wave] = ys;
    }
    if (tid == 0) {
        G.pre[0] = 0;
        for (int g = 0; g < GV; ++g) G.pre[g + 1] += G.pre[g];
    }
    __syncthreads();
    ym = ys = 0.0f;
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        ym = fmaxf(ym, G.red[0][i]);
        ys += G.red[1][i];
    }
    float F = 0.0f, N = 0.0f;
    float npx = 0.0f;   // (a view holds < 2^28 pixels; a group may hold more than an int32)
#pragma unroll
    for (int g = 0; g < GV; ++g) {
        F = fmaxf(F, G.f[g]);
        N += G.most[g];
        npx += (float)(G.w[g] * G.h[g]);
    }
    if (!(ym > 0.0f)) return 0;
    const int bit = N < 0x1p12f * F ? 1 : 0;
    if (bit) N *= 1.01f;
    ex[0] = ex[1] = fixed_exp(N, ym) + bit;
    if (ys <= 0x1.fffffep127f) ex[0] = ex[1] = max(ex[0], fixed_exp(F, ys));
    cut = ys / npx * 8.0f;
    if (cut < ym && cut > 0.0f) ex[0] = max(ex[0], fixed_exp(N, cut) + bit);
    else cut = CTMI_INF;
    const int last = __builtin_amdgcn_readfirstlane(G.pre[GV]);
    return PACK ? (last + 63) / 64 : last;
}

template <typename T>
__device__ __forceinline__ T pick3(int i, T v0, T v1, T v2)
{
    return i == 0 ? v0 : (i == 1 ? v1 : v2);
}

__device__ __forceinline__ SiddonAxis pick_axis(int i, const SiddonAxis& x, const SiddonAxis& y, const SiddonAxis& z)
{
    SiddonAxis r;
    r.inv = pick3(i, x.inv, y.inv, z.inv);
    r.c = pick3(i, x.c, y.c, z.c);
    r.step = pick3(i, x.step, y.step, z.step);
    return r;
}

// Cell pitches of the Siddon accumulator: 17 per row, 279 per plane keep the
// lanes of one step in different banks for rays one voxel apart in z (a plane
// of 256 would put them all in one).
constexpr int SPX = BX + 1, SPXY = SPX * BY + 7;

__device__ __forceinline__ unsigned lds_address(const int* p)
{
    return (unsigned)(uintptr_t)(__attribute__((address_space(3))) const char*)p;
}

// add round(q) to the cell at LDS address o 2^149
__device__ __forceinline__ void add_at(float o, float q)
{
    typedef __attribute__((address_space(3))) int lds_int;
    __hip_atomic_fetch_add((lds_int*)(uintptr_t)__float_as_uint(o), round_int(q), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_WORKGROUP);
}

template <int BZ, int NW, int GV, int WPE, bool PACK>
__global__ void __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(WPE, 8)))
k_backward_siddon(const float* __restrict__ proj, float* __restrict__ vol, const ViewGeo* __restrict__ tab,
                  const ViewGeo64* __restrict__ tab64, int view0, int nviews, VolDims v, DetDims det, BrickMap m,
                  float beta, float cmax)
{
    constexpr int T = 64 * NW, OWN = BX * BY * BZ / T;
    __shared__ int acc[SPXY * BZ];
    __shared__ GroupLds<GV> G;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    for (int i = tid; i < SPXY * BZ; i += T) acc[i] = 0;
    float own[OWN];
#pragma unroll
    for (int i = 0; i < OWN; ++i) own[i] = 0.0f;
    int bx, by, bz;
    brick_origin(m, (int)blockIdx.x, bx, by, bz);
    const int x0 = bx * BX, y0 = by * BY, z0 = bz * BZ;
    const int x1 = min(x0 + BX, v.nx), y1 = min(y0 + BY, v.ny), z1 = min(z0 + BZ, v.nz);
    const float lo[3] = {x0 - 0.5f, y0 - 0.5f, z0 - 0.5f};   // cell box in voxel-centre coordinates
    const float hi[3] = {x1 - 0.5f, y1 - 0.5f, z1 - 0.5f};

    for (int k = 0; k < nviews; k += GV) {
        int exs[2] = {0, 0};
        float cut = CTMI_INF;
        const int nbat = group_scale<true, PACK, NW, GV>(G, tab, proj, view0, k, min(GV, nviews - k), lo, hi, det, v, 0.0f,
                                                   cmax, exs, cut);
        for (int cls = 0; cls < (cut < CTMI_INF ? 2 : 1); ++cls) {
        const int ex = exs[cls];
        int gv = 0;
        for (int bt = wave; bt < nbat; bt += NW) {
            int iu, iv;
            const bool in = group_pixel<true, PACK>(G, bt, lane, gv, iu, iv);
            float y = 0.0f;
            if (in) y = finite_or_zero(proj[((int64_t)(k + gv) * det.nv + iv) * det.nu + iu]);
            if (y == 0.0f || (fabsf(y) > cut) != (cls != 0)) continue;
            float S[3], d[3], amin, amax;
            siddon_ray(tab64[view0 + k + gv], iu, iv, v, S, d, amin, amax);
            const SiddonAxis ax = siddon_axis(S[0], d[0]), ay = siddon_axis(S[1], d[1]), az = siddon_axis(S[2], d[2]);
            bool hit = slab_clip(ax, S[0], (float)x0, (float)x1, amin, amax);
            hit &= slab_clip(ay, S[1], (float)y0, (float)y1, amin, amax);
            hit &= slab_clip(az, S[2], (float)z0, (float)z1, amin, amax);
            if (!hit || !(amin < amax)) continue;
            // the ray's dominant axis (largest |d|, never parallel to its
            // planes) and the two others (b, c); selected by value so nothing
            // is indexed at run time
            const int dom = (fabsf(d[0]) >= fabsf(d[1]) && fabsf(d[0]) >= fabsf(d[2])) ? 0
                            : (fabsf(d[1]) >= fabsf(d[2]) ? 1 : 2);
            const int b = dom == 0 ? 1 : 0, c = dom == 2 ? 1 : 2;
            const float Dd = pick3(dom, d[0], d[1], d[2]), Db = pick3(b, d[0], d[1], d[2]), Dc = pick3(c, d[0], d[1], d[2]);
            // scaled before the length factor: |y 2^e| <= 2^30 / chord
            const float yl = __builtin_ldexpf(y, ex) * world_length(d, v);
            if (fabsf(Db) <= 0.99f * fabsf(Dd) && fabsf(Dc) <= 0.99f * fabsf(Dd)) {
                // layer walk: within one dominant-axis cell the ray crosses at
                // most one plane of b and one of c (it runs below 0.99 along
                // both), so the cell's at most three segments follow from the
                // two next crossing parameters (the forward kernel's form)
                const SiddonAxis A = pick_axis(dom, ax, ay, az), B = pick_axis(b, ax, ay, az), C = pick_axis(c, ax, ay, az);
                const float Sd = pick3(dom, S[0], S[1], S[2]);
                const int lod = pick3(dom, x0, y0, z0), hid = pick3(dom, x1, y1, z1);
                // dominant-axis cells from entry to exit
                const int c0 = entry_cell(Sd, Dd, amin, A.step, lod, hid);
                const int c1 = entry_cell(Sd, -Dd, -amax, -A.step, lod, hid);
                const int ob = pick3(b, x0, y0, z0), oc = pick3(c, x0, y0, z0);
                const int ib = ordered_cell(B, pick3(b, S[0], S[1], S[2]), Db, amin, ob, pick3(b, x1, y1, z1));
                const int ic = ordered_cell(C, pick3(c, S[0], S[1], S[2]), Dc, amin, oc, pick3(c, x1, y1, z1));
                float qb = (float)(ib + (B.step > 0)), qc = (float)(ic + (C.step > 0));
                // a parallel axis has inv = 0 and c = inf: its crossings stay at inf
                float anb = __builtin_fmaf(qb, B.inv, B.c), anc = __builtin_fmaf(qc, C.inv, C.c);
                // The cell's LDS address is kept in FP32 as a multiple of 2^-149 (a
                // denormal has its integer as bits; exact), so that a crossing
                // moves it by a fused multiply-add with the axis' step.  No
                // crossing lies before acur (ordered_cell), so the segments
                // need no lower bound.  Empty second and third ones are added too (VALU bounds the walk,
                // and a test costs more than the LDS atomic of a zero): 256^3 x 90
                // views on 512^2 8.25 ms with integer offsets and tests, 7.98 with
                // the tests, 7.68 so.
                const int pa = pick3(dom, 4, 4 * SPX, 4 * SPXY), pb = b == 0 ? 4 : 4 * SPX, pc = c == 1 ? 4 * SPX : 4 * SPXY;
                const float DB = __int_as_float(pb), DC = __int_as_float(pc);
                const float DA = A.step > 0 ? __int_as_float(pa) : -__int_as_float(pa);
                float o = __int_as_float((int)lds_address(acc) + (c0 - lod) * pa + (ib - ob) * pb + (ic - oc) * pc);
                float qa = (float)(c0 + (A.step > 0));   // exit plane of the current layer
                const float fa = (float)A.step, fb = (float)B.step, fc = (float)C.step;
                float acur = amin;
                for (int l = (c1 - c0) * A.step; l >= 0; --l) {
                    const float ae = __builtin_amdgcn_fmed3f(__builtin_fmaf(qa, A.inv, A.c), acur, amax);
                    const bool bfirst = anb <= anc;
                    const float t1 = fminf(fminf(anb, anc), ae), t2 = fminf(bfirst ? anc : anb, ae);
                    const float gb = anb < ae ? fb : 0.0f, gc = anc < ae ? fc : 0.0f;
                    const float ob1 = __builtin_fmaf(gb, DB, o), oc1 = __builtin_fmaf(gc, DC, o);
                    const float o2 = __builtin_fmaf(gc, DC, ob1);
                    const float s1 = t2 - t1, s2 = ae - t2;
                    add_at(o, (t1 - acur) * yl);
                    add_at(bfirst ? ob1 : oc1, s1 * yl);
                    add_at(o2, s2 * yl);
                    acur = ae;
                    o = o2 + DA;
                    qa += fa;
                    qb += gb;
                    qc += gc;
                    anb = __builtin_fmaf(qb, B.inv, B.c);
                    anc = __builtin_fmaf(qc, C.inv, C.c);
                }
            } else {
                // a ray as steep along b or c as along its dominant axis (to 1 %)
                // may cross two planes of one axis in a layer: plane-by-plane walk
                int ix = ordered_cell(ax, S[0], d[0], amin, x0, x1);
                int iy = ordered_cell(ay, S[1], d[1], amin, y0, y1);
                int iz = ordered_cell(az, S[2], d[2], amin, z0, z1);
                float qx = (float)(ix + (ax.step > 0)), qy = (float)(iy + (ay.step > 0)), qz = (float)(iz + (az.step > 0));
                float anx = plane_alpha(ax, qx), any = plane_alpha(ay, qy), anz = plane_alpha(az, qz);
                int li = (iz - z0) * SPXY + (iy - y0) * SPX + (ix - x0);
                const int sx = ax.step, sy = ay.step * SPX, sz = az.step * SPXY;
                float acur = amin;
                const float fx = (float)ax.step, fy = (float)ay.step, fz = (float)az.step;
                // the crossing axis advances by selects, so lanes walking
                // different rays do not diverge over it
                for (int step = 0; step < BX + BY + BZ + 3; ++step) {
                    const float an = fminf(anx, fminf(any, anz));
                    const float ae = fminf(an, amax);
                    atomicAdd(&acc[li], round_int(fmaxf(ae - acur, 0.0f) * yl));
                    if (an >= amax) break;
                    acur = an;
                    const bool mx = an == anx, my = !mx && an == any, mz = !mx && !my;
                    ix += mx ? ax.step : 0;
                    iy += my ? ay.step : 0;
                    iz += mz ? az.step : 0;
                    if (ix < x0 || ix >= x1 || iy < y0 || iy >= y1 || iz < z0 || iz >= z1) break;
                    li += mx ? sx : (my ? sy : sz);
                    qx += mx ? fx : 0.0f;
                    qy += my ? fy : 0.0f;
                    qz += mz ? fz : 0.0f;
                    anx = mx ? plane_alpha(ax, qx) : anx;
                    any = my ? plane_alpha(ay, qy) : any;
                    anz = mz ? plane_alpha(az, qz) : anz;
                }
            }
        }
        __syncthreads();   // the pass's sums are complete, and after the last one G is free
        if (nbat == 0) break;
        // (each cell is read and cleared by one thread; the next group's
        // atomics come after two more barriers)
#pragma unroll
        for (int i = 0; i < OWN; ++i) {
            const int j = tid + T * i;
            int* q = acc + (j / (BX * BY)) * SPXY + ((j / BX) % BY) * SPX + j % BX;
            own[i] += __builtin_ldexpf((float)*q, -ex);
            *q = 0;
        }
        if (cls == 0 && cut < CTMI_INF) __syncthreads();   // before the second class's atomics
        }
    }
    store_owned<BZ, T>(vol, own, v, x0, y0, z0, beta);
}

// ---------------------------------------------------------- interpolated
// Each interpolation sample is processed once, by the brick that holds its
// lower corner (the first brick of an axis also takes corners at -1, whose
// cell lies outside the volume).  Its upper corners may fall one voxel past
// the brick: those cells form the brick's upper shell, 553 cells in three
// faces (x = BX with y, z in [0, BY] x [0, BZ]; y = BY with x < BX; z = BZ
// with x < BX, y < BY), written to the workspace and added to the
// neighbouring bricks' voxels by k_halo_add in a fixed order.
//
// The two corners of a sample along x are added with one 64-bit atomic: the
// accumulator has one 64-bit slot per pair (x, x + 1), the lower cell's
// integer in the low word and the upper one's in the high word, the sum
// (hi << 32) + lo of signed integers.  A cell's total is the low word of its
// own slot plus the (borrow-corrected) high word of the slot to its left.
// Four 64-bit atomics per sample cost 50 clocks on scattered addresses
// against 60 for eight 32-bit ones.
constexpr int HX = BX + 1, HY = BY + 2;   // slots x0 - 1 .. x1 - 1; one-voxel halo in y (and z)
// (odd pitches of rows and planes: an even row pitch puts rays side by side along y
// into the same banks, 512^3 x 120 views 134 to 209 ms; planes of 306 slots 103.1 ms,
// of 307 101.4)
constexpr int HXY = HX * HY + 1;

// The total of cell (lx, ly, lz), lx in [0, BX], from its two slots (slot
// index 0 is the pair that starts at x0 - 1; the last pair starts at BX - 1).
__device__ __forceinline__ int pair_sum(const u64* acc, int lx, int ly, int lz)
{
    const u64* r = acc + (lz + 1) * HXY + (ly + 1) * HX + lx;
    const u64 left = r[0];
    const int low = (int)(unsigned)left, high = (int)(unsigned)(left >> 32) - (low >> 31);
    return lx < BX ? high + (int)(unsigned)r[1] : high;
}

__device__ __forceinline__ void add_pair(u64* a, float q0, float q1)
{
    const int i0 = round_int(q0), i1 = round_int(q1) + (i0 >> 31);
    atomicAdd(a, (u64)(unsigned)i0 | ((u64)(unsigned)i1 << 32));
}

// Samples of ray r (relative to its anchor kc) that may lie in the box
// [lo, hi): per axis the interval between its faces, widened by 1e-3 of a
// sample against the reciprocal's rounding and by the samples within 2^-22
// |face| of a face (a position that close may round onto either side of it,
// and for a ray nearly parallel to the face that span holds many samples).
__device__ __forceinline__ void box_samples(const InterpRay& r, const float lo[3], const float hi[3], float& kmin,
                                            float& kmax)
{
    kmin = (float)(r.k0 - r.kc);
    kmax = (float)(r.k1 - r.kc);
    const float wface = 0x1p-22f * fmaxf(hi[0], fmaxf(hi[1], hi[2]));
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        if (r.st[a] != 0.0f) {
            const float ka = (lo[a] - r.base[a]) * r.inv[a], kb = (hi[a] - r.base[a]) * r.inv[a];
            const float wk = __builtin_fmaf(wface, fabsf(r.inv[a]), 1e-3f);
            kmin = fmaxf(kmin, __builtin_ceilf(fminf(ka, kb) - wk));
            kmax = fminf(kmax, __builtin_floorf(fmaxf(ka, kb) + wk));
        }
    }
}

template <int BZ, int NW, int GV, int WPE, bool PACK>
__global__ void __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(WPE, 8)))
k_backward_interp(const float* __restrict__ proj, float* __restrict__ vol, const ViewGeo* __restrict__ tab,
                  const ViewGeo64* __restrict__ tab64, int view0, int nviews, VolDims v, DetDims det, BrickMap m,
                  float beta, float ds, float cmax, float* __restrict__ shell)
{
    constexpr int T = 64 * NW, OWN = BX * BY * BZ / T, HZ = BZ + 2, HALO_SLOTS = Shell<BZ>::N;
    constexpr int NH = (HALO_SLOTS + T - 1) / T;
    __shared__ u64 acc[HXY * HZ];
    __shared__ GroupLds<GV> G;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    for (int i = tid; i < HXY * HZ; i += T) acc[i] = 0;
    float own[OWN], hown[NH];
#pragma unroll
    for (int i = 0; i < OWN; ++i) own[i] = 0.0f;
#pragma unroll
    for (int i = 0; i < NH; ++i) hown[i] = 0.0f;
    int bx, by, bz;
    brick_origin(m, (int)blockIdx.x, bx, by, bz);
    const int x0 = bx * BX, y0 = by * BY, z0 = bz * BZ;
    const int x1 = min(x0 + BX, v.nx), y1 = min(y0 + BY, v.ny), z1 = min(z0 + BZ, v.nz);
    // the brick takes samples whose lower corner (the floor of the position)
    // lies in [x0, x1) (from -1 for the first brick of an axis); their
    // positions lie in [lo, hi) (voxel-centre coordinates)
    const float lo[3] = {x0 > 0 ? (float)x0 : -1.0f, y0 > 0 ? (float)y0 : -1.0f, z0 > 0 ? (float)z0 : -1.0f};
    const float hi[3] = {(float)x1, (float)y1, (float)z1};
    // a corner's byte offset 8 ((c_z - z0 + 1) HXY + (c_y - y0 + 1) HX +
    // (c_x - x0 + 1)) is formed in FP32 (integers below 2^24)
    constexpr float AB = (float)sizeof(u64);
    const float aoff = -AB * ((float)(z0 - 1) * (float)HXY + (float)(y0 - 1) * (float)HX + (float)(x0 - 1));
    char* const accb = reinterpret_cast<char*>(acc);
    const float inv_ds = 1.0f / ds;

    for (int k = 0; k < nviews; k += GV) {
        int exs[2] = {0, 0};
        float cut = CTMI_INF;
        const int nbat = group_scale<false, PACK, NW, GV>(G, tab, proj, view0, k, min(GV, nviews - k), lo, hi, det, v, ds,
                                                    cmax, exs, cut);
        for (int cls = 0; cls < (cut < CTMI_INF ? 2 : 1); ++cls) {
        const int ex = exs[cls];
        int gv = 0;
        for (int bt = wave; bt < nbat; bt += NW) {
            int iu, iv;
            const bool in = group_pixel<false, PACK>(G, bt, lane, gv, iu, iv);
            float y = 0.0f;
            if (in) y = finite_or_zero(proj[((int64_t)(k + gv) * det.nv + iv) * det.nu + iu]);
            InterpRay r;
            if (y == 0.0f || (fabsf(y) > cut) != (cls != 0) || !interp_ray(tab64[view0 + k + gv], iu, iv, v, ds, inv_ds, r)) continue;
            float kmin, kmax;
            box_samples(r, lo, hi, kmin, kmax);
            // then trimmed to the samples whose lower corner is in the box:
            // FP32 positions are monotone in the sample index along every
            // axis, so these are consecutive
            auto inside = [&](float j) {
                bool ok = true;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const float p = __builtin_fmaf(j, r.st[a], r.base[a]);
                    ok &= p >= lo[a] && p < hi[a];
                }
                return ok;
            };
            while (kmin <= kmax && !inside(kmin)) kmin += 1.0f;
            while (kmin <= kmax && !inside(kmax)) kmax -= 1.0f;
            // scaled before ds: |y 2^e| <= 2^30 / N and N >= ds
            const float yv = __builtin_ldexpf(y, ex) * ds;
            // j runs over the samples as an exact FP32 integer
            for (float j = kmin; j <= kmax; j += 1.0f) {
                // same FP32 position as the forward kernel's sample k
                const float px = __builtin_fmaf(j, r.st[0], r.base[0]);
                const float py = __builtin_fmaf(j, r.st[1], r.base[1]);
                const float pz = __builtin_fmaf(j, r.st[2], r.base[2]);
                const float fx = __builtin_floorf(px), fy = __builtin_floorf(py), fz = __builtin_floorf(pz);
                const int boff = (int)__builtin_fmaf(fz, AB * (float)HXY,
                                                     __builtin_fmaf(fy, AB * (float)HX, __builtin_fmaf(fx, AB, aoff)));
                const float ax_ = px - fx, ay_ = py - fy, az_ = pz - fz;
                // trilinear weights times y, each pair split as (w - a w, a w)
                const float yz1 = az_ * yv, yz0 = yv - yz1;
                const float w10 = ay_ * yz0, w00 = yz0 - w10;
                const float w11 = ay_ * yz1, w01 = yz1 - w11;
                const float u00 = ax_ * w00, u10 = ax_ * w10, u01 = ax_ * w01, u11 = ax_ * w11;
                u64* a0 = reinterpret_cast<u64*>(accb + boff);
                add_pair(a0, w00 - u00, u00);
                add_pair(a0 + HX, w10 - u10, u10);
                add_pair(a0 + HXY, w01 - u01, u01);
                add_pair(a0 + HXY + HX, w11 - u11, u11);
            }
        }
        __syncthreads();   // the pass's sums are complete, and after the last one G is free
        if (nbat == 0) break;
#pragma unroll
        for (int i = 0; i < OWN; ++i) {
            const int j = tid + T * i;
            own[i] += __builtin_ldexpf((float)pair_sum(acc, j % BX, (j / BX) % BY, j / (BX * BY)), -ex);
        }
#pragma unroll
        for (int i = 0; i < NH; ++i) {
            const int h = tid + T * i;
            if (h < HALO_SLOTS) {
                int lx, ly, lz;
                Shell<BZ>::cell(h, lx, ly, lz);
                hown[i] += __builtin_ldexpf((float)pair_sum(acc, lx, ly, lz), -ex);
            }
        }
        __syncthreads();   // a slot is read for both of its cells
        // (the next group's atomics come after two more barriers)
        for (int i = tid; i < HXY * HZ; i += T) acc[i] = 0;
        if (cls == 0 && cut < CTMI_INF) __syncthreads();   // before the second class's atomics
        }
    }
    store_owned<BZ, T>(vol, own, v, x0, y0, z0, beta);
    float* out = shell + (size_t)blockIdx.x * HALO_SLOTS;
#pragma unroll
    for (int i = 0; i < NH; ++i) {
        const int h = tid + T * i;
        if (h < HALO_SLOTS) out[h] = hown[i];
    }
}

// Adds the upper shells of the lower neighbour bricks to the voxels on each
// brick's lower faces, in a fixed order (x, y, z, xy, xz, yz, xyz neighbours).
// A workgroup takes the face cells of one brick (a fifth to a quarter of its
// voxels): with a thread for every voxel of the volume, most of them with nothing
// to add, the index divisions bound it (256^3: 72 us, 38 us so).
template <int BZ>
__global__ void __launch_bounds__(256) k_halo_add(float* __restrict__ vol, const float* __restrict__ shell, VolDims v,
                                                  BrickMap m)
{
    constexpr int HSX = Shell<BZ>::SX, HSY = Shell<BZ>::SY, HALO_SLOTS = Shell<BZ>::N;
    constexpr int FZ = BX * BY, FY = BX * (BZ - 1), FX = (BY - 1) * (BZ - 1);   // cells of the lower z, y and x faces
    int bx, by, bz;
    brick_origin(m, (int)blockIdx.x, bx, by, bz);
    for (int c = threadIdx.x; c < FZ + FY + FX; c += 256) {
        int lx = c % BX, ly = c / BX, lz = 0;
        if (c >= FZ + FY) {
            lx = 0;
            ly = 1 + (c - FZ - FY) % (BY - 1);
            lz = 1 + (c - FZ - FY) / (BY - 1);
        } else if (c >= FZ) {
            lz = 1 + (c - FZ) / BX;
            ly = 0;
        }
        const int gx = bx * BX + lx, gy = by * BY + ly, gz = bz * BZ + lz;
        if (gx >= v.nx || gy >= v.ny || gz >= v.nz) continue;
        auto cell = [&](int ex, int ey, int ez, int slot) {
            return shell[((size_t)((ez * m.nby + ey) * m.nbx + ex)) * HALO_SLOTS + slot];
        };
        const bool X = lx == 0 && bx > 0, Y = ly == 0 && by > 0, Z = lz == 0 && bz > 0;
        float add = 0.0f;
        if (X) add += cell(bx - 1, by, bz, ly + (BY + 1) * lz);
        if (Y) add += cell(bx, by - 1, bz, HSX + lx + BX * lz);
        if (Z) add += cell(bx, by, bz - 1, HSX + HSY + lx + BX * ly);
        if (X && Y) add += cell(bx - 1, by - 1, bz, BY + (BY + 1) * lz);
        if (X && Z) add += cell(bx - 1, by, bz - 1, ly + (BY + 1) * BZ);
        if (Y && Z) add += cell(bx, by - 1, bz - 1, HSX + lx + BX * BZ);
        if (X && Y && Z) add += cell(bx - 1, by - 1, bz - 1, BY + (BY + 1) * BZ);
        if (X || Y || Z) vol[((int64_t)gz * v.ny + gy) * v.nx + gx] += add;
    }
}

// Non-finite projection values.  The adjoints above add finite values only
// (a NaN or infinite y_i counts as 0 there, which keeps the fixed-point
// scales finite); this pass then sets every voxel that such a ray reaches to
// NaN, since a_ij y_i is NaN or infinite there.  A voxel is reached when the
// Siddon walk gives it a piece of positive length, or when it is a corner of
// an interpolation sample inside the interpolant's support.  Rays are taken
// grid-stride, one per thread; a ray with a finite value costs one coalesced
// load.
template <bool SIDDON>
__global__ void __launch_bounds__(256) k_nonfinite(const float* __restrict__ proj, float* __restrict__ vol,
                                                   const ViewGeo64* __restrict__ tab64, int view0, int64_t nrays,
                                                   VolDims v, DetDims det, float ds, float inv_ds)
{
    const int64_t npix = (int64_t)det.nu * det.nv;
    const float qnan = __builtin_nanf("");
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nrays; i += (int64_t)gridDim.x * blockDim.x) {
        if (finite_or_zero(proj[i]) == proj[i]) continue;
        const int view = (int)(i / npix);
        const int pix = (int)(i - (int64_t)view * npix);
        const int iu = pix % det.nu, iv = pix / det.nu;
        const ViewGeo64& g = tab64[view0 + view];
        if (SIDDON) {
            float S[3], d[3], amin, amax;
            siddon_ray(g, iu, iv, v, S, d, amin, amax);
            const SiddonAxis ax = siddon_axis(S[0], d[0]), ay = siddon_axis(S[1], d[1]), az = siddon_axis(S[2], d[2]);
            bool hit = slab_clip(ax, S[0], 0.0f, (float)v.nx, amin, amax);
            hit &= slab_clip(ay, S[1], 0.0f, (float)v.ny, amin, amax);
            hit &= slab_clip(az, S[2], 0.0f, (float)v.nz, amin, amax);
            if (!hit || !(amin < amax)) continue;
            int ix = ordered_cell(ax, S[0], d[0], amin, 0, v.nx);
            int iy = ordered_cell(ay, S[1], d[1], amin, 0, v.ny);
            int iz = ordered_cell(az, S[2], d[2], amin, 0, v.nz);
            float anx = plane_alpha(ax, (float)(ix + (ax.step > 0)));
            float any = plane_alpha(ay, (float)(iy + (ay.step > 0)));
            float anz = plane_alpha(az, (float)(iz + (az.step > 0)));
            float acur = amin;
            for (int step = 0; step < v.nx + v.ny + v.nz + 3; ++step) {
                const float an = fminf(anx, fminf(any, anz));
                if (fminf(an, amax) > acur) vol[((int64_t)iz * v.ny + iy) * v.nx + ix] = qnan;
                if (an >= amax) break;
                acur = an;
                if (an == anx) {
                    ix += ax.step;
                    if (ix < 0 || ix >= v.nx) break;
                    anx = plane_alpha(ax, (float)(ix + (ax.step > 0)));
                } else if (an == any) {
                    iy += ay.step;
                    if (iy < 0 || iy >= v.ny) break;
                    any = plane_alpha(ay, (float)(iy + (ay.step > 0)));
                } else {
                    iz += az.step;
                    if (iz < 0 || iz >= v.nz) break;
                    anz = plane_alpha(az, (float)(iz + (az.step > 0)));
                }
            }
        } else {
            InterpRay r;
            if (!interp_ray(g, iu, iv, v, ds, inv_ds, r)) continue;
            for (int k = r.k0; k <= r.k1; ++k) {
                float p[3];
                interp_pos(r, k, p);
                if (!(p[0] > -1.0f && p[0] < (float)v.nx && p[1] > -1.0f && p[1] < (float)v.ny && p[2] > -1.0f &&
                      p[2] < (float)v.nz))
                    continue;
                const int fx = (int)__builtin_floorf(p[0]), fy = (int)__builtin_floorf(p[1]),
                          fz = (int)__builtin_floorf(p[2]);
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    const int cx = fx + (c & 1), cy = fy + ((c >> 1) & 1), cz = fz + (c >> 2);
                    if (cx >= 0 && cx < v.nx && cy >= 0 && cy < v.ny && cz >= 0 && cz < v.nz)
                        vol[((int64_t)cz * v.ny + cy) * v.nx + cx] = qnan;
                }
            }
        }
    }
}

template <bool SIDDON>
hipError_t launch_nonfinite(const Plan& p, const float* proj, float* vol, int64_t view0, int64_t nviews, hipStream_t s)
{
    const int64_t nrays = nviews * (int64_t)p.det.nu * p.det.nv;
    if (nrays == 0) return hipSuccess;
    const int64_t blocks = std::min<int64_t>((nrays + 255) / 256, 65536);
    hipLaunchKernelGGL(k_nonfinite<SIDDON>, dim3((unsigned)blocks), dim3(256), 0, s, proj, vol, p.d_views64,
                       (int)view0, nrays, p.vol, p.det, p.ds, 1.0f / p.ds);
    return hipGetLastError();
}

}  // namespace

int64_t adjoint_bricks(const Plan& p)
{
    const BrickMap m = brick_map(p, CTMI_BWD_BZ);
    return (int64_t)m.nbx * m.nby * m.nbz;
}

size_t interp_adjoint_ws_bytes(const Plan& p) { return sizeof(float) * (size_t)adjoint_bricks(p) * CTMI_HALO_SLOTS; }

// Views per call up to which the interpolated adjoint keeps a fixed-point unit
// per round of rays (backward_few.hip); ordered-subset blocks lie below.  Neither
// side's unit is the coarser one for such blocks: against FP64 sums of finely
// rounded single-view parts, the quotients A_s^T r / A_s^T 1 of SART and EM
// iterations (36 to 64 views, volumes of 64^3 to 256^3 and one wider than its
// detector) have 0.2 to 0.5 of the rounds' error at the 99.99th percentile of the
// voxels with a unit per group; the worst single voxel, reached by little more than a
// unit, 0.1 to 1.4 of it.  (Siddon, a unit per group at every view count: 1, 5, 12 and 36
// views, 0.02 to 0.6 and 0.001 to 3 of the former rounds'.)  The bricks above are faster there
// too (18 views of 512x512 on 256^3, an OS-SART block: 5.27 ms against 6.46).
// The line keeps the rounding of short blocks as it was: such single voxels move by as
// much as their error, up to 2e-4 over blocks of 5 to 27 views.
constexpr int64_t FEW_VIEWS = 32;

template <int BZ>
hipError_t launch_halo_add(const Plan& p, float* vol, const float* shell, hipStream_t s)
{
    const BrickMap m = brick_map(p, BZ);
    if (m.nbx * m.nby * m.nbz == 1) return hipSuccess;   // no neighbours
    hipLaunchKernelGGL(k_halo_add<BZ>, dim3((unsigned)m.nbx * m.nby * m.nbz), dim3(256), 0, s, vol, shell, p.vol, m);
    return hipGetLastError();
}

template <bool SIDDON, int BZ, int NW, int GV, int WPE, bool PACK = false>
hipError_t launch_bricks(const Plan& p, const float* proj, float* vol, int64_t view0, int64_t nviews, float beta,
                         float* shell, hipStream_t s)
{
    const BrickMap m = brick_map(p, BZ);
    const dim3 grid((unsigned)m.nbx * m.nby * m.nbz), block(64 * NW);
    if constexpr (SIDDON) {
        hipLaunchKernelGGL((k_backward_siddon<BZ, NW, GV, WPE, PACK>), grid, block, 0, s, proj, vol, p.d_views, p.d_views64,
                           (int)view0, (int)nviews, p.vol, p.det, m, beta, p.round_siddon);
        return hipGetLastError();
    } else {
        hipLaunchKernelGGL((k_backward_interp<BZ, NW, GV, WPE, PACK>), grid, block, 0, s, proj, vol, p.d_views, p.d_views64,
                           (int)view0, (int)nviews, p.vol, p.det, m, beta, p.ds, p.round_interp, shell);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        return launch_halo_add<BZ>(p, vol, shell, s);
    }
}

// Brick height and waves per brick, by the number of 16x16x8 bricks.  From
// 1280 on, bricks of 16 planes with 8 waves (24 waves per CU in three
// workgroups) fill the GPU's 256 CUs: fewer rays are cut short by a brick's
// upper and lower face, so a wave's lanes run more alike, and the footprint,
// scale and flush of a group are shared by twice the voxels (interpolated, 512^3
// x 120 views: 114 -> 104 ms against bricks of 8 planes with 4 waves; Siddon,
// 256^3 x 90 views: 9.6 -> 8.5 ms).  Below that the bricks of 8 planes keep more
// CUs at work (128^3 x 12 views, Siddon: 205 us against 215; 1 127 bricks, Siddon,
// 46 views: 555 against 580, where 1 352 gain: 480 -> 463 us, interpolated 1 120 ->
// 907, and 1 519: 636 -> 537 and 2 738 -> 2 209), and below 512 a
// brick takes 16 waves; the Siddon adjoint, which has no shells whose size the
// workspace fixes, then also halves the brick (64^3 x 64 views, forward and
// adjoint: 199 -> 177 us).  A volume of up to 8 planes has one layer of bricks
// either way, and its workspace holds the shells of bricks of 8.
//
// Where a brick of 8 planes has few rays in a view (pixels of about two voxels and
// more, detectors of a row or two), batches of 64 lanes run over the views' ends, in
// groups of 16 or 32 views: a batch per view leaves most of its lanes idle.  Footprints of
// 160 pixels gain 5 to 10 % so (more gain nothing), those of 30 a third to a half: 64 views
// on pixels of 5 voxels, Siddon, 256^3 644 -> 477 us, 128^3 182 -> 94, interpolated 1058 -> 807
// and 276 -> 131 (at 128^3 with four waves per brick, since every brick has its few
// rays; on a detector of one row with eight).  Up to 8 views there is one group
// either way, and the 16-plane bricks' is the faster one without.
struct AdjointForm {
    bool tall, mid;    // bricks of 16 planes; of 8 planes with 8 waves
    bool sparse;       // few rays per brick and view
    bool whole;        // the detector is larger than a brick's footprint
};
static AdjointForm adjoint_form(const Plan& p)
{
    const int64_t bricks = adjoint_bricks(p);
    const float w = 22.6f / p.pix[0] + 1.0f, h = 8.8f / p.pix[1] + 1.0f;   // a brick's footprint at the volume's centre
    const float nu = (float)p.det.nu, nv = (float)p.det.nv;
    AdjointForm f;
    f.tall = p.vol.nz > 8 && bricks >= 1280;
    f.mid = !f.tall && bricks >= 512;
    // (fewer than 2^26 pixels: a group's padded footprints are counted in an int32)
    f.sparse = fminf(w, nu) * fminf(h, nv) <= 160.0f && nu * nv < 0x1p26f;
    f.whole = w <= nu && h <= nv;
    return f;
}

template <bool SIDDON>
hipError_t launch_adjoint(const Plan& p, const float* proj, float* vol, int64_t view0, int64_t nviews, float beta,
                          float* shell, hipStream_t s)
{
    const AdjointForm f = adjoint_form(p);
    if (f.tall) {
        if (f.sparse && nviews > 8)
            return launch_bricks<SIDDON, 16, 8, 16, 6, true>(p, proj, vol, view0, nviews, beta, shell, s);
        return launch_bricks<SIDDON, 16, 8, 8, 6>(p, proj, vol, view0, nviews, beta, shell, s);
    }
    if (f.mid) {
        constexpr int GV = SIDDON ? 16 : 32, WPE = SIDDON ? 6 : 4;
        if (f.sparse && f.whole)
            return launch_bricks<SIDDON, 8, 4, GV, WPE, true>(p, proj, vol, view0, nviews, beta, shell, s);
        if (f.sparse) return launch_bricks<SIDDON, 8, 8, GV, WPE, true>(p, proj, vol, view0, nviews, beta, shell, s);
        return launch_bricks<SIDDON, 8, 8, 8, 6>(p, proj, vol, view0, nviews, beta, shell, s);
    }
    if (f.sparse) return launch_bricks<SIDDON, SIDDON ? 4 : 8, 16, 16, 4, true>(p, proj, vol, view0, nviews, beta, shell, s);
    return launch_bricks<SIDDON, SIDDON ? 4 : 8, 16, 16, 4>(p, proj, vol, view0, nviews, beta, shell, s);
}

hipError_t launch_backward_siddon(const Plan& p, const float* proj, float* vol, int64_t view0, int64_t nviews,
                                  float beta, hipStream_t s)
{
    const hipError_t e = launch_adjoint<true>(p, proj, vol, view0, nviews, beta, nullptr, s);
    if (e != hipSuccess) return e;
    return launch_nonfinite<true>(p, proj, vol, view0, nviews, s);
}

hipError_t launch_backward_interp(const Plan& p, const float* proj, float* vol, int64_t view0, int64_t nviews,
                                  float beta, float* shell, hipStream_t s)
{
    hipError_t e;
    if (nviews <= FEW_VIEWS) {
        e = launch_backward_interp_few_bricks(p, proj, vol, view0, nviews, beta, shell, s);
        if (e == hipSuccess) e = launch_halo_add<CTMI_BWD_BZ>(p, vol, shell, s);
    } else {
        e = launch_adjoint<false>(p, proj, vol, view0, nviews, beta, shell, s);
    }
    if (e != hipSuccess) return e;
    return launch_nonfinite<false>(p, proj, vol, view0, nviews, s);
}

}  // namespace ctmi
