// Forward projectors A (the linear model A x = b of section 2.1): one thread
// per detector pixel, projection-major ray tiles, LDS-staged volume slabs.
//
// A workgroup of 256 threads owns a 16x16 pixel tile of one view.  The tile's
// rays run mostly along one axis (the dominant axis of the tile's central
// ray); the volume is cut into slabs of a few cells across that axis and the
// workgroup visits the slabs in the direction of travel.  For each slab it
// stages in LDS the box of voxels the tile's rays can touch there (bounded by
// the four corner rays of the tile, which enclose the whole ray bundle), then
// every thread advances its own ray through the slab reading the volume from
// LDS.  Global reads are coalesced box loads instead of per-sample gathers
// from scattered cache lines.  A sample whose voxels fall outside the staged
// box (box clipped to the LDS capacity, rounding at the box edge) reads them
// from global memory, so the result never depends on the box estimate.
//
// Blocks are ordered (tile row, groups of 16 views, tile column, view in
// group), and renumbered so that each XCD runs a contiguous run of that
// order: the workgroups in flight on one XCD share one detector row band,
// hence one z-band of the volume, and stage overlapping boxes for nearby
// views under one L2.
//
// The interpolated projector stages its boxes one slab ahead: the next
// slab's first 4096 box elements are loaded into registers while the
// current slab is sampled (the register budget is held at six waves per SIMD,
// the LDS limit).  The Siddon walk keeps more state per ray, so it stages each
// box when it needs it, at five waves per SIMD (six spill: 4163 against 4084 us
// for 256^3 x 90 on 512^2).
//
// Both are bound by VALU and LDS about equally: 512^3 x 120 on 1024 x 768
// interpolated 80.8 -> 61.2 ms (1.40 VALU instructions and 0.83 LDS steps per CU
// and clock), 256^3 x 90 on 512^2 Siddon 5.87 -> 4.08 ms, with staging in quads,
// pitches without bank conflicts, slabs fitted to each tile and LDS addresses formed
// in FP32.
#include "ctmi_internal.h"

namespace ctmi {

namespace {

#ifndef CTMI_FWD_TU
#define CTMI_FWD_TU 16
#endif
#ifndef CTMI_FWD_TV
#define CTMI_FWD_TV 16
#endif
// interpolated forward: groups of four box elements per thread fetched ahead
// into registers, and the waves per SIMD the register budget is sized for
#ifndef CTMI_FWD_PF
#define CTMI_FWD_PF 4
#endif
#ifndef CTMI_FWD_WAVES
#define CTMI_FWD_WAVES 6
#endif
// Siddon forward: waves per SIMD the register budget is sized for
#ifndef CTMI_FWD_SID_WAVES
#define CTMI_FWD_SID_WAVES 5
#endif
constexpr int TU = CTMI_FWD_TU, TV = CTMI_FWD_TV;   // ray tile (pixels), TU * TV = 256
#ifndef CTMI_FWD_SID_PF
#define CTMI_FWD_SID_PF 4
#endif
// Slab thickness along the dominant axis: the thickest of these of which every
// slab's box fits the LDS capacity (a clipped box sends its slab's samples through
// the checked path), the last if none does.  Thin slabs pay more for their
// barriers, setup and, in the interpolated projector, three planes of overlap, but
// boxes of rays at 45 degrees and of pixels of a voxel or more are wide: 24 views of
// 256 x 256 x 128 on 256 x 200 pixels of a voxel, one thickness (10; Siddon 12)
// 1532 us, Siddon 785, so 993 and 490.  Along x the planes are the box's rows: 4 n +
// 1 and the overlap make rows of 4 n + 4 words.
#ifndef CTMI_FWD_THICK
#define CTMI_FWD_THICK {16, 13, 10, 8, 6, 4, 4}
#endif
#ifndef CTMI_FWD_THICK_X
#define CTMI_FWD_THICK_X {17, 13, 9, 9, 5, 5, 5}
#endif
#ifndef CTMI_FWD_SID_THICK
#define CTMI_FWD_SID_THICK {24, 20, 16, 12, 8, 4, 8}
#endif
constexpr int NTHICK = 7;
__device__ __forceinline__ int interp_thickness(int a, int c)
{
    constexpr int t[NTHICK] = CTMI_FWD_THICK, tx[NTHICK] = CTMI_FWD_THICK_X;
    int r = 0;
#pragma unroll
    for (int i = 0; i < NTHICK; ++i) r = i == c ? (a == 0 ? tx[i] : t[i]) : r;
    return r;
}
__device__ __forceinline__ int siddon_thickness(int c)
{
    constexpr int t[NTHICK] = CTMI_FWD_SID_THICK;
    int r = 0;
#pragma unroll
    for (int i = 0; i < NTHICK; ++i) r = i == c ? t[i] : r;
    return r;
}
constexpr int SLABTAB = 64;                         // slab boxes formed up front per block
constexpr int BOXCAP_MAX = 15360;                   // most LDS floats for the staged box
static_assert(TU * TV == 256, "one ray per thread");

struct TileMap {
    int tiles_u, tiles_v;
    int64_t nviews;
};

// Staged box: voxel index origin and extent per axis (x, y, z); LDS layout
// [z][y][x] with x fastest (coalesced global loads), the x extent a multiple of 4.
struct Box {
    int o[3];
    int e[3];
    int w, wz;   // pitch of rows and planes in LDS
};

// Pitches of a box of e0 x e1 cells per plane.  A read takes 32 lanes (two
// detector rows of 16 rays) a clock from 32 banks.  Where the dominant axis is y or
// z, rays side by side read along x, so the two rows' banks are disjoint if the
// planes lie 16 banks apart; rows and planes stay on 16 bytes, and the box is
// written four words at a time.  Along x, rays side by side read rows side by side
// (and cells of two columns): even pitches of 2 mod 4 with odd planes.  A model of
// the tile's reads gives 1.33 and 1.36 clocks per 32 lanes for these, 1.72 for
// unpadded planes and 1.86, 2.3 and 3 for row pitches of 13, 12 and 16 along x;
// interpolated A, 512^3 x 120: 89 ms at
// 12 words and unpadded planes, 195 at 16, 68.4 at 13, 61.2 so.
__device__ __forceinline__ int row_pad(int a) { return a == 0 ? 2 : 0; }
__device__ __forceinline__ int plane_pitch(int a, int w, int e1)
{
    const int n = w * e1;
    return a == 0 ? n | 1 : ((n + 15) & ~31) + 16;
}

#ifndef CTMI_FWD_XCD
#define CTMI_FWD_XCD 1
#endif
#ifndef CTMI_FWD_ORDER
#define CTMI_FWD_ORDER 1
#endif
#ifndef CTMI_FWD_VG
#define CTMI_FWD_VG 16
#endif

// With CTMI_FWD_XCD each XCD runs a contiguous run of the tile order, so
// tiles that stage overlapping volume boxes (neighbouring tiles of nearby
// views) share an L2 (A 640 -> 582 ms, Siddon 690 -> 592 ms at 512^3 x 720).
__device__ __forceinline__ int64_t xcd_order(int64_t b, int64_t nblocks)
{
    return CTMI_FWD_XCD ? xcd_contiguous(b, nblocks) : b;
}

__device__ __forceinline__ void tile_of_block(const TileMap& m, int64_t b, int& view, int& tu0, int& tv0)
{
    b = xcd_order(b, (int64_t)m.tiles_u * m.tiles_v * m.nviews);
    int tu, tv;
    if (CTMI_FWD_ORDER == 0) {
        // (tile row, view, tile column)
        const int64_t per_row = m.nviews * m.tiles_u;
        tv = (int)(b / per_row);
        const int64_t rem = b - (int64_t)tv * per_row;
        view = (int)(rem / m.tiles_u);
        tu = (int)(rem - (int64_t)view * m.tiles_u);
    } else {
        // (tile row, groups of VG views, tile column, view in group)
        const int64_t per_row = m.nviews * m.tiles_u;
        tv = (int)(b / per_row);
        int64_t rem = b - (int64_t)tv * per_row;
        const int64_t gsz = (int64_t)CTMI_FWD_VG * m.tiles_u;
        const int64_t g = rem / gsz;
        rem -= g * gsz;
        const int64_t nvg = min((int64_t)CTMI_FWD_VG, m.nviews - g * CTMI_FWD_VG);   // views in this group
        tu = (int)(rem / nvg);
        view = (int)(g * CTMI_FWD_VG + (rem - (int64_t)tu * nvg));
    }
    tu0 = tu * TU;
    tv0 = tv * TV;
}

// Dominant axis and travel direction of the tile's central ray (uniform).
__device__ __forceinline__ void tile_axis(const ViewGeo& g, const DetDims& det, int tu0, int tv0, int& a, int& dir)
{
    const float uc = (float)tu0 + 0.5f * (float)(min(TU, det.nu - tu0) - 1);
    const float vc = (float)tv0 + 0.5f * (float)(min(TV, det.nv - tv0) - 1);
    float dc[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) dc[i] = g.P00[i] + uc * g.DU[i] + vc * g.DV[i] - g.S[i];
    const float ax = fabsf(dc[0]), ay = fabsf(dc[1]), az = fabsf(dc[2]);
    a = (ax >= ay && ax >= az) ? 0 : (ay >= az ? 1 : 2);
    dir = dc[a] >= 0.0f ? 1 : -1;
}

// Bounds along the two non-dominant axes of the tile's ray bundle between
// planes pa0 and pa1 of axis a, in coordinates shifted by `shift` (0 for
// voxel-cell coordinates, 0.5 for voxel-centre coordinates).
__device__ __forceinline__ void bundle_bounds(const ViewGeo& g, const DetDims& det, int tu0, int tv0, int a,
                                              float pa0, float pa1, float shift, float lo[3], float hi[3])
{
    const int iu1 = min(tu0 + TU, det.nu) - 1, iv1 = min(tv0 + TV, det.nv) - 1;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        lo[i] = CTMI_INF;
        hi[i] = -CTMI_INF;
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        float S[3], d[3];
        pixel_ray(g, (c & 1) ? iu1 : tu0, (c & 2) ? iv1 : tv0, S, d);
#pragma unroll
        for (int i = 0; i < 3; ++i) S[i] -= shift;
        const float inv = 1.0f / d[a];
#pragma unroll
        for (int pl = 0; pl < 2; ++pl) {
            const float t = ((pl ? pa1 : pa0) - S[a]) * inv;
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const float x = __builtin_fmaf(t, d[i], S[i]);
                lo[i] = fminf(lo[i], x);
                hi[i] = fmaxf(hi[i], x);
            }
        }
    }
}

// Box covering index range [lo_i, hi_i] per axis, clipped to [clo_i, chi_i]
// and to the LDS capacity (the non-dominant axes shrink first).  Returns 0 if
// it is empty, BOX_SOME, or BOX_SOME | BOX_CLIPPED where the capacity cut it.
constexpr int BOX_SOME = 1, BOX_CLIPPED = 2;
__device__ __forceinline__ int make_box(const int lo[3], const int hi[3], const int clo[3], const int chi[3], int a, int cap,
                                         Box& b)
{
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const int l = max(lo[i], clo[i]), h = min(hi[i], chi[i]);
        if (h < l) return 0;
        b.o[i] = l;
        b.e[i] = h - l + 1;
    }
    b.e[0] = (b.e[0] + 3) & ~3;
    // capacity: shrink the larger non-dominant extent until the box fits
    const int pad = row_pad(a);
    auto size = [&]() { return plane_pitch(a, b.e[0] + pad, b.e[1]) * b.e[2]; };
    const bool clipped = size() > cap;
    for (int it = 0; it < 4 && size() > cap; ++it) {
        const int e1 = a == 0 ? b.e[1] : b.e[0];      // first non-dominant extent
        const int e2 = a == 2 ? b.e[1] : b.e[2];      // second non-dominant extent
        const bool first = e1 >= e2;
        const int cut = first ? (a == 0 ? 1 : 0) : (a == 2 ? 1 : 2);
        const int room = max(cap / b.e[2] - 31, 0);   // for a plane without its padding
        if (cut == 0)
            b.e[0] = max((room / b.e[1] - pad) & ~3, 4);
        else if (cut == 1)
            b.e[1] = max(room / (b.e[0] + pad), 1);
        else
            b.e[2] = max(cap / plane_pitch(a, b.e[0] + pad, b.e[1]), 1);
    }
    if (size() > cap) {   // (at most the thickest slab's planes of one row: always fits)
        b.e[0] = a == 0 ? b.e[0] : 4;
        b.e[1] = a == 1 ? b.e[1] : 1;
        b.e[2] = a == 2 ? b.e[2] : 1;
    }
    b.w = b.e[0] + pad;
    b.wz = plane_pitch(a, b.w, b.e[1]);
    return clipped ? BOX_SOME | BOX_CLIPPED : BOX_SOME;
}

// Box staging by rows, four consecutive x at a time.  A row is the box's x
// extent at one (y, z), W = e[0] / 4 quads; thread t takes quad t mod W of rows
// t div W + m RG (pass m), RG = floor(256 / W) whole rows per pass, so a thread's
// column and its x bounds check stay fixed.  From one pass to the next a
// thread's row advances by RG = RGz e[1] + RGy, so its (y, z), its global index
// and its LDS index advance by constants, with one carry from y into z.  (Element by
// element, and with the quotients formed by every thread for every slab, staging
// took 360 of the interpolated projector's 1160 VALU instructions per slab and
// wave; global loads of four words need only their word's alignment.)  Initial
// quotients use float reciprocals: floor((i + 1/2) r), r = fl(1/e), equals i div
// e for every i < 2^22, because (i + 1/2)/e is at least 1/(2e) away from an
// integer while the FP32 error is below (i + 1/2) 2^-23 / e.  The global index is
// kept modulo 2^32 (a cell inside the volume has an index below 2^31, checked at
// plan creation).  A box wider than 1024 along x (not produced by tile-sized
// bundles) is staged element by element.
typedef float quad __attribute__((ext_vector_type(4), aligned(4)));
typedef float pair __attribute__((ext_vector_type(2), aligned(4)));
typedef float quad16 __attribute__((ext_vector_type(4)));

// What staging a slab's box needs, the same for the whole block: one row of the
// block's slab table.
struct Slab {
    Box b;
    int flags;
    float r0, r1;        // 1 / W, 1 / e[1]
    int rg, rgy, rgz;    // rows per pass (0: box wider than 1024) and the pass advance
};

__device__ __forceinline__ Slab slab_of_box(const Box& b, int flags)
{
    Slab s;
    s.b = b;
    s.flags = flags;
    const int w = b.e[0] >> 2;
    s.r0 = 1.0f / (float)w;
    s.r1 = 1.0f / (float)b.e[1];
    s.rg = w <= 256 ? (int)__builtin_floorf(256.5f * s.r0) : 0;
    s.rgz = (int)__builtin_floorf(((float)s.rg + 0.5f) * s.r1);
    s.rgy = s.rg - s.rgz * b.e[1];
    return s;
}

// A table row is eight words: origin, e0 | e1 << 16, e2 | flags << 16, the two
// reciprocals (the pitches follow from the extents), rg | rgz << 9 | rgy << 18 (rg and rgz at most 256, rgy below e1 <= the capacity)
static_assert(BOXCAP_MAX < 1 << 14, "rgy in 14 bits");
__device__ __forceinline__ void put_slab(int4* row, const Slab& s)
{
    row[0] = make_int4(s.b.o[0], s.b.o[1], s.b.o[2], s.b.e[0] | s.b.e[1] << 16);
    row[1] = make_int4(s.b.e[2] | s.flags << 16, __float_as_int(s.r0), __float_as_int(s.r1),
                       s.rg | s.rgz << 9 | (int)((unsigned)s.rgy << 18));
}

__device__ __forceinline__ Slab get_slab(const int4* row, int a)
{
    const int4 p = row[0], q = row[1];
    Slab s;
    s.b.o[0] = __builtin_amdgcn_readfirstlane(p.x);
    s.b.o[1] = __builtin_amdgcn_readfirstlane(p.y);
    s.b.o[2] = __builtin_amdgcn_readfirstlane(p.z);
    const int e01 = __builtin_amdgcn_readfirstlane(p.w), e2f = __builtin_amdgcn_readfirstlane(q.x);
    const int adv = __builtin_amdgcn_readfirstlane(q.w);
    s.b.e[0] = e01 & 0xffff;
    s.b.e[1] = (int)((unsigned)e01 >> 16);
    s.b.e[2] = e2f & 0xffff;
    s.flags = (int)((unsigned)e2f >> 16);
    s.b.w = s.b.e[0] + row_pad(a);
    s.b.wz = plane_pitch(a, s.b.w, s.b.e[1]);
    s.r0 = __int_as_float(q.y);
    s.r1 = __int_as_float(q.z);
    s.rg = adv & 511;
    s.rgz = (adv >> 9) & 511;
    s.rgy = (int)((unsigned)adv >> 18);
    return s;
}

struct Stage {
    int gx;            // this thread's volume x
    int ly, lz;        // its current row as box (y, z); lz past the box when the thread is done (or holds no column)
    unsigned gi;       // global index of its current quad (mod 2^32)
    int li;            // its LDS index
};

// this thread's position at pass m0
__device__ __forceinline__ Stage stage_of(const Slab& sl, const VolDims& v, int m0)
{
    Stage s;
    const Box& b = sl.b;
    const int w = b.e[0] >> 2, t = (int)threadIdx.x;
    const int tr = (int)__builtin_floorf(((float)t + 0.5f) * sl.r0);
    const int row = tr + m0 * sl.rg;
    s.lz = (int)__builtin_floorf(((float)row + 0.5f) * sl.r1);
    s.ly = row - (int)__umul24(s.lz, b.e[1]);
    const int tx = 4 * (t - (int)__umul24(tr, w));
    s.gx = b.o[0] + tx;
    const unsigned nx = (unsigned)v.nx, nxy = (unsigned)v.nx * (unsigned)v.ny;
    s.gi = ((unsigned)b.o[2] * nxy + (unsigned)b.o[1] * nx) + ((unsigned)s.lz * nxy + (unsigned)s.ly * nx) + (unsigned)s.gx;
    s.li = (int)__umul24(s.lz, b.wz) + (int)__umul24(s.ly, b.w) + tx;
    if (t >= sl.rg * w) s.lz = 1 << 20;
    return s;
}

__device__ __forceinline__ void stage_step(Stage& s, const Slab& sl, const VolDims& v)
{
    const unsigned nx = (unsigned)v.nx, nxy = (unsigned)v.nx * (unsigned)v.ny;
    const unsigned d1 = (unsigned)sl.rgz * nxy + (unsigned)sl.rgy * nx;   // and on a carry into z:
    const unsigned d2 = d1 + nxy - (unsigned)sl.b.e[1] * nx;
    const int l1 = sl.rgz * sl.b.wz + sl.rgy * sl.b.w, l2 = l1 + sl.b.wz - sl.b.e[1] * sl.b.w;
    s.ly += sl.rgy;
    const bool c = s.ly >= sl.b.e[1];
    s.ly -= c ? sl.b.e[1] : 0;
    s.lz += sl.rgz + (c ? 1 : 0);
    s.gi += c ? d2 : d1;
    s.li += c ? l2 : l1;
}

// values of the current quad (0 outside the volume)
template <bool CHECK>
__device__ __forceinline__ quad stage_value(const Stage& s, const Slab& sl, const float* __restrict__ vol, const VolDims& v)
{
    // (CHECK false: the caller knows the box lies inside the volume)
    if (!CHECK) return *reinterpret_cast<const quad*>(vol + s.gi);
    quad r = {0.0f, 0.0f, 0.0f, 0.0f};
    if ((unsigned)(sl.b.o[1] + s.ly) < (unsigned)v.ny && (unsigned)(sl.b.o[2] + s.lz) < (unsigned)v.nz) {
        if (s.gx >= 0 && s.gx + 3 < v.nx) {
            r = *reinterpret_cast<const quad*>(vol + s.gi);
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if ((unsigned)(s.gx + c) < (unsigned)v.nx) r[c] = vol[s.gi + (unsigned)c];
        }
    }
    return r;
}

// element i of a box wider than 1024 along x
__device__ __forceinline__ float element_value(const float* __restrict__ vol, const VolDims& v, const Box& b, int i,
                                               int& li)
{
    const float r0 = 1.0f / (float)b.e[0], r1 = 1.0f / (float)b.e[1];
    const int q = (int)__builtin_floorf(((float)i + 0.5f) * r0);
    const int lx = i - (int)__umul24(q, b.e[0]);
    const int lz = (int)__builtin_floorf(((float)q + 0.5f) * r1);
    const int ly = q - (int)__umul24(lz, b.e[1]);
    const int gx = b.o[0] + lx, gy = b.o[1] + ly, gz = b.o[2] + lz;
    li = lz * b.wz + ly * b.w + lx;
    float val = 0.0f;
    if ((unsigned)gx < (unsigned)v.nx && (unsigned)gy < (unsigned)v.ny && (unsigned)gz < (unsigned)v.nz)
        val = vol[(__umul24((unsigned)gz, (unsigned)v.ny) + (unsigned)gy) * (unsigned)v.nx + (unsigned)gx];
    return val;
}

// the box lies inside the volume (no staged cell needs a bounds check)
__device__ __forceinline__ bool box_inside(const Box& b, const VolDims& v)
{
    return b.o[0] >= 0 && b.o[1] >= 0 && b.o[2] >= 0 && b.o[0] + b.e[0] <= v.nx && b.o[1] + b.e[1] <= v.ny &&
           b.o[2] + b.e[2] <= v.nz;
}

// The first PF passes of a box go through registers: the loads are issued
// together (by the interpolated projector a slab ahead, while the current slab
// is sampled), then written to LDS; any further passes are loaded when the box
// is written.
template <int PF>
struct Fetched {
    quad v[PF];
    int li[PF];   // LDS index, negative where there is nothing to write
};

template <int PF, bool CHECK>
__device__ __forceinline__ void fetch_passes(Fetched<PF>& r, Stage s, const Slab& sl, const float* __restrict__ vol,
                                             const VolDims& v)
{
#pragma unroll
    for (int m = 0; m < PF; ++m) {
        r.v[m] = quad{0.0f, 0.0f, 0.0f, 0.0f};
        r.li[m] = -1;
        if (s.lz < sl.b.e[2]) {
            r.v[m] = stage_value<CHECK>(s, sl, vol, v);
            r.li[m] = s.li;
        }
        if (m + 1 < PF) stage_step(s, sl, v);
    }
}

template <int PF>
__device__ __forceinline__ void fetch_box(Fetched<PF>& r, const float* __restrict__ vol, const VolDims& v, const Slab& sl)
{
    if (!sl.rg) return;
    const Stage s = stage_of(sl, v, 0);
    if (box_inside(sl.b, v))
        fetch_passes<PF, false>(r, s, sl, vol, v);
    else
        fetch_passes<PF, true>(r, s, sl, vol, v);
}

template <int PF>
__device__ __forceinline__ void put_box(float* box, const Fetched<PF>& r, const float* __restrict__ vol, const VolDims& v,
                                        const Slab& sl, int a)
{
    if (!sl.rg) {
        const int n = sl.b.e[0] * sl.b.e[1] * sl.b.e[2];
        for (int i = threadIdx.x; i < n; i += blockDim.x) {
            int li;
            const float val = element_value(vol, v, sl.b, i, li);
            box[li] = val;
        }
        return;
    }
    if (a == 0) {
#pragma unroll
        for (int m = 0; m < PF; ++m)
            if (r.li[m] >= 0) *reinterpret_cast<quad*>(box + r.li[m]) = r.v[m];
    } else {
#pragma unroll
        for (int m = 0; m < PF; ++m)
            if (r.li[m] >= 0) *reinterpret_cast<quad16*>(box + r.li[m]) = r.v[m];
    }
    if (PF * sl.rg < sl.b.e[1] * sl.b.e[2]) {
        const bool in = box_inside(sl.b, v);
        for (Stage s = stage_of(sl, v, PF); s.lz < sl.b.e[2]; stage_step(s, sl, v))
            *reinterpret_cast<quad*>(box + s.li) = in ? stage_value<false>(s, sl, vol, v) : stage_value<true>(s, sl, vol, v);
    }
}

// LDS addresses kept in FP32: the float n 2^-149 (a denormal, at full rate here)
// has the integer n as its bits, so an address formed by exact fused multiply-adds
// on such floats is read without a conversion.
typedef const __attribute__((address_space(3))) float lds_float;
__device__ __forceinline__ unsigned lds_address(const float* p)
{
    return (unsigned)(uintptr_t)(__attribute__((address_space(3))) const char*)p;
}
__device__ __forceinline__ lds_float* lds_at(unsigned address) { return (lds_float*)(uintptr_t)address; }

// ------------------------------------------------------------------ Siddon
// The Siddon sum is taken one layer at a time along the tile's dominant
// axis a (a layer is one cell thick along a; the two other axes are b and
// c).  Inside a layer a ray whose direction has |d_b| and |d_c| below
// 0.99 |d_a| crosses at most one plane of b and one of c, so it passes
// through at most three cells; the three lengths follow from the two next
// crossing parameters by a min, a max and two clamps, and the three cells
// from which crossings fall inside the layer.  Every lane of a wave then
// does the same work per layer (no data-dependent branch), instead of one
// loop trip per crossing with the crossing axis chosen per lane.  The
// crossing parameters are the plane-by-plane walk's (plane q at q inv + c,
// FP32), so the lengths are that walk's, in the same cells.
//
// Two cases leave the three-cell form: a tile holding a ray steeper than
// 0.99 along b or c (it may cross two planes of one axis in a layer) and a
// ray whose path through a slab leaves the staged box (a box clipped to the
// LDS capacity).  Those lanes walk the layer plane by plane, reading cells
// outside the box from global memory.
__device__ __forceinline__ float sid_cell(const float* box, const float* __restrict__ vol, const VolDims& v,
                                          const Box& bx, int x, int y, int z)
{
    const int lx = x - bx.o[0], ly = y - bx.o[1], lz = z - bx.o[2];
    if ((unsigned)lx < (unsigned)bx.e[0] && (unsigned)ly < (unsigned)bx.e[1] && (unsigned)lz < (unsigned)bx.e[2])
        return box[lz * bx.wz + ly * bx.w + lx];
    if ((unsigned)x < (unsigned)v.nx && (unsigned)y < (unsigned)v.ny && (unsigned)z < (unsigned)v.nz)
        return vol[(__umul24((unsigned)z, (unsigned)v.ny) + (unsigned)y) * (unsigned)v.nx + (unsigned)x];
    return 0.0f;
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

// One ray's position in the layer walk: current parameter, end of the
// clipped ray, and per non-dominant axis the plane coordinate of the next
// crossing (an exact integer in FP32) with its parameter.
struct LayerRay {
    float acur, aend, qb, qc, anb, anc, acc;
};

// Plane-by-plane walk of one layer (cell k along a) up to parameter ae.
__device__ __forceinline__ void walk_layer(LayerRay& r, float ae, int k, int a, const SiddonAxis& B,
                                           const SiddonAxis& C, const float* box, const float* __restrict__ vol,
                                           const VolDims& v, const Box& bx)
{
    // at most two crossings of each of b and c fall inside one layer of a
    // ray that runs within 45 degrees of a (the tile's dominant axis); the
    // bound only caps the loop
    for (int it = 0; it < 8 && r.acur < ae; ++it) {
        const float an = fminf(fminf(r.anb, r.anc), ae);
        const int ib = (int)r.qb - (B.step > 0), ic = (int)r.qc - (C.step > 0);
        const int x = a == 0 ? k : ib, y = a == 1 ? k : (a == 0 ? ib : ic), z = a == 2 ? k : ic;
        r.acc = __builtin_fmaf(an - r.acur, sid_cell(box, vol, v, bx, x, y, z), r.acc);
        r.acur = an;
        if (an >= ae) break;
        if (r.anb <= r.anc) {
            r.qb += (float)B.step;
            r.anb = __builtin_fmaf(r.qb, B.inv, B.c);
        } else {
            r.qc += (float)C.step;
            r.anc = __builtin_fmaf(r.qc, C.inv, C.c);
        }
    }
    r.acur = ae;
}

__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(CTMI_FWD_SID_WAVES, 8))) k_forward_siddon(const float* __restrict__ vol, float* __restrict__ proj,
                                                        const ViewGeo* __restrict__ tab,
                                                        const ViewGeo64* __restrict__ tab64, int view0, TileMap m,
                                                        VolDims v, DetDims det, int cap)
{
    extern __shared__ __attribute__((aligned(16))) float box[];   // cap floats
    __shared__ int4 sbox[SLABTAB][2];   // the first SLABTAB slabs
    __shared__ int thick;               // planes per slab
    int view, tu0, tv0;
    tile_of_block(m, blockIdx.x, view, tu0, tv0);
    const int iu = tu0 + (int)(threadIdx.x % TU), iv = tv0 + (int)(threadIdx.x / TU);
    const bool active = iu < det.nu && iv < det.nv;
    const ViewGeo& g = tab[view0 + view];

    float S[3], d[3], a_lo, a_hi;
    siddon_ray(tab64[view0 + view], active ? iu : 0, active ? iv : 0, v, S, d, a_lo, a_hi);
    const float L = world_length(d, v);
    const SiddonAxis ax = siddon_axis(S[0], d[0]);
    const SiddonAxis ay = siddon_axis(S[1], d[1]);
    const SiddonAxis az = siddon_axis(S[2], d[2]);
    float amin = a_lo, amax = a_hi;
    bool hit = slab_clip(ax, S[0], 0.0f, (float)v.nx, amin, amax);
    hit &= slab_clip(ay, S[1], 0.0f, (float)v.ny, amin, amax);
    hit &= slab_clip(az, S[2], 0.0f, (float)v.nz, amin, amax);
    const bool alive = active && hit && amin < amax;

    int a, dir;
    tile_axis(g, det, tu0, tv0, a, dir);
    const int b = a == 0 ? 1 : 0, c = a == 2 ? 1 : 2;
    const SiddonAxis A = pick_axis(a, ax, ay, az), B = pick_axis(b, ax, ay, az), C = pick_axis(c, ax, ay, az);
    const float Sa = pick3(a, S[0], S[1], S[2]), Da = pick3(a, d[0], d[1], d[2]);
    const float Sb = pick3(b, S[0], S[1], S[2]), Db = pick3(b, d[0], d[1], d[2]);
    const float Sc = pick3(c, S[0], S[1], S[2]), Dc = pick3(c, d[0], d[1], d[2]);
    const int na = pick3(a, v.nx, v.ny, v.nz), nb = pick3(b, v.nx, v.ny, v.nz), nc = pick3(c, v.nx, v.ny, v.nz);

    // a ray that runs against the tile's direction along a (only possible
    // at extreme fan angles) is walked plane by plane from global memory at
    // the end instead
    const bool odd = alive && A.step != dir;
    const bool lay = alive && !odd;
    LayerRay r;
    r.acc = 0.0f;
    r.acur = lay ? amin : 0.0f;
    r.aend = lay ? amax : 0.0f;
    {
        const int ib = ordered_cell(B, Sb, Db, amin, 0, nb), ic = ordered_cell(C, Sc, Dc, amin, 0, nc);
        r.qb = (float)(ib + (B.step > 0));
        r.qc = (float)(ic + (C.step > 0));
        // a parallel axis has inv = 0 and c = inf, so its crossings stay at inf
        r.anb = lay ? __builtin_fmaf(r.qb, B.inv, B.c) : CTMI_INF;
        r.anc = lay ? __builtin_fmaf(r.qc, C.inv, C.c) : CTMI_INF;
    }
    // the wave's layer range (cells along a that some lane's ray reaches)
    int klo = 0x7fffffff, khi = -1;
    if (lay) {
        const float p0 = __builtin_fmaf(amin, Da, Sa), p1 = __builtin_fmaf(amax, Da, Sa);
        klo = max((int)__builtin_floorf(fminf(p0, p1)) - 1, 0);
        khi = min((int)__builtin_floorf(fmaxf(p0, p1)) + 1, na - 1);
    }
    const int kmin = klo, kmax = khi;   // this ray's own (its layers only: a length of 0 in any other times a NaN would count)
    // the three-cell form needs every ray of the wave below 0.99 along b and c
    bool steep = lay && (fabsf(Db) > 0.99f * fabsf(Da) || fabsf(Dc) > 0.99f * fabsf(Da));
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        klo = min(klo, __shfl_xor(klo, off));
        khi = max(khi, __shfl_xor(khi, off));
    }
    // (the same in every lane now: keep them in scalar registers)
    klo = __builtin_amdgcn_readfirstlane(klo);
    khi = __builtin_amdgcn_readfirstlane(khi);
    const bool wave_steep = __any(steep);

    int slab = 0, nslab = 0;
    const int clo[3] = {0, 0, 0}, chi[3] = {v.nx - 1, v.ny - 1, v.nz - 1};
    // the staged box of slab si (in the direction of travel): the cells
    // under the bundle, no margin (a ray whose walk rounds into a cell
    // outside, a corner ray within ulps of a plane, finds out below and
    // reads that slab plane by plane)
    auto slab_box = [&](int si) -> Slab {
        const int s = dir > 0 ? si : nslab - 1 - si;
        const int c0 = s * slab, c1 = min(c0 + slab, na);   // cells [c0, c1) along a
        float blo[3], bhi[3];
        bundle_bounds(g, det, tu0, tv0, a, (float)c0, (float)c1, 0.0f, blo, bhi);
        int lo[3], hi[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            lo[i] = (int)__builtin_floorf(fmaxf(blo[i], -4.0f));
            hi[i] = (int)__builtin_floorf(fminf(bhi[i], 1.0e7f));
        }
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            lo[i] = i == a ? c0 : lo[i];
            hi[i] = i == a ? c1 - 1 : hi[i];
        }
        Box bx;
        const int f = make_box(lo, hi, clo, chi, a, cap, bx);
        if (!f) return slab_of_box(Box{{0, 0, 0}, {4, 1, 1}, 4, 4}, 0);
        // (a row rounded up past the volume starts earlier instead)
        bx.o[0] = max(min(bx.o[0], v.nx - bx.e[0]), 0);
        return slab_of_box(bx, f);
    };
    // the first wave picks the slab thickness and forms the boxes, one per lane
    // (not every wave at every slab)
    if (threadIdx.x < 64) {
        Slab mine;
        for (int c = 0; c < NTHICK; ++c) {
            slab = siddon_thickness(c);
            nslab = (na + slab - 1) / slab;
            mine = slab_box((int)threadIdx.x);
            bool cut = (int)threadIdx.x < nslab && (mine.flags & BOX_CLIPPED);
            for (int si = (int)threadIdx.x + 64; si < nslab; si += 64) cut |= (slab_box(si).flags & BOX_CLIPPED) != 0;
            if (!__any(cut)) break;
        }
        if ((int)threadIdx.x < min(nslab, SLABTAB)) put_slab(sbox[threadIdx.x], mine);
        if (threadIdx.x == 0) thick = slab;
    }
    __syncthreads();
    slab = __builtin_amdgcn_readfirstlane(thick);
    nslab = (na + slab - 1) / slab;

    for (int si = 0; si < nslab; ++si) {
        const int s = dir > 0 ? si : nslab - 1 - si;
        const int c0 = s * slab, c1 = min(c0 + slab, na);   // cells [c0, c1) along a
        Slab sl;
        if (si < SLABTAB) {
            sl = get_slab(sbox[si], a);
        } else {
            int4 row[2];
            put_slab(row, slab_box(si));
            sl = get_slab(row, a);   // (the same in every lane: scalar registers)
        }
        if (!sl.flags) continue;
        const Box& bx = sl.b;
        __syncthreads();
        {
            Fetched<CTMI_FWD_SID_PF> q;
            fetch_box<CTMI_FWD_SID_PF>(q, vol, v, sl);
            put_box<CTMI_FWD_SID_PF>(box, q, vol, v, sl, a);
        }
        __syncthreads();
        const int k0 = max(c0, klo), k1 = min(c1 - 1, khi);
        if (k0 > k1) continue;   // no ray of this wave reaches these layers

        // box strides (elements) and origins of the three axes
        const int st_a = pick3(a, 1, bx.w, bx.wz);
        const int st_b = pick3(b, 1, bx.w, bx.wz);
        const int st_c = pick3(c, 1, bx.w, bx.wz);
        const int oa = pick3(a, bx.o[0], bx.o[1], bx.o[2]);
        const int ob = pick3(b, bx.o[0], bx.o[1], bx.o[2]), eb = pick3(b, bx.e[0], bx.e[1], bx.e[2]);
        const int oc = pick3(c, bx.o[0], bx.o[1], bx.o[2]), ec = pick3(c, bx.e[0], bx.e[1], bx.e[2]);
        // does this ray's path through the slab stay inside the box?  Its
        // cells along b (and c) run monotonically from its current one to
        // the one it holds at the end of its stretch here, which
        // ordered_cell gives in the walk's crossing order; a ray with no
        // stretch here sits the slab out
        bool inbox = true, idle = true;
        int roff = 0;   // byte offset of the ray's (b, c) cell in a layer of the box
        {
            const float s0 = __builtin_fmaf((float)c0, A.inv, A.c), s1 = __builtin_fmaf((float)c1, A.inv, A.c);
            const float t0 = fmaxf(fminf(s0, s1), r.acur), t1 = fminf(fmaxf(s0, s1), r.aend);
            const int ib = (int)r.qb - (B.step > 0), ic = (int)r.qc - (C.step > 0);
            if (t0 < t1) {
                idle = false;
                const int ibe = ordered_cell(B, Sb, Db, t1, 0, nb), ice = ordered_cell(C, Sc, Dc, t1, 0, nc);
                inbox = min(ib, ibe) >= ob && max(ib, ibe) < ob + eb && min(ic, ice) >= oc && max(ic, ice) < oc + ec;
                roff = inbox ? 4 * ((ib - ob) * st_b + (ic - oc) * st_c) : 0;
            }
        }
        // layers, and the first in the direction of travel
        const int l0 = max(c0, kmin), l1 = min(c1 - 1, kmax), n = idle ? 0 : l1 - l0 + 1, kf = dir > 0 ? l0 : l1;
        if (inbox && !wave_steep) {
            // The three-cell form, 26 VALU per layer.  o is the LDS address of the
            // ray's cell in FP32 (lds_at); plane numbers and steps are exact too.  No
            // crossing lies before acur (ordered_cell), so no length is negative.
            const float DB = __int_as_float(4 * st_b), DC = __int_as_float(4 * st_c);
            const float DA = dir > 0 ? __int_as_float(4 * st_a) : -__int_as_float(4 * st_a);
            const float fdir = (float)dir, sb = (float)B.step, sc = (float)C.step;
            float o = __int_as_float((int)lds_address(box) + roff + 4 * (kf - oa) * st_a);
            float q = (float)(kf + (dir > 0));
#pragma unroll 4
            for (int i = 0; i < n; ++i) {
                const float ae = __builtin_amdgcn_fmed3f(__builtin_fmaf(q, A.inv, A.c), r.acur, r.aend);   // exit plane
                const bool bfirst = r.anb <= r.anc;
                const float t1 = fminf(fminf(r.anb, r.anc), ae), t2 = fminf(fmaxf(r.anb, r.anc), ae);
                const float fb = r.anb < ae ? sb : 0.0f, fc = r.anc < ae ? sc : 0.0f;
                const float ob1 = __builtin_fmaf(fb, DB, o), oc1 = __builtin_fmaf(fc, DC, o);
                const float o2 = __builtin_fmaf(fc, DC, ob1);
                const float v0 = *lds_at(__float_as_uint(o));
                const float v1 = *lds_at(__float_as_uint(bfirst ? ob1 : oc1));
                const float v2 = *lds_at(__float_as_uint(o2));
                r.acc = __builtin_fmaf(t1 - r.acur, v0, r.acc);
                r.acc = __builtin_fmaf(t2 - t1, v1, r.acc);
                r.acc = __builtin_fmaf(ae - t2, v2, r.acc);
                r.acur = ae;
                o = o2 + DA;
                q += fdir;
                r.qb += fb;
                r.qc += fc;
                r.anb = __builtin_fmaf(r.qb, B.inv, B.c);
                r.anc = __builtin_fmaf(r.qc, C.inv, C.c);
            }
        } else {
            for (int i = 0; i < n; ++i) {
                const int k = kf + i * dir;
                const float aa = __builtin_fmaf((float)(k + (dir > 0)), A.inv, A.c);   // exit plane of layer k
                walk_layer(r, __builtin_amdgcn_fmed3f(aa, r.acur, r.aend), k, a, B, C, box, vol, v, bx);
            }
        }
    }
    if (odd) {
        // plane-by-plane walk over the whole ray from global memory
        int ix = ordered_cell(ax, S[0], d[0], amin, 0, v.nx);
        int iy = ordered_cell(ay, S[1], d[1], amin, 0, v.ny);
        int iz = ordered_cell(az, S[2], d[2], amin, 0, v.nz);
        float qx = (float)(ix + (ax.step > 0)), qy = (float)(iy + (ay.step > 0)), qz = (float)(iz + (az.step > 0));
        float anx = plane_alpha(ax, qx), any = plane_alpha(ay, qy), anz = plane_alpha(az, qz);
        float acur = amin;
        for (int left = v.nx + v.ny + v.nz + 3; left > 0; --left) {
            const float an = fminf(anx, fminf(any, anz));
            const float ae = fminf(an, amax);
            r.acc = __builtin_fmaf(fmaxf(ae - acur, 0.0f),
                                   vol[(__umul24((unsigned)iz, (unsigned)v.ny) + (unsigned)iy) * (unsigned)v.nx +
                                       (unsigned)ix],
                                   r.acc);
            if (an >= amax) break;
            acur = an;
            if (an == anx) {
                ix += ax.step;
                if ((unsigned)ix >= (unsigned)v.nx) break;
                qx += (float)ax.step;
                anx = plane_alpha(ax, qx);
            } else if (an == any) {
                iy += ay.step;
                if ((unsigned)iy >= (unsigned)v.ny) break;
                qy += (float)ay.step;
                any = plane_alpha(ay, qy);
            } else {
                iz += az.step;
                if ((unsigned)iz >= (unsigned)v.nz) break;
                qz += (float)az.step;
                anz = plane_alpha(az, qz);
            }
        }
    }
    if (active) proj[((int64_t)view * det.nv + iv) * det.nu + iu] = r.acc * L;
}

// ------------------------------------------------------------ interpolated
__device__ __forceinline__ float lerp1(float a, float r0, float r1) { return __builtin_fmaf(a, r1 - r0, r0); }

// Trilinear sample of the volume at voxel-centre coordinates p, zero outside
// the grid (out-of-grid corners read as 0, indices clamped so every load is
// in bounds).  Same lerp sequence as the LDS path, so both give the same bits.
__device__ __forceinline__ float trilinear_global(const float* __restrict__ vol, const VolDims& v, const float p[3])
{
    const float fx = __builtin_floorf(p[0]), fy = __builtin_floorf(p[1]), fz = __builtin_floorf(p[2]);
    const int ix = (int)fx, iy = (int)fy, iz = (int)fz;
    const float ax = p[0] - fx, ay = p[1] - fy, az = p[2] - fz;
    float r[8];
    if ((unsigned)ix < (unsigned)(v.nx - 1) && (unsigned)iy < (unsigned)(v.ny - 1) && (unsigned)iz < (unsigned)(v.nz - 1)) {
        const float* q = vol + (((int64_t)iz * v.ny + iy) * v.nx + ix);
        const int64_t nxy = (int64_t)v.nx * v.ny;
        const pair p0 = *reinterpret_cast<const pair*>(q), p1 = *reinterpret_cast<const pair*>(q + v.nx);
        const pair p2 = *reinterpret_cast<const pair*>(q + nxy), p3 = *reinterpret_cast<const pair*>(q + nxy + v.nx);
        r[0] = p0.x, r[1] = p0.y, r[2] = p1.x, r[3] = p1.y, r[4] = p2.x, r[5] = p2.y, r[6] = p3.x, r[7] = p3.y;
    } else
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        const int jx = ix + (c & 1), jy = iy + ((c >> 1) & 1), jz = iz + (c >> 2);
        const bool in = (unsigned)jx < (unsigned)v.nx && (unsigned)jy < (unsigned)v.ny && (unsigned)jz < (unsigned)v.nz;
        const int cx = min(max(jx, 0), v.nx - 1), cy = min(max(jy, 0), v.ny - 1), cz = min(max(jz, 0), v.nz - 1);
        const float val = vol[((int64_t)cz * v.ny + cy) * v.nx + cx];
        r[c] = in ? val : 0.0f;
    }
    const float c00 = lerp1(ax, r[0], r[1]), c01 = lerp1(ax, r[2], r[3]);
    const float c10 = lerp1(ax, r[4], r[5]), c11 = lerp1(ax, r[6], r[7]);
    return lerp1(az, lerp1(ay, c00, c01), lerp1(ay, c10, c11));
}

// Per-tile ray-bundle description in LDS: for each corner ray c and axis i,
// the coordinate on plane P of the dominant axis is K[c][i] + P * G[c][i].
struct Bundle {
    float K[4][3], G[4][3];
};

__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(CTMI_FWD_WAVES, 8))) k_forward_interp(const float* __restrict__ vol, float* __restrict__ proj,
                                                        const ViewGeo* __restrict__ tab,
                                                        const ViewGeo64* __restrict__ tab64, int view0, TileMap m,
                                                        VolDims v, DetDims det, float ds, int cap)
{
    extern __shared__ __attribute__((aligned(16))) float box[];   // cap floats
    __shared__ Bundle bun;
    __shared__ int4 sbox[SLABTAB][2];   // the first SLABTAB slabs
    __shared__ int thick;               // planes per slab
    int view, tu0, tv0;
    tile_of_block(m, blockIdx.x, view, tu0, tv0);
    const int iu = tu0 + (int)(threadIdx.x % TU), iv = tv0 + (int)(threadIdx.x / TU);
    const bool active = iu < det.nu && iv < det.nv;
    const ViewGeo& g = tab[view0 + view];
    int a, dir;
    tile_axis(g, det, tu0, tv0, a, dir);
    if (threadIdx.x < 4) {
        // corner rays of the tile, voxel-centre coordinates
        const int c = threadIdx.x;
        const int cu = (c & 1) ? min(tu0 + TU, det.nu) - 1 : tu0, cv = (c & 2) ? min(tv0 + TV, det.nv) - 1 : tv0;
        float S[3], d[3];
        pixel_ray(g, cu, cv, S, d);
        const float inv = 1.0f / d[a];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const float Gi = d[i] * inv;
            bun.G[c][i] = Gi;
            bun.K[c][i] = (S[i] - 0.5f) - (S[a] - 0.5f) * Gi;
        }
    }

    InterpRay r;
    const bool has = interp_ray(tab64[view0 + view], active ? iu : 0, active ? iv : 0, v, ds, 1.0f / ds, r) && active;
    int k = has ? r.k0 : 0;
    int k1 = has ? r.k1 : -1;
    if (ds > fminf(v.hx, fminf(v.hy, v.hz))) {
        // the samples one step beyond the support lie further out than the
        // boxes' margin of one voxel: they add nothing, so the range ends here
        auto outside = [&](int j) {
            float p[3];
            interp_pos(r, j, p);
            return p[0] < -2.0f || p[1] < -2.0f || p[2] < -2.0f || p[0] >= (float)(v.nx + 1) ||
                   p[1] >= (float)(v.ny + 1) || p[2] >= (float)(v.nz + 1);
        };
        while (k <= k1 && outside(k)) ++k;
        while (k <= k1 && outside(k1)) --k1;
    }
    // sample k sits at base + (k - kc) st; along the dominant axis the slab
    // boundary plane P is reached at (k - kc) = (P - base_a) / st_a
    const float sa = a == 0 ? r.st[0] : (a == 1 ? r.st[1] : r.st[2]);
    const float ba = a == 0 ? r.base[0] : (a == 1 ? r.base[1] : r.base[2]);
    // the slab bookkeeping needs the ray to advance along the tile's direction
    // (always true for tile-sized bundles); any other ray takes the checked
    // path in the first slab
    const bool mono = dir > 0 ? sa > 1e-6f : sa < -1e-6f;
    const float inv_sa = mono ? 1.0f / sa : 0.0f;
    float acc = 0.0f;
    __syncthreads();

    const int na = a == 0 ? v.nx : (a == 1 ? v.ny : v.nz);
    // a sample's lower corner A = floor(pos_a) lies in [-2, n] (the sample
    // range reaches one step beyond the interpolant's support, and FP32
    // positions may round across its edge); slab s takes the samples before
    // the plane s slab + slab - 1 (direction +) or from the plane s slab - 1
    // on (direction -), and stages planes [s slab - 2, s slab + slab] so a
    // sample assigned one step early or late by rounding still finds its
    // corners in the box.  Boxes may reach one plane of zeros beyond each
    // halo plane, so every corner of such a sample is staged.
    int slab = 0, nslab = 0;
    const int clo[3] = {-2, -2, -2}, chi[3] = {v.nx + 1, v.ny + 1, v.nz + 1};

    // slab si's plane range [A0, A1], its staged box and whether the box
    // holds the whole bundle range (uniform over the block)
    auto slab_box = [&](int si) -> Slab {
        const int s = dir > 0 ? si : nslab - 1 - si;
        const int A0 = s * slab - 1, A1 = A0 + slab;
        // bundle bounds over the staged plane range [A0 - 1, A1 + 1]
        float blo[3] = {CTMI_INF, CTMI_INF, CTMI_INF}, bhi[3] = {-CTMI_INF, -CTMI_INF, -CTMI_INF};
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const float x0 = __builtin_fmaf((float)(A0 - 1), bun.G[c][i], bun.K[c][i]);
                const float x1 = __builtin_fmaf((float)(A1 + 1), bun.G[c][i], bun.K[c][i]);
                blo[i] = fminf(blo[i], fminf(x0, x1));
                bhi[i] = fmaxf(bhi[i], fmaxf(x0, x1));
            }
        int lo[3], hi[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            lo[i] = (int)__builtin_floorf(fmaxf(blo[i], -4.0f)) - 1;
            hi[i] = (int)__builtin_floorf(fminf(bhi[i], 1.0e7f)) + 2;
        }
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            lo[i] = i == a ? A0 - 1 : lo[i];
            hi[i] = i == a ? A1 + 1 : hi[i];
        }
        Box b;
        const int f = make_box(lo, hi, clo, chi, a, cap, b);
        return f ? slab_of_box(b, f) : slab_of_box(Box{{0, 0, 0}, {4, 1, 1}, 4, 4}, 0);
    };
    // the first wave picks the slab thickness and forms the boxes, one per lane
    // (not every wave at every slab)
    if (threadIdx.x < 64) {
        Slab mine;
        for (int c = 0; c < NTHICK; ++c) {
            slab = interp_thickness(a, c);
            nslab = (na + slab) / slab;
            mine = slab_box((int)threadIdx.x);
            bool cut = (int)threadIdx.x < nslab && (mine.flags & BOX_CLIPPED);
            for (int si = (int)threadIdx.x + 64; si < nslab; si += 64) cut |= (slab_box(si).flags & BOX_CLIPPED) != 0;
            if (!__any(cut)) break;
        }
        if ((int)threadIdx.x < min(nslab, SLABTAB)) put_slab(sbox[threadIdx.x], mine);
        if (threadIdx.x == 0) thick = slab;
    }
    __syncthreads();
    slab = __builtin_amdgcn_readfirstlane(thick);
    nslab = (na + slab) / slab;
    auto slab_of = [&](int si) -> Slab {
        if (si < SLABTAB) return get_slab(sbox[si], a);
        int4 row[2];
        put_slab(row, slab_box(si));
        return get_slab(row, a);   // (the same in every lane: scalar registers)
    };
    // the next slab's box is fetched into registers while this one is sampled
    constexpr int PF = CTMI_FWD_PF;
    Fetched<PF> pf;
    Slab next = slab_of(0);
    if (next.flags & BOX_SOME) fetch_box<PF>(pf, vol, v, next);

    for (int si = 0; si < nslab; ++si) {
        const Slab sl = next;
        const Box& b = sl.b;
        const bool fits = (sl.flags & BOX_SOME) != 0, clipped = (sl.flags & BOX_CLIPPED) != 0;
        const int A0 = (dir > 0 ? si : nslab - 1 - si) * slab - 1, A1 = A0 + slab;
        // this thread's last sample in the slab
        int kl;
        {
            const float P = dir > 0 ? (float)A1 : (float)A0;
            const float t = (P - ba) * inv_sa;
            kl = r.kc + (dir > 0 ? (int)__builtin_ceilf(t) - 1 : (int)__builtin_floorf(t));
            kl = (si == nslab - 1 || !mono) ? k1 : min(kl, k1);
        }
        __syncthreads();
        if (fits) put_box<PF>(box, pf, vol, v, sl, a);
        __syncthreads();
        if (si + 1 < nslab) {
            next = slab_of(si + 1);
            if (next.flags & BOX_SOME) fetch_box<PF>(pf, vol, v, next);
        }
        if (fits && !clipped && mono) {
            // fast path: every sample of the slab has its 2x2x2 corners in the box.
            // The LDS address is formed in FP32 as a multiple of 2^-149 (see
            // lds_at).
            const float SX = __int_as_float(4), SY = __int_as_float(4 * b.w), SZ = __int_as_float(4 * b.wz);
            const unsigned o01 = 4 * (unsigned)b.w, o10 = 4 * (unsigned)b.wz, o11 = o10 + o01;
            // samples k..kl by their offset j = k - kc from the ray's anchor, an
            // exact FP32 integer (interp_pos's position, without an int->float
            // conversion per sample).  Only a ray with samples here enters: its
            // offsets are below its sample count, far below 2^24, so the FP32
            // counter steps exactly and the loop ends.
            const float jl = (float)(kl - r.kc);
            auto samples = [&](float ox, float oy, float oz, float C) {
                for (float j = (float)(k - r.kc); k <= kl && j <= jl; j += 1.0f) {
                    float p[3];
#pragma unroll
                    for (int i = 0; i < 3; ++i) p[i] = __builtin_fmaf(j, r.st[i], r.base[i]);
                    const float fx = __builtin_floorf(p[0]), fy = __builtin_floorf(p[1]), fz = __builtin_floorf(p[2]);
                    const unsigned off = __float_as_uint(
                        __builtin_fmaf(fz - oz, SZ, __builtin_fmaf(fy - oy, SY, __builtin_fmaf(fx - ox, SX, C))));
                    const lds_float *r0 = lds_at(off), *r1 = lds_at(off + o01), *r2 = lds_at(off + o10),
                                    *r3 = lds_at(off + o11);
                    const float ax = p[0] - fx, ay = p[1] - fy, az = p[2] - fz;
                    const float c00 = lerp1(ax, r0[0], r0[1]), c01 = lerp1(ax, r1[0], r1[1]);
                    const float c10 = lerp1(ax, r2[0], r2[1]), c11 = lerp1(ax, r3[0], r3[1]);
                    acc += lerp1(az, lerp1(ay, c00, c01), lerp1(ay, c10, c11));
                }
            };
            const int at = (int)lds_address(box);
            // The box's origin is the first product's addend where byte offsets
            // over the whole grid and its margins stay exact FP32 integers;
            // elsewhere (some thousand planes with wide boxes) it is taken off
            // each coordinate, three instructions per sample more.
            if ((int64_t)b.wz * (v.nz + 4) + (int64_t)b.w * (v.ny + 4) + v.nx + 4 < 1 << 22)
                samples(0.0f, 0.0f, 0.0f, (float)(at - 4 * (b.o[0] + b.w * b.o[1] + b.wz * b.o[2])) * 0x1p-149f);
            else
                samples((float)b.o[0], (float)b.o[1], (float)b.o[2], (float)at * 0x1p-149f);
            k = max(k, kl + 1);
        } else {
            for (; k <= kl; ++k) {
                float p[3];
                interp_pos(r, k, p);
                const float fx = __builtin_floorf(p[0]), fy = __builtin_floorf(p[1]), fz = __builtin_floorf(p[2]);
                const int lx = (int)fx - b.o[0], ly = (int)fy - b.o[1], lz = (int)fz - b.o[2];
                if (fits && (unsigned)lx < (unsigned)(b.e[0] - 1) && (unsigned)ly < (unsigned)(b.e[1] - 1) &&
                    (unsigned)lz < (unsigned)(b.e[2] - 1)) {
                    const float* q = box + lz * b.wz + ly * b.w + lx;
                    const int sy = b.w, sz = b.wz;
                    const float ax = p[0] - fx, ay = p[1] - fy, az = p[2] - fz;
                    const float c00 = lerp1(ax, q[0], q[1]), c01 = lerp1(ax, q[sy], q[sy + 1]);
                    const float c10 = lerp1(ax, q[sz], q[sz + 1]), c11 = lerp1(ax, q[sz + sy], q[sz + sy + 1]);
                    acc += lerp1(az, lerp1(ay, c00, c01), lerp1(ay, c10, c11));
                } else {
                    acc += trilinear_global(vol, v, p);
                }
            }
        }
    }
    for (; k <= k1; ++k) {   // anything left (never expected) reads global memory
        float p[3];
        interp_pos(r, k, p);
        acc += trilinear_global(vol, v, p);
    }
    if (active) proj[((int64_t)view * det.nv + iv) * det.nu + iu] = acc * ds;
}

TileMap tile_map(const Plan& p, int64_t nviews)
{
    TileMap m;
    m.tiles_u = (p.det.nu + TU - 1) / TU;
    m.tiles_v = (p.det.nv + TV - 1) / TV;
    m.nviews = nviews;
    return m;
}

}  // namespace

// LDS floats for a workgroup's box: six, five, four or two workgroups per CU (the
// Siddon walk's registers allow five).  A wider box costs wavefronts in flight, a
// narrower one thin slabs, and clipped boxes where pixels span several voxels.
// The lines lie where neighbours measured equal on cubes of 256 voxels, 24 views, by
// voxels per pixel (interpolated, us at 6144 / 7424 / 9472 / 15360 floats: 0.75:
// 1617 1670 1777 2894; 0.98: 1287 1220 1298 1972; 1.17: 1640 1377 1207 1628; 1.69: 3083
// 2500 1824 1637; Siddon 0.65: 1211 1185 1276 2124; 1.43: 809 668 649 835; 2.6 (128
// planes): 473 487 475 662; 3.9 (24 x 256 x 48): 125 123 127 106).
static int box_capacity(const Plan& p, bool siddon)
{
    if (p.tile_area <= (siddon ? 790.0f : 540.0f)) return siddon ? 7424 : 6144;
    if (p.tile_area <= 790.0f) return 7424;
    return p.tile_area <= (siddon ? 5000.0f : 1450.0f) ? 9472 : BOXCAP_MAX;
}

hipError_t launch_forward_siddon(const Plan& p, const float* vol, float* proj, int64_t view0, int64_t nviews,
                                 hipStream_t s)
{
    const TileMap m = tile_map(p, nviews);
    const int64_t blocks = (int64_t)m.tiles_u * m.tiles_v * nviews;
    const int cap = box_capacity(p, true);
    hipLaunchKernelGGL(k_forward_siddon, dim3((unsigned)blocks), dim3(256), cap * sizeof(float), s, vol, proj, p.d_views, p.d_views64,
                       (int)view0, m, p.vol, p.det, cap);
    return hipGetLastError();
}

hipError_t launch_forward_interp(const Plan& p, const float* vol, float* proj, int64_t view0, int64_t nviews,
                                 hipStream_t s)
{
    const TileMap m = tile_map(p, nviews);
    const int64_t blocks = (int64_t)m.tiles_u * m.tiles_v * nviews;
    const int cap = box_capacity(p, false);
    hipLaunchKernelGGL(k_forward_interp, dim3((unsigned)blocks), dim3(256), cap * sizeof(float), s, vol, proj, p.d_views, p.d_views64,
                       (int)view0, m, p.vol, p.det, p.ds, cap);
    return hipGetLastError();
}

}  // namespace ctmi
