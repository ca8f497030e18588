// What the two forms of the matched adjoints share (backward.hip, backward_few.hip):
// the bricks, the footprints' margin, the shells' layout and the fixed point.
#pragma once

#include "ctmi_internal.h"

namespace ctmi {

namespace {

constexpr int BX = CTMI_BWD_BX, BY = CTMI_BWD_BY;   // brick extents along x and y

struct BrickMap {
    int nbx, nby, nbz;
};

__device__ __forceinline__ void brick_origin(const BrickMap& m, int b, int& bx, int& by, int& bz)
{
    bx = b % m.nbx;
    const int r = b / m.nbx;
    by = r % m.nby;
    bz = r / m.nby;
}

inline BrickMap brick_map(const Plan& p, int BZ)
{
    BrickMap m;
    m.nbx = (p.vol.nx + BX - 1) / BX;
    m.nby = (p.vol.ny + BY - 1) / BY;
    m.nbz = (p.vol.nz + BZ - 1) / BZ;
    return m;
}

// Pixels whose rays may cross a box whose corners project into [umin, umax] x [vmin,
// vmax]: the pixel centres in that rectangle (the box's silhouette is the corners'
// convex hull, so a ray through a centre outside it misses the box), widened by
// FOOT_EPS pixel against the FP32 rounding of the projection (about 1e-4 pixel; a ray
// that close to the box lies within 0.01 pixel of it, some 100 FP32 position rounding
// units, so a sample the FP32 walk might still place in the box is never left out),
// clamped to the detector; empty when u0 > u1 or v0 > v1.
constexpr float FOOT_EPS = 0.01f;
__device__ __forceinline__ void foot_pixels(float umin, float umax, float vmin, float vmax, const DetDims& det, int& u0,
                                            int& u1, int& v0, int& v1)
{
    // clamp in float first: the corners may project far outside the detector
    umin = fminf(fmaxf(umin, -2.0f), (float)det.nu + 1.0f);
    vmin = fminf(fmaxf(vmin, -2.0f), (float)det.nv + 1.0f);
    umax = fminf(fmaxf(umax, -2.0f), (float)det.nu + 1.0f);
    vmax = fminf(fmaxf(vmax, -2.0f), (float)det.nv + 1.0f);
    u0 = max((int)__builtin_ceilf(umin - FOOT_EPS), 0);
    v0 = max((int)__builtin_ceilf(vmin - FOOT_EPS), 0);
    u1 = min((int)__builtin_floorf(umax + FOOT_EPS), det.nu - 1);
    v1 = min((int)__builtin_floorf(vmax + FOOT_EPS), det.nv - 1);
}

// Fixed-point scale: the exponent e of the largest power of two (up to exact powers of
// two) with 2^e c m <= 2^30, c > 0 (what one ray adds at most) and m > 0 (values).  Formed from the operands' exponents, so neither a product nor a
// quotient can overflow or underflow: with c = a 2^ec and m = b 2^em (a, b in
// [1/2, 1)), 2^(30 - ec - em) c m = 2^30 a b < 2^30, and one more power of two
// fits when a b < 1/2.  Contributions are scaled by 2^e and the integer sums by
// 2^-e with ldexp (exact), so the fixed point works at every magnitude of y
// that FP32 holds.
__device__ __forceinline__ int fixed_exp(float c, float m)
{
    int ec, em;
    const float a = __builtin_frexpf(c, &ec);
    const float b = __builtin_frexpf(m, &em);
    return 30 - ec - em + (a * b < 0.5f ? 1 : 0);
}

// y for finite y, 0 for NaN and infinities (those rays are handled by
// k_nonfinite after the accumulation)
__device__ __forceinline__ float finite_or_zero(float y)
{
    return __builtin_fabsf(y) <= 0x1.fffffep127f ? y : 0.0f;
}

// floor(q + 1/2) as an int32 in one instruction (rintf costs a round and a
// convert); it differs from round-half-even only on exact ties
__device__ __forceinline__ int round_int(float q)
{
    int r;
    asm("v_cvt_rpi_i32_f32 %0, %1" : "=v"(r) : "v"(q));
    return r;
}

// The brick's voxels, T threads, voxel tid + T m in own[m] (added to beta times the volume)
template <int BZ, int T>
__device__ __forceinline__ void store_owned(float* __restrict__ vol, const float* own, const VolDims& v, int x0,
                                            int y0, int z0, float beta)
{
#pragma unroll
    for (int m = 0; m < BX * BY * BZ / T; ++m) {
        const int i = threadIdx.x + T * m;
        const int gx = x0 + i % BX, gy = y0 + (i / BX) % BY, gz = z0 + i / (BX * BY);
        if (gx >= v.nx || gy >= v.ny || gz >= v.nz) continue;
        float* o = vol + ((int64_t)gz * v.ny + gy) * v.nx + gx;
        *o = beta == 0.0f ? own[m] : __builtin_fmaf(beta, *o, own[m]);
    }
}

// Upper shell of a brick of BZ planes: cells of the x, y and z faces
template <int BZ>
struct Shell {
    static constexpr int SX = (BY + 1) * (BZ + 1), SY = BX * (BZ + 1), SZ = BX * BY, N = SX + SY + SZ;

    static __device__ __forceinline__ void cell(int h, int& lx, int& ly, int& lz)
    {
        if (h < SX) {
            lx = BX;
            ly = h % (BY + 1);
            lz = h / (BY + 1);
        } else if (h < SX + SY) {
            h -= SX;
            lx = h % BX;
            ly = BY;
            lz = h / BX;
        } else {
            h -= SX + SY;
            lx = h % BX;
            ly = h / BX;
            lz = BZ;
        }
    }
};
static_assert(Shell<CTMI_BWD_BZ>::N == CTMI_HALO_SLOTS, "shell of the workspace's brick");

}  // namespace

}  // namespace ctmi
