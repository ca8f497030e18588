// Curved detectors (section 2.4: curved detectors are taken in through a
// flattening transformation): projections measured on a cylindrically
// curved detector are resampled onto the plan's flat detector, after which
// every operator of the flat geometry applies to them.
//
// The arc's axis is parallel to v, at distance R from the flat detector's
// centre towards the source (R = DSD: every pixel of a row equidistant
// from the source); u pixel positions are arc lengths.  A flat pixel's ray
// meets the cylinder at parameter t along source -> flat pixel, the
// positive root of (DSD^2 + u^2) t^2 - 2 DSD (DSD - R) t + (DSD - R)^2 - R^2
// = 0, at arc length R atan2(t u, t DSD - DSD + R) and height t v; the flat
// value is the curved projection there, bilinear between pixel centres and
// 0 outside the curved detector.  The map is the same for every view of a
// circular orbit and for every row of a column except the height, so each
// thread owns FLAT_R pixels of one column, forms its column's arc position and
// each pixel's height once in FP64 (the arc coordinates of a large radius cancel
// heavily), and applies them to its slice of the views; neighbouring lanes hold
// neighbouring columns, so the writes and most reads coalesce.  HBM-bound: one
// read and one write per pixel.  (One thread per view and column, with the heights
// formed again for every view, left most of the chip idle: 91 views of 299 x
// 365 pixels 214 us, 50 us so.)
#include "ctmi_internal.h"

namespace ctmi {

namespace {

constexpr int FLAT_R = 4;   // rows per thread

__global__ void __launch_bounds__(256) k_flatten_curved(const float* __restrict__ curved, float* __restrict__ flat,
                                                        int nviews, FlatDet f, CurvedDet c, double DSD)
{
    const int iu = blockIdx.x * 64 + threadIdx.x % 64;
    if (iu >= f.nu) return;
    const int slices = gridDim.z;
    const int k0 = (int)((int64_t)nviews * blockIdx.z / slices), k1 = (int)((int64_t)nviews * (blockIdx.z + 1) / slices);
    const double R = c.R;
    const double uf = ((double)iu + 0.5 - 0.5 * f.nu) * f.du + f.ou;
    const double a = DSD * DSD + uf * uf;
    const double b = -2.0 * DSD * (DSD - R);
    const double cc = (DSD - R) * (DSD - R) - R * R;
    const double t = (-b + sqrt(b * b - 4.0 * a * cc)) / (2.0 * a);
    const double s = R * atan2(t * uf, t * DSD - DSD + R);
    const double cu = (s - c.ou) / c.du + 0.5 * c.nu - 0.5;
    const double fl_u = floor(cu);
    const int u0 = (int)fl_u;
    const float wu1 = (float)(cu - fl_u), wu0 = 1.0f - wu1;
    const bool ok0 = u0 >= 0 && u0 < c.nu, ok1 = u0 + 1 >= 0 && u0 + 1 < c.nu;
    // height coordinate: cv = (t v - ov) / dv + nv/2 - 1/2 = kv * iv + cv0
    const double kv = t * f.dv / c.dv;
    const double cv0 = (t * ((0.5 - 0.5 * f.nv) * f.dv + f.ov) - c.ov) / c.dv + 0.5 * c.nv - 0.5;
    const int64_t cpix = (int64_t)c.nv * c.nu, fpix = (int64_t)f.nv * f.nu;
    const int64_t rows_per_pass = (int64_t)gridDim.y * 4 * FLAT_R;
    for (int64_t iv0 = ((int64_t)blockIdx.y * 4 + threadIdx.x / 64) * FLAT_R; iv0 < f.nv; iv0 += rows_per_pass) {
        for (int iv = (int)iv0; iv < min((int)iv0 + FLAT_R, f.nv); ++iv) {
            const double cv = __builtin_fma((double)iv, kv, cv0);
            const double fl_v = floor(cv);
            const int v0 = (int)fl_v;
            const float wv1 = (float)(cv - fl_v), wv0 = 1.0f - wv1;
            const bool in0 = v0 >= 0 && v0 < c.nv, in1 = v0 + 1 >= 0 && v0 + 1 < c.nv;
            const float w00 = wv0 * wu0, w01 = wv0 * wu1, w10 = wv1 * wu0, w11 = wv1 * wu1;
            const float* q = curved + (k0 * cpix + (int64_t)v0 * c.nu + u0);
            float* o = flat + (k0 * fpix + (int64_t)iv * f.nu + iu);
#pragma unroll 4
            for (int k = k0; k < k1; ++k, q += cpix, o += fpix) {
                float acc = 0.0f;
                if (in0 && ok0) acc = __builtin_fmaf(w00, q[0], acc);
                if (in0 && ok1) acc = __builtin_fmaf(w01, q[1], acc);
                if (in1 && ok0) acc = __builtin_fmaf(w10, q[c.nu], acc);
                if (in1 && ok1) acc = __builtin_fmaf(w11, q[c.nu + 1], acc);
                *o = acc;
            }
        }
    }
}

}  // namespace

hipError_t launch_flatten_curved(const Plan& p, const CurvedDet& c, const float* curved, float* flat, int64_t nviews,
                                 hipStream_t s)
{
    FlatDet f;
    f.nu = p.det.nu;
    f.nv = p.det.nv;
    f.du = p.geo.dDetector[1];
    f.dv = p.geo.dDetector[0];
    f.ou = p.geo.offDetector[1];
    f.ov = p.geo.offDetector[0];
    // enough slices of the views for 32 waves per CU
    const int64_t cols = (f.nu + 63) / 64, rows = std::min<int64_t>((f.nv + 4 * FLAT_R - 1) / (4 * FLAT_R), 65535);
    const int64_t slices = std::min<int64_t>(std::max<int64_t>(2048 / (cols * rows), 1), nviews);
    const dim3 grid((unsigned)cols, (unsigned)rows, (unsigned)slices);
    hipLaunchKernelGGL(k_flatten_curved, grid, dim3(256), 0, s, curved, flat, (int)nviews, f, c, p.geo.DSD);
    return hipGetLastError();
}

}  // namespace ctmi
