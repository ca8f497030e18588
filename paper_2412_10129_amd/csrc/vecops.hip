// Vector kernels of the iterative methods: CGLS (section 2.2.1), OS-SART
// (section 2.2.2) and the error history (section 2.2.3).  All are streaming
// HBM-bound loops; reductions accumulate in FP64 with a fixed blocking and
// a fixed tree order, so results are bit-reproducible for a given n.
#include "ctmi_internal.h"

namespace ctmi {

namespace {

constexpr int RB = 256;          // threads per reduction block
constexpr int RMAX = 1024;       // max partial sums

__device__ __forceinline__ double block_sum(double v, double* sh)
{
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int s = RB / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
        __syncthreads();
    }
    return sh[0];
}

__global__ void __launch_bounds__(RB) k_final_sum(const double* __restrict__ part, int nparts, int nvals,
                                                  double* out)
{
    __shared__ double sh[RB];
    for (int c = 0; c < nvals; ++c) {
        double s = 0.0;
        for (int i = threadIdx.x; i < nparts; i += RB) s += part[c * RMAX + i];
        s = block_sum(s, sh);
        if (threadIdx.x == 0) out[c] = s;
        __syncthreads();
    }
}

// Partial FP64 dot products, one per block (a fixed blocking: the result
// depends only on n).  With V4 (both arrays 16-byte aligned) each lane
// takes float4 pairs, two per step so that four loads are in flight; block
// 0 adds the n mod 4 tail.  Products of two floats are exact in FP64.
template <bool V4>
__global__ void __launch_bounds__(RB) k_dot_partial(const float* __restrict__ a, const float* __restrict__ b,
                                                    int64_t n, double* __restrict__ part)
{
    __shared__ double sh[RB];
    double s = 0.0, t = 0.0;
    const int64_t stride = (int64_t)gridDim.x * RB;
    if (V4) {
        const float4* __restrict__ a4 = reinterpret_cast<const float4*>(a);
        const float4* __restrict__ b4 = reinterpret_cast<const float4*>(b);
        const int64_t n4 = n >> 2;
        int64_t i = (int64_t)blockIdx.x * RB + threadIdx.x;
        for (; i + stride < n4; i += 2 * stride) {
            const float4 x0 = a4[i], y0 = b4[i], x1 = a4[i + stride], y1 = b4[i + stride];
            s = __builtin_fma((double)x0.x, (double)y0.x, s);
            t = __builtin_fma((double)x1.x, (double)y1.x, t);
            s = __builtin_fma((double)x0.y, (double)y0.y, s);
            t = __builtin_fma((double)x1.y, (double)y1.y, t);
            s = __builtin_fma((double)x0.z, (double)y0.z, s);
            t = __builtin_fma((double)x1.z, (double)y1.z, t);
            s = __builtin_fma((double)x0.w, (double)y0.w, s);
            t = __builtin_fma((double)x1.w, (double)y1.w, t);
        }
        if (i < n4) {
            const float4 x0 = a4[i], y0 = b4[i];
            s = __builtin_fma((double)x0.x, (double)y0.x, s);
            s = __builtin_fma((double)x0.y, (double)y0.y, s);
            s = __builtin_fma((double)x0.z, (double)y0.z, s);
            s = __builtin_fma((double)x0.w, (double)y0.w, s);
        }
        if (blockIdx.x == 0 && (int64_t)threadIdx.x < (n & 3)) {
            const int64_t k = 4 * n4 + threadIdx.x;
            t = __builtin_fma((double)a[k], (double)b[k], t);
        }
    } else {
        for (int64_t i = (int64_t)blockIdx.x * RB + threadIdx.x; i < n; i += stride)
            s += (double)a[i] * (double)b[i];
    }
    s = block_sum(s + t, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = s;
}

__global__ void __launch_bounds__(256) k_axpby(int64_t n, float a, const float* __restrict__ x, float b,
                                               float* __restrict__ y)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
        y[i] = __builtin_fmaf(a, x[i], b * y[i]);
}

__device__ __forceinline__ float safe_ratio(const double* num, const double* den)
{
    const double d = *den;
    return d != 0.0 ? (float)(*num / d) : 0.0f;
}

__global__ void __launch_bounds__(256) k_cgls_x(float* __restrict__ x, const float* __restrict__ p, int64_t n,
                                                const double* gamma, const double* delta)
{
    const float alpha = safe_ratio(gamma, delta);
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
        x[i] = __builtin_fmaf(alpha, p[i], x[i]);
}

// r -= alpha q with |r|^2 (FP64) per block; V4 as in k_dot_partial.
template <bool V4>
__global__ void __launch_bounds__(RB) k_cgls_r(float* __restrict__ r, const float* __restrict__ q, int64_t n,
                                               const double* gamma, const double* delta, double* __restrict__ part)
{
    __shared__ double sh[RB];
    const float alpha = safe_ratio(gamma, delta);
    double s = 0.0, t = 0.0;
    const int64_t stride = (int64_t)gridDim.x * RB;
    if (V4) {
        float4* __restrict__ r4 = reinterpret_cast<float4*>(r);
        const float4* __restrict__ q4 = reinterpret_cast<const float4*>(q);
        const int64_t n4 = n >> 2;
        int64_t i = (int64_t)blockIdx.x * RB + threadIdx.x;
        for (; i + stride < n4; i += 2 * stride) {
            float4 x0 = r4[i], x1 = r4[i + stride];
            const float4 y0 = q4[i], y1 = q4[i + stride];
            x0.x = __builtin_fmaf(-alpha, y0.x, x0.x);
            x0.y = __builtin_fmaf(-alpha, y0.y, x0.y);
            x0.z = __builtin_fmaf(-alpha, y0.z, x0.z);
            x0.w = __builtin_fmaf(-alpha, y0.w, x0.w);
            x1.x = __builtin_fmaf(-alpha, y1.x, x1.x);
            x1.y = __builtin_fmaf(-alpha, y1.y, x1.y);
            x1.z = __builtin_fmaf(-alpha, y1.z, x1.z);
            x1.w = __builtin_fmaf(-alpha, y1.w, x1.w);
            r4[i] = x0;
            r4[i + stride] = x1;
            s = __builtin_fma((double)x0.x, (double)x0.x, s);
            t = __builtin_fma((double)x1.x, (double)x1.x, t);
            s = __builtin_fma((double)x0.y, (double)x0.y, s);
            t = __builtin_fma((double)x1.y, (double)x1.y, t);
            s = __builtin_fma((double)x0.z, (double)x0.z, s);
            t = __builtin_fma((double)x1.z, (double)x1.z, t);
            s = __builtin_fma((double)x0.w, (double)x0.w, s);
            t = __builtin_fma((double)x1.w, (double)x1.w, t);
        }
        if (i < n4) {
            float4 x0 = r4[i];
            const float4 y0 = q4[i];
            x0.x = __builtin_fmaf(-alpha, y0.x, x0.x);
            x0.y = __builtin_fmaf(-alpha, y0.y, x0.y);
            x0.z = __builtin_fmaf(-alpha, y0.z, x0.z);
            x0.w = __builtin_fmaf(-alpha, y0.w, x0.w);
            r4[i] = x0;
            s = __builtin_fma((double)x0.x, (double)x0.x, s);
            s = __builtin_fma((double)x0.y, (double)x0.y, s);
            s = __builtin_fma((double)x0.z, (double)x0.z, s);
            s = __builtin_fma((double)x0.w, (double)x0.w, s);
        }
        if (blockIdx.x == 0 && (int64_t)threadIdx.x < (n & 3)) {
            const int64_t k = 4 * n4 + threadIdx.x;
            const float v = __builtin_fmaf(-alpha, q[k], r[k]);
            r[k] = v;
            t = __builtin_fma((double)v, (double)v, t);
        }
    } else {
        for (int64_t i = (int64_t)blockIdx.x * RB + threadIdx.x; i < n; i += stride) {
            const float v = __builtin_fmaf(-alpha, q[i], r[i]);
            r[i] = v;
            s += (double)v * (double)v;
        }
    }
    s = block_sum(s + t, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = s;
}

__global__ void __launch_bounds__(256) k_cgls_p(float* __restrict__ p, const float* __restrict__ s_, int64_t n,
                                                const double* g0, const double* g1)
{
    const float beta = safe_ratio(g1, g0);
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
        p[i] = __builtin_fmaf(beta, p[i], s_[i]);
}

__global__ void __launch_bounds__(256) k_recip(const float* in, float* out, int64_t n)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const float v = in[i];
        out[i] = v != 0.0f ? 1.0f / v : 0.0f;
    }
}

__global__ void __launch_bounds__(256) k_sart_residual(const float* __restrict__ b, const float* ax,
                                                       const float* __restrict__ w, float* out, int64_t n)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
        out[i] = w[i] * (b[i] - ax[i]);
}

__global__ void __launch_bounds__(256) k_sart_update(float* __restrict__ x, const float* __restrict__ v,
                                                     const float* __restrict__ bp, int64_t n, float lam, int nonneg)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        float y = __builtin_fmaf(lam * v[i], bp[i], x[i]);
        if (nonneg) y = fmaxf(y, 0.0f);
        x[i] = y;
    }
}

// Adaptive-weighted TV (section 2.2.3, extended to 3-D): the term of voxel
// u (all three backward neighbours present) is s_u = sqrt(sum_a w_a d_a^2 +
// eps), d_a = x_u - x_{u - e_a}, w_a = exp(-(d_a / delta)^2) (1 for plain
// TV); q_a(u) = w_a d_a / s_u (0 when s_u = 0).  The gradient with the
// weights lagged is g_v = sum_a q_a(v) - sum_a q_a(v + e_a).
//
// A wave owns TVX voxels along x (its lanes, with one more on either side) by
// TVY rows and marches up z on its own: the neighbours along x come from the
// next lanes (DPP), those along y and z from the thread's registers, so there
// is no LDS and no barrier, and the terms formed twice are the lanes' and rows'
// ends (64 / 62 and 9 / 8).  The next plane's rows are loaded a step ahead.  VALU
// bounds it (three exponentials, a correctly rounded root and a division per
// term): 512^3, adaptive weights, 400 us as 64 x 8 tiles staged in LDS, with 2.3
// rounds of terms per tile and step between barriers; 322 us so (1.07 GB).
struct TvTerm {
    float qz, qy, qx;
};

template <bool ADAPTIVE>
__device__ __forceinline__ TvTerm tv_term(float dz, float dy, float dx, float nid2, float eps)
{
    float wz = 1.0f, wy = 1.0f, wx = 1.0f;
    if (ADAPTIVE) {   // nid2 = -1 / delta^2
        wz = __expf(dz * dz * nid2);
        wy = __expf(dy * dy * nid2);
        wx = __expf(dx * dx * nid2);
    }
    const float az = wz * dz, ay = wy * dy, ax = wx * dx;
    const float s2 = __builtin_fmaf(az, dz, __builtin_fmaf(ay, dy, __builtin_fmaf(ax, dx, eps)));
    const float r = s2 > 0.0f ? 1.0f / __builtin_sqrtf(s2) : 0.0f;
    return TvTerm{az * r, ay * r, ax * r};
}

__device__ __forceinline__ float lane_below(float v)   // of lane - 1 (0 for lane 0)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xf, 0xf, false));
}
__device__ __forceinline__ float lane_above(float v)   // of lane + 1 (0 for lane 63)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130, 0xf, 0xf, false));
}

constexpr int TVX = 62, TVY = 8;

template <bool ADAPTIVE>
__global__ void __launch_bounds__(256, 6) k_awtv_grad(const float* __restrict__ x, float* __restrict__ g, int nz, int ny,
                                                   int nx, int tz, int nbx, int nby, float nid2, float eps)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // layers of tz planes from the top down (what is written last, the low planes, is
    // what a pass over g reads first); in a layer each XCD takes a contiguous
    // run (tiles side by side along x share cache lines)
    const int per = (nbx * nby + 7) / 8, layers = (nz + tz - 1) / tz;
    const int layer = (int)(blockIdx.x / (8 * per)), r = (int)(blockIdx.x % (8 * per));
    const int b = r % 8 * per + r / 8;
    if (b >= nbx * nby) return;
    const int by = b / nbx, bx = b - by * nbx;
    const int X = bx * TVX + lane - 1;
    const int y0 = (by * 4 + wave) * TVY;
    const int z0 = (layers - 1 - layer) * tz, z1 = min(z0 + tz, nz);
    if (y0 >= ny) return;
    const int64_t sz = (int64_t)nx * ny;
    const bool in = X >= 0 && X < nx;                       // this lane's column is in the volume
    const bool term_x = X >= 1 && X < nx;                   // and has a term
    const bool out_x = in && lane >= 1 && lane <= TVX;      // and is this wave's
    // rows y0 - 1 ... y0 + TVY of a plane (0 outside the volume)
    auto load = [&](int Z, float (&r)[TVY + 2]) {
        const float* pz = x + (int64_t)Z * sz;
#pragma unroll
        for (int j = 0; j < TVY + 2; ++j) {
            const int Y = y0 - 1 + j;
            r[j] = 0.0f;
            if (Z >= 0 && Z < nz && Y >= 0 && Y < ny && in) r[j] = pz[(int64_t)Y * nx + X];
        }
    };
    float prev[TVY + 2], cur[TVY + 2], next[TVY + 2];
    float own[TVY], upy[TVY], upx[TVY];   // the plane below: a voxel's own terms, its upper neighbours' in y and x
    load(z0 - 1, prev);
    load(z0, cur);
    for (int z = z0; z <= z1; ++z) {   // terms of plane z, gradient of plane z - 1
        if (z < z1) load(z + 1, next);
        TvTerm t[TVY + 1];
#pragma unroll
        for (int j = 0; j <= TVY; ++j) {
            const int Y = y0 + j;
            t[j] = TvTerm{0.0f, 0.0f, 0.0f};
            const float c = cur[j + 1], cx = lane_below(c);
            if (z >= 1 && z < nz && Y >= 1 && Y < ny && term_x)
                t[j] = tv_term<ADAPTIVE>(c - prev[j + 1], c - cur[j], c - cx, nid2, eps);
        }
        if (z > z0) {
            float* gz = g + (int64_t)(z - 1) * sz;
#pragma unroll
            for (int j = 0; j < TVY; ++j)
                if (y0 + j < ny && out_x) gz[(int64_t)(y0 + j) * nx + X] = own[j] - t[j].qz - upy[j] - upx[j];
        }
#pragma unroll
        for (int j = 0; j < TVY; ++j) {
            own[j] = t[j].qz + t[j].qy + t[j].qx;
            upy[j] = t[j + 1].qy;
            upx[j] = lane_above(t[j].qx);
        }
#pragma unroll
        for (int j = 0; j < TVY + 2; ++j) {
            prev[j] = cur[j];
            cur[j] = next[j];
        }
    }
}

// TV steepest-descent step: x -= step * g / sqrt(gnorm2) (gnorm2 a device
// double; nothing happens when it is 0).
__global__ void __launch_bounds__(256) k_tv_step(float* __restrict__ x, const float* __restrict__ g, int64_t n,
                                                 const double* __restrict__ gnorm2, float step)
{
    const double gn2 = *gnorm2;
    if (!(gn2 > 0.0)) return;
    const float f = (float)((double)step / sqrt(gn2));
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
        x[i] = __builtin_fmaf(-f, g[i], x[i]);
}

// EM ratio (MLEM/OSEM, section 2.2): out = b / ax where ax > 0, else 0.
__global__ void __launch_bounds__(256) k_em_ratio(const float* __restrict__ b, const float* ax, float* out, int64_t n)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const float a = ax[i];
        out[i] = a > 0.0f ? b[i] / a : 0.0f;
    }
}

// EM update: x = x * v * bp, v = 1 / (A^T 1) (0 where no ray reaches).
__global__ void __launch_bounds__(256) k_em_update(float* __restrict__ x, const float* __restrict__ v,
                                                   const float* __restrict__ bp, int64_t n)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) x[i] = x[i] * v[i] * bp[i];
}

__global__ void __launch_bounds__(RB) k_fov_partial(const float* __restrict__ x, const float* __restrict__ gt,
                                                    VolDims v, float cx, float cy, float r2,
                                                    double* __restrict__ part)
{
    __shared__ double sh[RB];
    const int64_t n = (int64_t)v.nx * v.ny * v.nz;
    double s = 0.0, c = 0.0;
    const int64_t stride = (int64_t)gridDim.x * RB;
    for (int64_t i = (int64_t)blockIdx.x * RB + threadIdx.x; i < n; i += stride) {
        const int ix = (int)(i % v.nx);
        const int iy = (int)((i / v.nx) % v.ny);
        const float X = ((float)ix - cx) * v.hx, Y = ((float)iy - cy) * v.hy;
        if (__builtin_fmaf(X, X, Y * Y) <= r2) {
            const double d = (double)x[i] - (double)gt[i];
            s += d * d;
            c += 1.0;
        }
    }
    s = block_sum(s, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = s;
    __syncthreads();
    c = block_sum(c, sh);
    if (threadIdx.x == 0) part[RMAX + blockIdx.x] = c;
}

unsigned stream_blocks(int64_t n)
{
    int64_t b = (n + 256 * 8 - 1) / (256 * 8);
    if (b < 1) b = 1;
    if (b > 8192) b = 8192;
    return (unsigned)b;
}

}  // namespace

static bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

int reduce_blocks(int64_t n)
{
    int64_t b = (n + RB * 16 - 1) / (RB * 16);
    if (b < 1) b = 1;
    if (b > RMAX) b = RMAX;
    return (int)b;
}

hipError_t launch_dot(const float* a, const float* b, int64_t n, double* out, double* ws, hipStream_t s)
{
    const int g = reduce_blocks(n);
    if (aligned16(a) && aligned16(b))
        hipLaunchKernelGGL(k_dot_partial<true>, dim3(g), dim3(RB), 0, s, a, b, n, ws);
    else
        hipLaunchKernelGGL(k_dot_partial<false>, dim3(g), dim3(RB), 0, s, a, b, n, ws);
    hipLaunchKernelGGL(k_final_sum, dim3(1), dim3(RB), 0, s, ws, g, 1, out);
    return hipGetLastError();
}

hipError_t launch_axpby(int64_t n, float a, const float* x, float b, float* y, hipStream_t s)
{
    hipLaunchKernelGGL(k_axpby, dim3(stream_blocks(n)), dim3(256), 0, s, n, a, x, b, y);
    return hipGetLastError();
}

hipError_t launch_cgls_xr(float* x, const float* p, int64_t nvol, float* r, const float* q, int64_t nproj,
                          const double* gamma, const double* delta, double* rnorm2, double* ws, hipStream_t s)
{
    hipLaunchKernelGGL(k_cgls_x, dim3(stream_blocks(nvol)), dim3(256), 0, s, x, p, nvol, gamma, delta);
    const int g = reduce_blocks(nproj);
    if (aligned16(r) && aligned16(q))
        hipLaunchKernelGGL(k_cgls_r<true>, dim3(g), dim3(RB), 0, s, r, q, nproj, gamma, delta, ws);
    else
        hipLaunchKernelGGL(k_cgls_r<false>, dim3(g), dim3(RB), 0, s, r, q, nproj, gamma, delta, ws);
    hipLaunchKernelGGL(k_final_sum, dim3(1), dim3(RB), 0, s, ws, g, 1, rnorm2);
    return hipGetLastError();
}

hipError_t launch_cgls_p(float* p, const float* s_, int64_t n, const double* g0, const double* g1, hipStream_t s)
{
    hipLaunchKernelGGL(k_cgls_p, dim3(stream_blocks(n)), dim3(256), 0, s, p, s_, n, g0, g1);
    return hipGetLastError();
}

hipError_t launch_recip(const float* in, float* out, int64_t n, hipStream_t s)
{
    hipLaunchKernelGGL(k_recip, dim3(stream_blocks(n)), dim3(256), 0, s, in, out, n);
    return hipGetLastError();
}

hipError_t launch_sart_residual(const float* b, const float* ax, const float* w, float* out, int64_t n,
                                hipStream_t s)
{
    hipLaunchKernelGGL(k_sart_residual, dim3(stream_blocks(n)), dim3(256), 0, s, b, ax, w, out, n);
    return hipGetLastError();
}

hipError_t launch_sart_update(float* x, const float* v, const float* bp, int64_t n, float lam, int nonneg,
                              hipStream_t s)
{
    hipLaunchKernelGGL(k_sart_update, dim3(stream_blocks(n)), dim3(256), 0, s, x, v, bp, n, lam, nonneg);
    return hipGetLastError();
}

hipError_t launch_awtv_grad(const float* x, float* g, int nz, int ny, int nx, float delta, float eps, hipStream_t s)
{
    // planes per wave: 8 (each march forms one plane of terms more than it writes, but
    // long ones keep waves in planes far apart in memory: 512^3 at 32 planes 329 us, at 16
    // 321, at 8 322 with the next pass 8 us faster), or 4 where that leaves the 256 CUs
    // short of waves
    const int nbx = (nx + TVX - 1) / TVX, nby = (ny + 4 * TVY - 1) / (4 * TVY);
    const int tz = (int64_t)nbx * nby * 4 * ((nz + 7) / 8) < 4096 ? 4 : 8;
    const dim3 grid((unsigned)((nbx * nby + 7) / 8 * 8 * ((nz + tz - 1) / tz)));
    const float nid2 = delta > 0.0f ? -1.0f / (delta * delta) : 0.0f;
    if (nid2 != 0.0f)
        hipLaunchKernelGGL(k_awtv_grad<true>, grid, dim3(256), 0, s, x, g, nz, ny, nx, tz, nbx, nby, nid2, eps);
    else   // plain TV (also a delta whose square is infinite: every weight is 1)
        hipLaunchKernelGGL(k_awtv_grad<false>, grid, dim3(256), 0, s, x, g, nz, ny, nx, tz, nbx, nby, 0.0f, eps);
    return hipGetLastError();
}

hipError_t launch_tv_step(float* x, const float* g, int64_t n, const double* gnorm2, float step, hipStream_t s)
{
    hipLaunchKernelGGL(k_tv_step, dim3(stream_blocks(n)), dim3(256), 0, s, x, g, n, gnorm2, step);
    return hipGetLastError();
}

hipError_t launch_em_ratio(const float* b, const float* ax, float* out, int64_t n, hipStream_t s)
{
    hipLaunchKernelGGL(k_em_ratio, dim3(stream_blocks(n)), dim3(256), 0, s, b, ax, out, n);
    return hipGetLastError();
}

hipError_t launch_em_update(float* x, const float* v, const float* bp, int64_t n, hipStream_t s)
{
    hipLaunchKernelGGL(k_em_update, dim3(stream_blocks(n)), dim3(256), 0, s, x, v, bp, n);
    return hipGetLastError();
}

hipError_t launch_fov_sq_err(const Plan& p, const float* x, const float* gt, double* out, double* ws,
                             hipStream_t s)
{
    const int64_t n = (int64_t)p.vol.nx * p.vol.ny * p.vol.nz;
    const int g = reduce_blocks(n);
    // voxel-centre index of the volume centre; the cylinder is centred on the
    // volume (its offset does not change the index geometry)
    const float cx = 0.5f * (float)p.vol.nx - 0.5f, cy = 0.5f * (float)p.vol.ny - 0.5f;
    const double R = 0.5 * ((double)p.vol.ny * p.vol.hy < (double)p.vol.nx * p.vol.hx ? (double)p.vol.ny * p.vol.hy
                                                                                       : (double)p.vol.nx * p.vol.hx);
    hipLaunchKernelGGL(k_fov_partial, dim3(g), dim3(RB), 0, s, x, gt, p.vol, cx, cy, (float)(R * R), ws);
    hipLaunchKernelGGL(k_final_sum, dim3(1), dim3(RB), 0, s, ws, g, 2, out);
    return hipGetLastError();
}

size_t reduce_ws_bytes() { return sizeof(double) * 2 * RMAX; }

}  // namespace ctmi
