// Kernels of the learned prior: a 3-D residual U-Net in BF16 with FP32
// accumulation, used plug-and-play inside CGLS.  The paper only says that
// trained networks call the projection operators; the network itself is
// the builder's choice (4 levels of 16/32/64/128 channels, 3x3x3 convs with
// ReLU, 2x2x2 average pooling, stride-2 2x2x2 transposed convs, skip
// concatenation, a 1x1x1 residual head).
//
// Layout: activations are channels-last BF16, [n][z][y][x][ld] with the
// tensor's channels at [0, C) of each voxel's ld-element row, so a channel
// concatenation is two (pointer, count, ld) operands and costs nothing.
// 3x3x3 weights are BF16 [cout][27][cin] with tap t = 9 kz + 3 ky + kx
// reading the input at (z + kz - 1, y + ky - 1, x + kx - 1).
//
// The 3x3x3 convolution is an implicit GEMM on the gfx950 BF16 MFMA
// (16x16x32, FP32 accumulators): D[co][voxel] = sum_k W[co][k] X[k][voxel]
// with k = (tap, ci), one MFMA step covering two taps x 16 channels.  Up to 32
// input channels (the fine levels, bound by memory) a workgroup marches along z
// (k_conv3z); above, it owns 2 x 8 x 16 output voxels and stages its input 16
// channels at a time as a halo brick in LDS (48-byte voxel stride: the sixteen
// 16-byte lane reads of a row hit disjoint banks; k_conv3).  The data gradient
// is the same kernels with flipped, transposed weights.
#include "ctmi_internal.h"

namespace ctmi {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint16_t u16;

__device__ __forceinline__ float bf2f(u16 h) { return __uint_as_float((uint32_t)h << 16); }

// FP32 -> BF16, round to nearest, ties to even (finite inputs).
__device__ __forceinline__ u16 f2bf(float f)
{
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (u16)(u >> 16);
}

__device__ __forceinline__ bool bf_pos(u16 h) { return h != 0 && !(h & 0x8000u); }

__device__ __forceinline__ void unpack8(const uint4 q, float* f)
{
    const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        f[2 * i] = __uint_as_float(w[i] << 16);
        f[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
    }
}

__device__ __forceinline__ uint4 pack8(const float* f)
{
    uint4 q;
    q.x = (uint32_t)f2bf(f[0]) | ((uint32_t)f2bf(f[1]) << 16);
    q.y = (uint32_t)f2bf(f[2]) | ((uint32_t)f2bf(f[3]) << 16);
    q.z = (uint32_t)f2bf(f[4]) | ((uint32_t)f2bf(f[5]) << 16);
    q.w = (uint32_t)f2bf(f[6]) | ((uint32_t)f2bf(f[7]) << 16);
    return q;
}

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 q)
{
    bf16x8 r;
    __builtin_memcpy(&r, &q, 16);
    return r;
}

// Voxel v of an [n][d][h][w] grid of nvox voxels.  Below 2^31 in 32 bits: three
// 64-bit divisions are several hundred instructions, most of what the kernels
// with little work per voxel did.
struct Vox {
    int x, y, z, n;
};
__device__ __forceinline__ Vox vox_of(int64_t v, int64_t nvox, int d, int h, int w)
{
    Vox q;
    if (nvox < (int64_t)1 << 31) {
        unsigned r = (unsigned)v;
        q.x = (int)(r % (unsigned)w);
        r /= (unsigned)w;
        q.y = (int)(r % (unsigned)h);
        r /= (unsigned)h;
        q.z = (int)(r % (unsigned)d);
        q.n = (int)(r / (unsigned)d);
    } else {
        q.x = (int)(v % w);
        v /= w;
        q.y = (int)(v % h);
        v /= h;
        q.z = (int)(v % d);
        q.n = (int)(v / d);
    }
    return q;
}

// ------------------------------------------------------------------ conv3
constexpr int CX = 16, CY = 8, CZ = 2;               // output tile (x fastest)
constexpr int HX = CX + 2, HY = CY + 2, HZ = CZ + 2;  // halo brick
constexpr int HVOX = HX * HY * HZ;                    // 720
constexpr int VS = 24;                                // LDS voxel stride (u16): 16 ch + 8 pad

// bias, ReLU, ReLU mask (m: the layer input's values) and BF16 rounding of
// four output channels
__device__ __forceinline__ uint2 conv_epilogue(const f32x4& acc, const float* bias, int relu, bool mask, uint2 m)
{
    float v[4] = {acc[0], acc[1], acc[2], acc[3]};
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] += bias[e];
    if (relu) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = fmaxf(v[e], 0.0f);
    }
    if (mask) {
        if (!bf_pos((u16)(m.x & 0xFFFF))) v[0] = 0.0f;
        if (!bf_pos((u16)(m.x >> 16))) v[1] = 0.0f;
        if (!bf_pos((u16)(m.y & 0xFFFF))) v[2] = 0.0f;
        if (!bf_pos((u16)(m.y >> 16))) v[3] = 0.0f;
    }
    uint2 o;
    o.x = (uint32_t)f2bf(v[0]) | ((uint32_t)f2bf(v[1]) << 16);
    o.y = (uint32_t)f2bf(v[2]) | ((uint32_t)f2bf(v[3]) << 16);
    return o;
}

// More than 32 input channels: a workgroup owns 2 x 8 x 16 output voxels and
// NT tiles of 16 output channels.  The next 16 channels of the halo are loaded
// into registers while the staged ones are worked on, and the next step's weights
// (from L1/L2) and LDS reads are issued before this step's MFMAs: without that the
// kernel waited for memory in each of its 14 steps per 16 channels.
template <int NT>
__global__ __launch_bounds__(256) void k_conv3(UnetConv3 a)
{
    __shared__ __attribute__((aligned(16))) u16 xs[HVOX * VS];

    const int tiles_x = (a.w + CX - 1) / CX, tiles_y = (a.h + CY - 1) / CY;
    const int x0 = (blockIdx.x % tiles_x) * CX;
    const int y0 = (blockIdx.x / tiles_x % tiles_y) * CY;
    const int co0 = (blockIdx.x / (tiles_x * tiles_y)) * 16 * NT;   // the workgroup's output channels
    const int z0 = blockIdx.y * CZ;
    const int nb = blockIdx.z;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int g = lane >> 4, li = lane & 15;
    const int cin = a.c0 + a.c1;

    f32x4 acc[4][NT];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int n = 0; n < NT; ++n) acc[r][n] = f32x4{0.f, 0.f, 0.f, 0.f};

    const size_t plane = (size_t)a.h * a.w;
    const size_t vbase = (size_t)nb * a.d * plane;

    // staged elements of this thread: item i = tid + 256 m is half i & 1 of
    // halo voxel i >> 1
    constexpr int LD = (2 * HVOX + 255) / 256;
    uint32_t off[LD];   // voxel distance from the halo's corner
    bool ok[LD];
#pragma unroll
    for (int m = 0; m < LD; ++m) {
        const int i = tid + 256 * m, hv = i >> 1;
        const int hx = hv % HX, hy = (hv / HX) % HY, hz = hv / (HX * HY);
        const int gx = x0 + hx - 1, gy = y0 + hy - 1, gz = z0 + hz - 1;
        ok[m] = hv < HVOX && gx >= 0 && gx < a.w && gy >= 0 && gy < a.h && gz >= 0 && gz < a.d;
        off[m] = (uint32_t)((hz * a.h + hy) * a.w + hx);
    }
    const int64_t corner = (int64_t)vbase + (int64_t)(z0 - 1) * (int64_t)plane + (int64_t)(y0 - 1) * a.w + (x0 - 1);
    // the next 16 channels' halo is loaded into registers while the current
    // ones are computed, and the next step's weights while a step is
    uint4 pf[LD];
    auto fetch = [&](int cc) {
        const bool second = cc >= a.c0;
        const u16* src = second ? a.in1 + (cc - a.c0) : a.in0 + cc;
        const int ld = second ? a.ld1 : a.ld0;
        src += corner * ld + (tid & 1) * 8;
#pragma unroll
        for (int m = 0; m < LD; ++m) {
            pf[m] = make_uint4(0, 0, 0, 0);
            if (ok[m]) pf[m] = *reinterpret_cast<const uint4*>(src + (uint64_t)off[m] * (uint32_t)ld);
        }
    };
    const int t1 = g >> 1, ch = (g & 1) * 8;
    // lane offset (bytes) of tap t1 of the lane's output channel; the rest of a
    // fragment's address is the same in every lane
    const uint32_t wl = 2u * (((uint32_t)(co0 + li) * 27u + (uint32_t)t1) * (uint32_t)cin + (uint32_t)ch);
    auto weights = [&](uint4 (&wf)[NT], uint32_t wc, int s) {
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            wf[n] = make_uint4(0, 0, 0, 0);
            if (s < 13 || t1 == 0)
                wf[n] = *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(a.wt) +
                                                        (size_t)(wc + (uint32_t)((n * 16 * 27 + 2 * s) * 2 * cin)) + wl);
        }
    };
    const u16* xl = xs + li * VS + ch;
    auto inputs = [&](uint4 (&xf)[4], int s) {
        // halo voxel of tap 2s, and of tap 2s + 1 in lanes 32-63 (tap 27 does not exist)
        const int ta = 2 * s, tb = s < 13 ? ta + 1 : ta;
        const int va = (ta / 9 * HY + ta / 3 % 3) * HX + ta % 3, vb = (tb / 9 * HY + tb / 3 % 3) * HX + tb % 3;
        const u16* xt = xl + (t1 ? vb : va) * VS;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int rr = wave * 4 + r;
            xf[r] = *reinterpret_cast<const uint4*>(xt + ((rr >> 3) * HY + (rr & 7)) * HX * VS);
            if (s == 13 && t1) xf[r] = make_uint4(0, 0, 0, 0);
        }
    };
    auto mfmas = [&](const uint4 (&wf)[NT], const uint4 (&xf)[4]) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int n = 0; n < NT; ++n)
                acc[r][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(wf[n]), as_bf16x8(xf[r]), acc[r][n], 0, 0, 0);
    };
    fetch(0);
    for (int cc = 0; cc < cin; cc += 16) {
        // (an opaque scalar: otherwise every fragment's address becomes a
        // 64-bit loop variable in vector registers)
        uint32_t wc = 2 * cc;
        asm volatile("" : "+s"(wc));
        uint4 wa[NT], wb[NT];
        weights(wa, wc, 0);
        __syncthreads();
#pragma unroll
        for (int m = 0; m < LD; ++m) {
            const int i = tid + 256 * m;
            if (i < 2 * HVOX) *reinterpret_cast<uint4*>(&xs[(i >> 1) * VS + (tid & 1) * 8]) = pf[m];
        }
        __syncthreads();
        if (cc + 16 < cin) fetch(cc + 16);
        uint4 xa[4], xb[4];
        inputs(xa, 0);
        // (the scheduling barriers keep the compiler from loading every step's
        // weights at once, which spills, and each step's reads ahead of the
        // MFMAs they follow)
#pragma unroll
        for (int s = 0; s < 14; s += 2) {
            weights(wb, wc, s + 1);
            inputs(xb, s + 1);
            __builtin_amdgcn_sched_barrier(0);
            mfmas(wa, xa);
            if (s + 2 < 14) {
                weights(wa, wc, s + 2);
                inputs(xa, s + 2);
            }
            __builtin_amdgcn_sched_barrier(0);
            mfmas(wb, xb);
        }
    }

    // epilogue: lane holds channels n*16 + 4g .. +3 of voxel (row, x0 + li)
    const int x = x0 + li;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int rr = wave * 4 + r;
        const int z = z0 + (rr >> 3), y = y0 + (rr & 7);
        if (x >= a.w || y >= a.h || z >= a.d) continue;
        const size_t vox = vbase + (size_t)z * plane + (size_t)y * a.w + x;
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            const int co = co0 + n * 16 + 4 * g;
            float bias[4] = {0.f, 0.f, 0.f, 0.f};
            if (a.bias)
#pragma unroll
                for (int e = 0; e < 4; ++e) bias[e] = a.bias[co + e];
            uint2 m = make_uint2(0, 0);
            if (a.mask) m = *reinterpret_cast<const uint2*>(a.mask + vox * a.ldm + co);
            *reinterpret_cast<uint2*>(a.out + vox * a.ldo + co) = conv_epilogue(acc[r][n], bias, a.relu, a.mask != nullptr, m);
        }
    }
}

// Values of another row of 16 lanes: MOVE 0: rows 1 and 3 take rows 0 and 2;
// 1: rows 2 and 3 take rows 0 and 1; 2: rows 0 and 2 take rows 1 and 3 (the
// other rows get values that are not used).
template <int MOVE>
__device__ __forceinline__ float from_row(float q)
{
    const uint32_t u = __float_as_uint(q);
    if (MOVE == 1) return __uint_as_float(__builtin_amdgcn_permlane32_swap(u, u, false, false)[0]);
    return __uint_as_float(__builtin_amdgcn_permlane16_swap(u, u, false, false)[MOVE == 0 ? 0 : 1]);
}

// The same convolution for up to 32 input channels, marching along z: a
// workgroup owns a 16 x YT column of output voxels over zc planes and keeps the
// four input planes it works on in an LDS ring (planes z - 1, z, z + 1 of the
// current output plane, and plane z + 2, loaded into registers while plane z
// is computed), so an input plane is staged once per workgroup (1.27 to 1.4
// voxels read per output voxel, against 2.8 of the 2 x 8 x 16 tiles) and a plane
// costs one barrier.  A wave works on one tile of 16 output channels, whose
// weights (14 fragments of 16 bytes per lane and 16 input channels) stay in
// registers for the whole march; NTW = 2 gives the workgroup's waves two
// channel tiles.  Every output is formed by the same MFMAs on the same operands
// in the same order as in k_conv3, so the bits are the same.
//
// LDS reads and memory bound it about equally: 256^3, 16 -> 16 channels 301 us
// (1.07 GB: 3.6 TB/s, of 4.7 that a copy reaches); the four layers at 256^3 with
// the input's packing and the head 4040 us as 2 x 8 x 16 tiles and 1650 us so.
//
// LDS layout: per plane and 16 input channels two halves of 8 channels, voxels
// 16 bytes apart within a half, so 16 lanes read 256 consecutive bytes and every
// tap is an immediate offset from a few base addresses.  A step's two taps sit
// in lanes 0-31 and 32-63: next to each other in x (base A), or at the ends of
// two rows (base B), or, once, of two planes (base C).
//
// An output plane is written after the barrier that ends its phase, and what
// its epilogue reads (mask, network input) is loaded a phase ahead: loads and
// stores complete in order, so a store before the staged plane's arrival would
// be waited for.
//
// FIRST reads the FP32 network input instead of 16-channel rows (channel 0 =
// bf16(x), the others 0).  HEAD also applies the residual 1x1x1 head and writes
// the FP32 network output instead of the activations.
template <int NCH>
constexpr int march_rows() { return NCH == 1 ? 16 : 8; }

template <int NCH, int NTW, bool FIRST, bool HEAD, bool MASK>
__global__ __launch_bounds__(256) void k_conv3z(UnetConv3 a, int zc)
{
    constexpr int YT = march_rows<NCH>(), RW = YT * NTW / 4;   // tile rows, rows per wave
    constexpr int PX = CX + 2, PV = PX * (YT + 2);             // staged voxels per plane
    constexpr int HP = PV * 8, PC = 2 * HP, PL = NCH * PC;     // u16 per half, per 16 channels, per plane
    constexpr int LD = FIRST ? (PV + 255) / 256 : (2 * PV + 255) / 256;   // loads per thread, plane and 16 channels
    __shared__ __attribute__((aligned(16))) u16 xs[4 * PL];

    const int tiles_x = (a.w + CX - 1) / CX, tiles_y = (a.h + YT - 1) / YT;
    const int x0 = (blockIdx.x % tiles_x) * CX;
    const int y0 = (blockIdx.x / tiles_x % tiles_y) * YT;
    const int cot = (blockIdx.x / (tiles_x * tiles_y)) * NTW;
    const int z0 = blockIdx.y * zc, z1 = min(z0 + zc, a.d);
    const int nb = blockIdx.z;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int g = lane >> 4, li = lane & 15;
    const int cin = a.c0 + a.c1;
    const int co0 = (cot + wave % NTW) * 16, row0 = (wave / NTW) * RW;
    const int64_t plane = (int64_t)a.h * a.w;
    const int64_t vbase = (int64_t)nb * a.d * plane;

    // output channels of this lane's accumulator: 4 gc .. 4 gc + 3.  For the
    // head lane groups 2 and 3 trade places (through the weights' rows), so
    // that the channel order runs over the groups as 0, 1, 3, 2 and a sum can be
    // handed on with v_permlane16_swap and v_permlane32_swap.
    const int gc = HEAD ? g ^ (g >> 1) : g;
    const int wrow = HEAD ? li ^ ((li & 8) >> 1) : li;
    const int co = co0 + 4 * gc;

    // weights of this wave's channel tile (step s: taps 2s and 2s + 1)
    uint4 wf[NCH][14];
#pragma unroll
    for (int c = 0; c < NCH; ++c)
#pragma unroll
        for (int s = 0; s < 14; ++s) {
            const int tap = 2 * s + (g >> 1);
            wf[c][s] = make_uint4(0, 0, 0, 0);
            if (tap < 27)
                wf[c][s] = *reinterpret_cast<const uint4*>(a.wt + ((size_t)(co0 + wrow) * 27 + tap) * cin + c * 16 + (g & 1) * 8);
        }

    // this thread's staged elements: item i = tid + 256 m is half i & 1 of
    // voxel i >> 1 (FIRST: voxel i); lane offsets below 2^31 bytes (the
    // launcher checks)
    int off[LD], dst[LD];
    bool ok[LD];
#pragma unroll
    for (int m = 0; m < LD; ++m) {
        const int i = tid + 256 * m;
        const int hv = FIRST ? i : i >> 1, half = FIRST ? 0 : i & 1;
        const int gx = x0 + hv % PX - 1, gy = y0 + hv / PX - 1;
        ok[m] = hv < PV && gx >= 0 && gx < a.w && gy >= 0 && gy < a.h;
        off[m] = ok[m] ? gy * a.w + gx : 0;
        dst[m] = hv < PV ? half * HP + hv * 8 : -1;
    }
    uint4 pf[NCH][LD];
    auto fetch = [&](int z) {
        const bool zin = z >= 0 && z < a.d;
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            const bool second = 16 * c >= a.c0;
            const u16* src = second ? a.in1 + (16 * c - a.c0) : a.in0 + 16 * c;
            const int ld = second ? a.ld1 : a.ld0;
#pragma unroll
            for (int m = 0; m < LD; ++m) {
                pf[c][m] = make_uint4(0, 0, 0, 0);
                if (zin && ok[m]) {
                    if (FIRST)
                        pf[c][m].x = f2bf((a.x32 + (vbase + z * plane))[off[m]]);
                    else
                        pf[c][m] = *reinterpret_cast<const uint4*>(src + (vbase + z * plane) * ld +
                                                                    (off[m] * ld + ((tid & 1) * 8)));
                }
            }
        }
    };
    auto put = [&](int slot) {
#pragma unroll
        for (int c = 0; c < NCH; ++c)
#pragma unroll
            for (int m = 0; m < LD; ++m)
                if (dst[m] >= 0) *reinterpret_cast<uint4*>(&xs[slot * PL + c * PC + dst[m]]) = pf[c][m];
    };
    if (FIRST)   // channels 8..15 stay zero
        for (int i = tid; i < 4 * PV; i += 256)
            *reinterpret_cast<uint4*>(&xs[(i / PV) * PL + HP + (i % PV) * 8]) = make_uint4(0, 0, 0, 0);
    // plane z sits in slot (z - z0 + 1) & 3
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        fetch(z0 - 1 + i);
        put(i);
    }
    __syncthreads();

    const int x = x0 + li;
    const int lb = (g & 1) * HP + (row0 * PX + li) * 8;   // this lane's voxel at tap (0, 0, 0), in u16
    const int t1 = g >> 1;                                // second tap of a step
    float bias[4] = {0.f, 0.f, 0.f, 0.f}, hwf[4] = {0.f, 0.f, 0.f, 0.f}, hb = 0.0f;
    if (a.bias)
#pragma unroll
        for (int e = 0; e < 4; ++e) bias[e] = a.bias[co + e];
    if (HEAD) {
#pragma unroll
        for (int e = 0; e < 4; ++e) hwf[e] = bf2f(a.hw[4 * gc + e]);
        hb = a.hb[0];
    }
    bool in[RW];
    int orow[RW];   // voxel of row r in a plane
#pragma unroll
    for (int r = 0; r < RW; ++r) {
        const int y = y0 + row0 + r;
        in[r] = x < a.w && y < a.h;
        orow[r] = in[r] ? y * a.w + x : 0;
    }
    for (int z = z0; z < z1; ++z) {
        const int q = z - z0;
        const int64_t vz = vbase + z * plane;
        if (z + 1 < z1) fetch(z + 2);
        uint2 mk[MASK ? RW : 1];
        float xi[HEAD ? RW : 1];
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            if (MASK) mk[r] = *reinterpret_cast<const uint2*>(a.mask + (vz + orow[r]) * a.ldm + co);
            if (HEAD) xi[r] = a.x32[vz + orow[r]];
        }
        const u16* bA[3];
        const u16* bB[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const u16* b = xs + ((q + k) & 3) * PL + lb;
            bA[k] = b + t1 * 8;
            bB[k] = b + t1 * (PX - 2) * 8;
        }
        // taps 8 (0, 2, 2) and 9 (1, 0, 0)
        const u16* bC = xs + ((q + t1) & 3) * PL + lb + (t1 ? 0 : (2 * PX + 2) * 8);
        f32x4 acc[RW];
#pragma unroll
        for (int r = 0; r < RW; ++r) acc[r] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < NCH; ++c)
#pragma unroll
            for (int s = 0; s < 14; ++s) {
                const int tap = 2 * s, tz = tap / 9, ty = tap / 3 % 3, tx = tap % 3;
                const u16* b = s == 4 ? bC : (tx == 2 ? bB[tz] : bA[tz]) + (ty * PX + tx) * 8;
                if (s == 13) b = bA[2] - t1 * 8 + (2 * PX + 2) * 8;   // tap 26 (lanes 32-63 read it too and drop it)
#pragma unroll
                for (int r = 0; r < RW; ++r) {
                    uint4 xf = *reinterpret_cast<const uint4*>(b + c * PC + r * PX * 8);
                    if (s == 13 && t1) xf = make_uint4(0, 0, 0, 0);
                    acc[r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(wf[c][s]), as_bf16x8(xf), acc[r], 0, 0, 0);
                }
            }
        if (z + 1 < z1) {
            // slot of plane z - 2, last read for output plane z - 1
            put((q + 3) & 3);
            __syncthreads();
        }
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            const uint2 o = conv_epilogue(acc[r], bias, a.relu, MASK, MASK ? mk[r] : make_uint2(0, 0));
            if (!HEAD) {
                if (in[r]) *reinterpret_cast<uint2*>(a.out + (vz + orow[r]) * a.ldo + co) = o;
                continue;
            }
            // head: sum over the 16 channels in order, 4 per lane group (the
            // activations' BF16 values), added to the FP32 input
            const float f[4] = {__uint_as_float(o.x << 16), __uint_as_float(o.x & 0xFFFF0000u),
                                __uint_as_float(o.y << 16), __uint_as_float(o.y & 0xFFFF0000u)};
            auto chain = [&](float t) {
#pragma unroll
                for (int e = 0; e < 4; ++e) t = fmaf(f[e], hwf[e], t);
                return t;
            };
            float t = chain(0.0f);                 // lane group 0
            t = chain(from_row<0>(t));             // group 1 continues group 0's sum
            t = chain(from_row<1>(t));             // group 3, group 1's
            t = chain(from_row<2>(t));             // group 2, group 3's
            if (in[r] && g == 2) a.out32[vz + orow[r]] = xi[r] + (hb + t);
        }
    }
}

// ------------------------------------------------------------ conv3 wgrad
// dW[co][t][ci] = sum_v dz[v][co] x[v + t][ci]: an MFMA GEMM with M = 16
// output channels, N = 16 input channels, K = voxels.  Both operands need 8
// consecutive voxels of one channel per lane: the workgroup stages its 2 x 8 x
// 16 voxel tile as it lies in memory ([voxel][16 channels], dz and the input
// halo) and reads the fragments transposed (ds_read_b64_tr_b16: four voxels of
// one channel per lane; lane group g takes row g / 2 and x half g % 2 of a row
// pair).  Waves 0 to 2 own the nine taps kx = wave; a row pair of the halo
// that the next step's ky = 0 shares with this one's ky = 2 stays in registers.
// The next tile is loaded into registers while one is computed.  A workgroup
// owns one (co tile, ci tile) pair and a strided share of the voxel tiles, and
// writes its FP32 partial sums; the blocks past them sum dz alone, for the bias
// gradient (channel_sums); a second kernel adds both in a fixed order.
// Against fragments transposed through 16-bit LDS writes and three x-shifted
// copies of the halo, and bias sums in launches of their own: the 17
// weight gradients of a training step on four 64^3 crops with their bias sums and
// the adding up 1414 us, now 608 us (382 of them here).
constexpr int WG_T = 256;
constexpr int WG_ITEMS = 2 * 256 + 2 * HVOX;           // 16-byte items: dz tile, then input halo
constexpr int WG_LD = (WG_ITEMS + WG_T - 1) / WG_T;

typedef short s16x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ s16x4 read_tr(const u16* p)
{
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)p);
}

__device__ __forceinline__ bf16x8 join(s16x4 a, s16x4 b)
{
    bf16x8 r;
    __builtin_memcpy(&r, &a, 8);
    __builtin_memcpy(reinterpret_cast<char*>(&r) + 8, &b, 8);
    return r;
}

// Fragment of 8 voxels x 1 channel per lane (two reads of four voxels; rows of
// 16 channels)
__device__ __forceinline__ bf16x8 read_tr8(const u16* p) { return join(read_tr(p), read_tr(p + 4 * 16)); }

// Channel sums of a BF16 tensor of c channels, block blk of nblk of 256 threads:
// partial[blk][c] (FP32).  Thread = (voxel lane, group of 8 channels); the voxel
// lanes' sums go through LDS (red: 2048 floats), where a thread adds those of
// one channel in order.
__device__ __forceinline__ void channel_sums(const u16* __restrict__ t, int ld, int c, int64_t nvox, int blk, int nblk,
                                             float* red, float* __restrict__ partial)
{
    const int groups = c / 8, lanes = 256 / groups;
    const int tid = threadIdx.x, cg = tid % groups, vl = tid / groups;
    float s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (vl < lanes) {
#pragma unroll 4
        for (int64_t v = (int64_t)blk * lanes + vl; v < nvox; v += (int64_t)nblk * lanes) {
            float f[8];
            unpack8(*reinterpret_cast<const uint4*>(t + v * ld + cg * 8), f);
#pragma unroll
            for (int i = 0; i < 8; ++i) s[i] += f[i];
        }
        *reinterpret_cast<float4*>(&red[vl * c + cg * 8]) = make_float4(s[0], s[1], s[2], s[3]);
        *reinterpret_cast<float4*>(&red[vl * c + cg * 8 + 4]) = make_float4(s[4], s[5], s[6], s[7]);
    }
    __syncthreads();
    for (int i = tid; i < c; i += 256) {
        float tot = 0.0f;
#pragma unroll 16
        for (int l = 0; l < lanes; ++l) tot += red[l * c + i];
        partial[(size_t)blk * c + i] = tot;
    }
}

__global__ __launch_bounds__(WG_T) void k_conv3_wgrad(UnetWgrad a, int nsplit, int nbias, float* __restrict__ bias)
{
    __shared__ __attribute__((aligned(16))) u16 ls[WG_ITEMS * 8];
    u16* const dzs = ls;
    u16* const xs = ls + 512 * 8;

    const int cin = a.c0 + a.c1;
    const int ci_tiles = cin / 16, pairs = ci_tiles * (a.cout / 16);
    const int pair = blockIdx.x % pairs, split = blockIdx.x / pairs;
    if (split >= nsplit) {
        channel_sums(a.dz, a.ldz, a.cout, (int64_t)a.n * a.d * a.h * a.w, blockIdx.x - pairs * nsplit, nbias,
                     reinterpret_cast<float*>(ls), bias);
        return;
    }
    const int cot = pair / ci_tiles, cit = pair % ci_tiles;
    const int tid = threadIdx.x, lane = tid & 63, kx = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, li = lane & 15;

    const u16* xsrc;
    int xld;
    if (cit * 16 < a.c0) {
        xsrc = a.in0 + cit * 16;
        xld = a.ld0;
    } else {
        xsrc = a.in1 + (cit * 16 - a.c0);
        xld = a.ld1;
    }
    const u16* dsrc = a.dz + cot * 16;

    const int tiles_x = (a.w + CX - 1) / CX, tiles_y = (a.h + CY - 1) / CY, tiles_z = (a.d + CZ - 1) / CZ;
    const int ntiles = tiles_x * tiles_y * tiles_z * a.n;
    const size_t plane = (size_t)a.h * a.w;

    // this thread's items tid + 256 m: tile-relative voxel (x, y, z), the halo's from -1
    int lx[WG_LD], ly[WG_LD], lz[WG_LD];
#pragma unroll
    for (int m = 0; m < WG_LD; ++m) {
        const int i = tid + WG_T * m;
        if (i < 512) {
            const int v = i >> 1;
            lx[m] = v & 15;
            ly[m] = (v >> 4) & 7;
            lz[m] = v >> 7;
        } else {
            const int v = (i - 512) >> 1;
            lx[m] = v % HX - 1;
            ly[m] = (v / HX) % HY - 1;
            lz[m] = v / (HX * HY) - 1;
        }
    }
    uint4 pf[WG_LD];
    auto fetch = [&](int t) {
        int rem = t;
        const int x0 = (rem % tiles_x) * CX;
        rem /= tiles_x;
        const int y0 = (rem % tiles_y) * CY;
        rem /= tiles_y;
        const int z0 = (rem % tiles_z) * CZ;
        const size_t vbase = (size_t)(rem / tiles_z) * a.d * plane;
#pragma unroll
        for (int m = 0; m < WG_LD; ++m) {
            const int i = tid + WG_T * m;
            const int gx = x0 + lx[m], gy = y0 + ly[m], gz = z0 + lz[m];
            pf[m] = make_uint4(0, 0, 0, 0);
            if (i < WG_ITEMS && gx >= 0 && gx < a.w && gy >= 0 && gy < a.h && gz >= 0 && gz < a.d) {
                const size_t v = vbase + (size_t)gz * plane + (size_t)gy * a.w + gx;
                pf[m] = *reinterpret_cast<const uint4*>((i < 512 ? dsrc + v * a.ldz : xsrc + v * xld) + (tid & 1) * 8);
            }
        }
    };

    f32x4 acc[3][3];   // [kz][ky]
#pragma unroll
    for (int j = 0; j < 9; ++j) acc[j / 3][j % 3] = f32x4{0.f, 0.f, 0.f, 0.f};
    // this lane's read addresses within a row pair
    const int la = ((g >> 1) * CX + 8 * (g & 1) + (li >> 2)) * 16 + (li & 3) * 4;
    const int lb = ((g >> 1) * HX + 8 * (g & 1) + (li >> 2) + kx) * 16 + (li & 3) * 4;

    fetch(split);
    for (int t = split; t < ntiles; t += nsplit) {
        __syncthreads();   // the previous tile's fragments have been read
#pragma unroll
        for (int m = 0; m < WG_LD; ++m) {
            const int i = tid + WG_T * m;
            if (i < WG_ITEMS) *reinterpret_cast<uint4*>(&ls[i * 8]) = pf[m];
        }
        __syncthreads();
        if (t + nsplit < ntiles) fetch(t + nsplit);
        if (kx == 3) continue;   // the fourth wave only loads
#pragma unroll
        for (int zl = 0; zl < CZ; ++zl) {
            bf16x8 first[3];
#pragma unroll
            for (int kz = 0; kz < 3; ++kz) first[kz] = read_tr8(xs + lb + (zl + kz) * HY * HX * 16);
#pragma unroll
            for (int y = 0; y < CY; y += 2) {
                const bf16x8 af = read_tr8(dzs + la + (zl * CY + y) * CX * 16);
#pragma unroll
                for (int kz = 0; kz < 3; ++kz) {
                    const u16* row = xs + lb + ((zl + kz) * HY + y) * HX * 16;
                    const bf16x8 b1 = read_tr8(row + HX * 16), b2 = read_tr8(row + 2 * HX * 16);
                    acc[kz][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, first[kz], acc[kz][0], 0, 0, 0);
                    acc[kz][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, b1, acc[kz][1], 0, 0, 0);
                    acc[kz][2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, b2, acc[kz][2], 0, 0, 0);
                    first[kz] = b2;
                }
            }
        }
    }
    if (kx == 3) return;

    // partial[split][co][t][ci]: lane holds rows co = 4g + e, column ci = li
    float* part = a.partial + (size_t)split * a.cout * 27 * cin;
#pragma unroll
    for (int j = 0; j < 9; ++j) {
        const int tap = 3 * j + kx;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int co = cot * 16 + 4 * g + e;
            part[((size_t)co * 27 + tap) * cin + cit * 16 + li] = acc[j / 3][j % 3][e];
        }
    }
}

// dw[i] (+)= sum over k of partial[k][i], k < nsplit, i < nw, and db[i] (+)= the
// sum over k of bias[k][i], k < nbias, i < nb: a 256-thread block takes 32
// consecutive i and 8 lanes of k (lane l sums k = l mod 8 in order), then one
// thread adds the 8 lane sums in order: a fixed summation order, so the result
// is reproducible.  Latency bounds it (each sum is a chain of up to 128 adds):
// SUM_F loads are in flight per thread, and dw and db share a launch.
constexpr int SUM_E = 32, SUM_L = 8, SUM_F = 32;
__global__ __launch_bounds__(256) void k_sum_partials(const float* __restrict__ partial, int nsplit, int64_t nw,
                                                      const float* __restrict__ bias, int nbias, int nb,
                                                      float* __restrict__ dw, float* __restrict__ db, int accumulate)
{
    __shared__ float red[SUM_L][SUM_E];
    const int64_t dwb = (nw + SUM_E - 1) / SUM_E;
    int64_t i0 = (int64_t)blockIdx.x * SUM_E, n = nw;
    const float* p = partial;
    float* out = dw;
    if (blockIdx.x >= dwb) {
        i0 -= dwb * SUM_E;
        n = nb;
        p = bias;
        out = db;
        nsplit = nbias;
    }
    const int e = threadIdx.x % SUM_E, l = threadIdx.x / SUM_E;
    const int64_t i = i0 + e;
    float s = 0.0f;
    if (i < n) {
        const float* q = p + i + l * n;
        int k = l;
        for (; k + (SUM_F - 1) * SUM_L < nsplit; k += SUM_F * SUM_L, q += SUM_F * SUM_L * n) {
            float v[SUM_F];
#pragma unroll
            for (int j = 0; j < SUM_F; ++j) v[j] = q[j * SUM_L * n];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < SUM_F; ++j) s += v[j];
        }
        float v[SUM_F];
#pragma unroll
        for (int j = 0; j < SUM_F; ++j) v[j] = k + j * SUM_L < nsplit ? q[j * SUM_L * n] : 0.0f;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < SUM_F; ++j) s = k + j * SUM_L < nsplit ? s + v[j] : s;
    }
    red[l][e] = s;
    __syncthreads();
    if (l == 0 && i < n) {
        float t = red[0][e];
#pragma unroll
        for (int m = 1; m < SUM_L; ++m) t += red[m][e];
        out[i] = accumulate ? out[i] + t : t;
    }
}

// ------------------------------------------------------------------ misc
// x (FP32, one channel) -> BF16 [v][16] with channel 0 = x, others 0: the
// first convolution then runs on the same MFMA kernel
__global__ void k_pack_input(const float* __restrict__ x, int64_t nvox, u16* __restrict__ out)
{
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= nvox) return;
    uint4* o = reinterpret_cast<uint4*>(out + v * 16);
    o[0] = make_uint4((uint32_t)f2bf(x[v]), 0, 0, 0);
    o[1] = make_uint4(0, 0, 0, 0);
}

// 2x2x2 average pooling, 8 channels per thread
__global__ void k_pool2(const u16* __restrict__ in, int ldi, int n, int d, int h, int w, int c, u16* __restrict__ out,
                        int ldo)
{
    const int groups = c / 8;
    const int64_t total = (int64_t)n * d * h * w * groups;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= total) return;
    const bool small = total < (int64_t)1 << 31;
    const int64_t v = small ? (int64_t)((unsigned)i / (unsigned)groups) : i / groups;
    const int cg = (int)(i - v * groups);
    const Vox q = vox_of(v, total / groups, d, h, w);
    const int x = q.x, y = q.y, z = q.z, nb = q.n;
    float s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int k = 0; k < 8; ++k) {
        const int zz = 2 * z + (k >> 2), yy = 2 * y + ((k >> 1) & 1), xx = 2 * x + (k & 1);
        const size_t fv = (((size_t)nb * 2 * d + zz) * 2 * h + yy) * 2 * w + xx;
        float f[8];
        unpack8(*reinterpret_cast<const uint4*>(in + fv * ldi + cg * 8), f);
#pragma unroll
        for (int e = 0; e < 8; ++e) s[e] += f[e];
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) s[e] *= 0.125f;
    const size_t cv = (((size_t)nb * d + z) * h + y) * w + x;
    *reinterpret_cast<uint4*>(out + cv * ldo + cg * 8) = pack8(s);
}

// gradient at a skip tensor e (fine grid) that feeds both a pooling and a
// concatenation: dz = mask(e) * (dp[parent] / 8 + dcat), rounded to BF16
__global__ void k_skip_grad(const u16* __restrict__ e, int lde, const u16* __restrict__ dp, int ldp,
                            const u16* __restrict__ dcat, int ldc, int n, int d, int h, int w, int c,
                            u16* __restrict__ out, int ldo)
{
    const int groups = c / 8;
    const int64_t total = (int64_t)n * d * h * w * groups;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= total) return;
    const bool small = total < (int64_t)1 << 31;
    const int64_t v = small ? (int64_t)((unsigned)i / (unsigned)groups) : i / groups;
    const int cg = (int)(i - v * groups);
    const Vox q = vox_of(v, total / groups, d, h, w);
    const int x = q.x, y = q.y, z = q.z, nb = q.n;
    const size_t fv = (((size_t)nb * d + z) * h + y) * w + x;
    const size_t pv = (((size_t)nb * (d / 2) + z / 2) * (h / 2) + y / 2) * (w / 2) + x / 2;
    float fe[8], fp[8], fc[8];
    const uint4 qe = *reinterpret_cast<const uint4*>(e + fv * lde + cg * 8);
    unpack8(*reinterpret_cast<const uint4*>(dp + pv * ldp + cg * 8), fp);
    unpack8(*reinterpret_cast<const uint4*>(dcat + fv * ldc + cg * 8), fc);
    unpack8(qe, fe);
    float o[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) o[k] = (fe[k] > 0.0f) ? fp[k] * 0.125f + fc[k] : 0.0f;
    *reinterpret_cast<uint4*>(out + fv * ldo + cg * 8) = pack8(o);
}

// stride-2 2x2x2 transposed convolution: out[2v + s][co] =
// bf16(b[co] + sum_ci x[v][ci] w[co][s][ci]); thread = (fine voxel, 8 co)
__global__ void k_up2(const u16* __restrict__ x, int ldx, int cin, const u16* __restrict__ wt,
                      const float* __restrict__ bias, int cout, int n, int d, int h, int w, u16* __restrict__ out,
                      int ldo)
{
    const int groups = cout / 8;
    const int D = 2 * d, H = 2 * h, W = 2 * w;
    const int64_t total = (int64_t)n * D * H * W * groups;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= total) return;
    const int cg = (int)(i % groups);
    int64_t v = i / groups;
    const int X = (int)(v % W);
    v /= W;
    const int Y = (int)(v % H);
    v /= H;
    const int Z = (int)(v % D);
    const int nb = (int)(v / D);
    const int s = ((Z & 1) << 2) | ((Y & 1) << 1) | (X & 1);
    const size_t cv = (((size_t)nb * d + (Z >> 1)) * h + (Y >> 1)) * w + (X >> 1);
    float acc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = bias ? bias[cg * 8 + e] : 0.0f;
    const u16* xp = x + cv * ldx;
    for (int c8 = 0; c8 < cin; c8 += 8) {
        float fx[8];
        unpack8(*reinterpret_cast<const uint4*>(xp + c8), fx);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float fw[8];
            unpack8(*reinterpret_cast<const uint4*>(wt + ((size_t)(cg * 8 + e) * 8 + s) * cin + c8), fw);
#pragma unroll
            for (int k = 0; k < 8; ++k) acc[e] = fmaf(fx[k], fw[k], acc[e]);
        }
    }
    const size_t fv = (((size_t)nb * D + Z) * H + Y) * W + X;
    *reinterpret_cast<uint4*>(out + fv * ldo + cg * 8) = pack8(acc);
}

// The same transposed convolution on the BF16 MFMA (16x16x32, FP32
// accumulators), for cin a multiple of 32 and cout of 16 * NT: per
// sub-position s, D_s[co][v] = sum_ci W[co][s][ci] X[ci][v] is a GEMM with
// M = cout, N = coarse voxels, K = cin.  A wave owns 16 consecutive coarse
// voxels (the N columns; lane li reads 8 consecutive channels of voxel
// v0 + li, a 16-byte load from the channels-last row) and computes all eight
// sub-positions and all output channels, so every input row is read once;
// the weights (at most 64 x 8 x 128 BF16) come through L1/L2.  Lane
// (li, g) ends with channels 16 nt + 4 g .. + 3 of fine voxel 2 v + s.
template <int NT>
__global__ __launch_bounds__(256) void k_up2_mfma(const u16* __restrict__ x, int ldx, int cin,
                                                  const u16* __restrict__ wt, const float* __restrict__ bias, int n,
                                                  int d, int h, int w, u16* __restrict__ out, int ldo)
{
    const int lane = threadIdx.x & 63, g = lane >> 4, li = lane & 15;
    const int64_t nvox = (int64_t)n * d * h * w;
    const int64_t v0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 16;
    if (v0 >= nvox) return;   // uniform over the wave
    const bool vok = v0 + li < nvox;
    const u16* xr = x + (vok ? v0 + li : v0) * ldx + 8 * g;
    // The fine voxels that this lane writes: sub-position odd (li / 8) along x of
    // coarse voxels v0 + li % 8 and 8 further
    const int odd = li >> 3;
    const int64_t va = v0 + (li & 7), vb = va + 8;
    const bool aok = va < nvox, bok = vb < nvox;
    const Vox pa = vox_of(aok ? va : v0, nvox, d, h, w), pb = vox_of(bok ? vb : v0, nvox, d, h, w);
    const int D = 2 * d, H = 2 * h, W = 2 * w;
    const size_t fa = (((size_t)pa.n * D + 2 * pa.z) * H + 2 * pa.y) * W + 2 * pa.x + odd;
    const size_t fb = (((size_t)pb.n * D + 2 * pb.z) * H + 2 * pb.y) * W + 2 * pb.x + odd;
    // this workgroup's output channels and sub-positions
    const int cb = (int)blockIdx.y * 16 * NT, ns = 4 / (int)gridDim.z;
    // two sub-positions along x at a time (the input row stays in L1 between them)
    for (int sp = (int)blockIdx.z * ns; sp < ((int)blockIdx.z + 1) * ns; ++sp) {
        f32x4 acc[2][NT];
#pragma unroll
        for (int q = 0; q < 2 * NT; ++q) acc[q / NT][q % NT] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int kc = 0; kc < cin; kc += 32) {
            const bf16x8 xb = as_bf16x8(vok ? *reinterpret_cast<const uint4*>(xr + kc) : make_uint4(0, 0, 0, 0));
#pragma unroll
            for (int q = 0; q < 2 * NT; ++q) {
                const uint4 wf = *reinterpret_cast<const uint4*>(
                    wt + ((size_t)(cb + q % NT * 16 + li) * 8 + 2 * sp + q / NT) * cin + kc + 8 * g);
                acc[q / NT][q % NT] =
                    __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(wf), xb, acc[q / NT][q % NT], 0, 0, 0);
            }
        }
        // The accumulators are read right after the last MFMA; the compiler
        // left too few wait states there (the first two of each four read
        // stale values), so 24 explicit ones are placed between the MFMAs
        // that define them and the reads, pinned by in/out operands.
#pragma unroll
        for (int q = 0; q < 2 * NT; ++q)
            asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" : "+a"(acc[q / NT][q % NT]));
        const size_t so = ((size_t)(sp >> 1) * H + (sp & 1)) * W;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const int co = cb + nt * 16 + 4 * g;
            uint2 o[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                float f[4] = {acc[q][nt][0], acc[q][nt][1], acc[q][nt][2], acc[q][nt][3]};
                if (bias) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) f[e] += bias[co + e];
                }
                o[q].x = (uint32_t)f2bf(f[0]) | ((uint32_t)f2bf(f[1]) << 16);
                o[q].y = (uint32_t)f2bf(f[2]) | ((uint32_t)f2bf(f[3]) << 16);
            }
            // Each store covers both sub-positions of eight voxels (rows without
            // gaps) instead of one of sixteen: lanes li and li ^ 8 exchange
            // what the other one writes.
            const uint2 send = odd ? o[0] : o[1];
            uint2 recv;
            recv.x = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)send.x, 0x128, 0xf, 0xf, false);   // row_ror:8
            recv.y = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)send.y, 0x128, 0xf, 0xf, false);
            if (aok) *reinterpret_cast<uint2*>(out + (fa + so) * ldo + co) = odd ? recv : o[0];
            if (bok) *reinterpret_cast<uint2*>(out + (fb + so) * ldo + co) = odd ? o[1] : recv;
        }
    }
}

// data gradient of up2 with the ReLU mask of its input:
// dx[v][ci] = bf16(mask(below[v][ci]) sum_s sum_co g[2v + s][co] w[co][s][ci])
__global__ void k_up2_dgrad(const u16* __restrict__ gr, int ldg, int cout, const u16* __restrict__ wt, int cin,
                            const u16* __restrict__ below, int ldb, int n, int d, int h, int w, u16* __restrict__ out,
                            int ldo)
{
    const int groups = cin / 8;
    const int64_t total = (int64_t)n * d * h * w * groups;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= total) return;
    const int cg = (int)(i % groups);
    int64_t v = i / groups;
    const int x = (int)(v % w);
    v /= w;
    const int y = (int)(v % h);
    v /= h;
    const int z = (int)(v % d);
    const int nb = (int)(v / d);
    float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int s = 0; s < 8; ++s) {
        const int Z = 2 * z + (s >> 2), Y = 2 * y + ((s >> 1) & 1), X = 2 * x + (s & 1);
        const size_t fv = (((size_t)nb * 2 * d + Z) * 2 * h + Y) * 2 * w + X;
        const u16* gp = gr + fv * ldg;
        for (int c8 = 0; c8 < cout; c8 += 8) {
            float fg[8];
            unpack8(*reinterpret_cast<const uint4*>(gp + c8), fg);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                float fw[8];
                unpack8(*reinterpret_cast<const uint4*>(wt + ((size_t)(c8 + e) * 8 + s) * cin + cg * 8), fw);
#pragma unroll
                for (int k = 0; k < 8; ++k) acc[k] = fmaf(fg[e], fw[k], acc[k]);
            }
        }
    }
    const size_t cv = (((size_t)nb * d + z) * h + y) * w + x;
    if (below) {
        float fb[8];
        unpack8(*reinterpret_cast<const uint4*>(below + cv * ldb + cg * 8), fb);
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (!(fb[k] > 0.0f)) acc[k] = 0.0f;
    }
    *reinterpret_cast<uint4*>(out + cv * ldo + cg * 8) = pack8(acc);
}

// The same data gradient on the MFMA: D[ci][v] = sum_k W'[ci][k] G[k][v]
// with k = s cout + co, W'[ci][s cout + co] = w[co][s][ci] and G[k][v] =
// g[2v + s][co].  A wave owns 2 x 16 coarse voxels (B columns: lane li
// reads 8 consecutive co of fine voxel 2v + s, one 16-byte load); the
// workgroup stages each 32-wide k chunk of W' transposed in LDS ([ci][32],
// one 16-byte A fragment per lane and ci tile).  Lane (li, g) ends with
// ci = 16 nt + 4 g .. + 3 of voxel v0 + li.
constexpr int UPD_VG = 2;   // 16-voxel groups per wave
template <int NT>
__global__ __launch_bounds__(256) void k_up2_dgrad_mfma(const u16* __restrict__ gr, int ldg, int cout,
                                                        const u16* __restrict__ wt, int cin,
                                                        const u16* __restrict__ below, int ldb, int n, int d, int h,
                                                        int w, u16* __restrict__ out, int ldo)
{
    constexpr int CIN = 16 * NT, WS = 40;   // this workgroup's channels; LDS row stride (u16): 32 k + 8 pad
    __shared__ __attribute__((aligned(16))) u16 wl[CIN * WS];
    const int cb = (int)blockIdx.y * CIN;
    const int lane = threadIdx.x & 63, g = lane >> 4, li = lane & 15;
    const int64_t nvox = (int64_t)n * d * h * w;
    const int64_t vw = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * (16 * UPD_VG);   // the wave's first voxel
    const int D2 = 2 * d, H2 = 2 * h, W2 = 2 * w;
    int64_t fb[UPD_VG];   // fine index of sub-position 0 of each group's voxel
    bool vok[UPD_VG];
#pragma unroll
    for (int q = 0; q < UPD_VG; ++q) {
        const int64_t v = vw + 16 * q + li;
        vok[q] = v < nvox;
        const Vox p = vox_of(vok[q] ? v : 0, nvox, d, h, w);
        fb[q] = (((int64_t)p.n * D2 + 2 * p.z) * H2 + 2 * p.y) * W2 + 2 * p.x;
    }
    f32x4 acc[UPD_VG][NT];
#pragma unroll
    for (int q = 0; q < UPD_VG; ++q)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[q][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int K = 8 * cout;
    for (int kc = 0; kc < K; kc += 32) {
        __syncthreads();   // the previous chunk's fragments have been read
        for (int i = threadIdx.x; i < CIN * 32; i += 256) {
            const int ci = i % CIN, kk = i / CIN;   // consecutive threads read consecutive ci
            const int k = kc + kk, s = k / cout, co = k - s * cout;
            wl[ci * WS + kk] = wt[((size_t)co * 8 + s) * cin + cb + ci];
        }
        __syncthreads();
        const int k = kc + 8 * g, s = k / cout, co0 = k - s * cout;
        const int64_t so = ((int64_t)(s >> 2) * H2 + ((s >> 1) & 1)) * W2 + (s & 1);   // fine offset of sub-position s
        bf16x8 af[NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
            af[nt] = as_bf16x8(*reinterpret_cast<const uint4*>(&wl[(nt * 16 + li) * WS + 8 * g]));
#pragma unroll
        for (int q = 0; q < UPD_VG; ++q) {
            const uint4 gq = vok[q] ? *reinterpret_cast<const uint4*>(gr + (fb[q] + so) * ldg + co0)
                                    : make_uint4(0, 0, 0, 0);
            const bf16x8 gb = as_bf16x8(gq);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                acc[q][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[nt], gb, acc[q][nt], 0, 0, 0);
        }
    }
    // explicit wait states between the last MFMAs and the reads of their
    // results (as in k_up2_mfma)
#pragma unroll
    for (int q = 0; q < UPD_VG; ++q)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" : "+a"(acc[q][nt]));
#pragma unroll
    for (int q = 0; q < UPD_VG; ++q) {
        if (!vok[q]) continue;
        const int64_t v = vw + 16 * q + li;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const int ci = cb + nt * 16 + 4 * g;
            float o[4] = {acc[q][nt][0], acc[q][nt][1], acc[q][nt][2], acc[q][nt][3]};
            if (below) {
                const uint2 m = *reinterpret_cast<const uint2*>(below + v * ldb + ci);
                if (!bf_pos((u16)(m.x & 0xFFFF))) o[0] = 0.0f;
                if (!bf_pos((u16)(m.x >> 16))) o[1] = 0.0f;
                if (!bf_pos((u16)(m.y & 0xFFFF))) o[2] = 0.0f;
                if (!bf_pos((u16)(m.y >> 16))) o[3] = 0.0f;
            }
            uint2 pk;
            pk.x = (uint32_t)f2bf(o[0]) | ((uint32_t)f2bf(o[1]) << 16);
            pk.y = (uint32_t)f2bf(o[2]) | ((uint32_t)f2bf(o[3]) << 16);
            *reinterpret_cast<uint2*>(out + v * ldo + ci) = pk;
        }
    }
}

// Weight gradient of up2 on the MFMA: dw[co][s][ci] = sum_v g[2v + s][co]
// x[v][ci], per (s, co tile, ci tile) block a 16 x 16 GEMM with K = coarse
// voxels.  Each wave stages its 64-voxel chunk in LDS as it lies in memory
// ([voxel][16 channels]), the next chunk being loaded meanwhile, and reads both
// operands transposed (as in k_conv3_wgrad).  The block's four waves take
// interleaved chunks of its voxel share and add their sums in a fixed order at
// the end (partial[split][co][s][ci]); the blocks past them sum g alone, for the
// bias gradient.
__global__ __launch_bounds__(256) void k_up2_wgrad_mfma(const u16* __restrict__ x, int ldx, int cin,
                                                        const u16* __restrict__ gr, int ldg, int cout, int n, int d,
                                                        int h, int w, float* __restrict__ partial, int nsplit,
                                                        int nbias, float* __restrict__ bias)
{
    __shared__ __attribute__((aligned(16))) u16 gt[4][64 * 16];
    __shared__ __attribute__((aligned(16))) u16 xt[4][64 * 16];
    __shared__ __attribute__((aligned(16))) float red[4][512];
    const int ci_tiles = cin / 16, co_tiles = cout / 16;
    const int blocks = 8 * ci_tiles * co_tiles;
    int b = blockIdx.x % blocks;
    const int cit = b % ci_tiles;
    b /= ci_tiles;
    const int cot = b % co_tiles;
    const int s = b / co_tiles;
    const int split = blockIdx.x / blocks;
    if (split >= nsplit) {
        channel_sums(gr, ldg, cout, (int64_t)n * 8 * d * h * w, blockIdx.x - blocks * nsplit, nbias, red[0], bias);
        return;
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane >> 4, li = lane & 15;
    const int64_t nvox = (int64_t)n * d * h * w;
    const int64_t nchunks = (nvox + 63) / 64;
    const int64_t mine = nchunks > split ? (nchunks - split + nsplit - 1) / nsplit : 0;   // chunks of this split
    const int64_t rounds = (mine + 3) / 4;
    const int D2 = 2 * d, H2 = 2 * h, W2 = 2 * w;
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
    const int lv = (8 * g + (li >> 2)) * 16 + (li & 3) * 4;
    uint4 g0, g1, x0, x1;
    auto fetch = [&](int64_t it) {
        const int64_t j = 4 * it + wave;               // this wave's chunk in the split's list
        const int64_t v = (split + j * nsplit) * 64 + lane;
        g0 = g1 = x0 = x1 = make_uint4(0, 0, 0, 0);
        if (j < mine && v < nvox) {
            const Vox p = vox_of(v, nvox, d, h, w);
            const int64_t fv =
                (((int64_t)p.n * D2 + 2 * p.z + (s >> 2)) * H2 + 2 * p.y + ((s >> 1) & 1)) * W2 + 2 * p.x + (s & 1);
            const u16* gp = gr + fv * ldg + cot * 16;
            const u16* xp = x + v * ldx + cit * 16;
            g0 = *reinterpret_cast<const uint4*>(gp);
            g1 = *reinterpret_cast<const uint4*>(gp + 8);
            x0 = *reinterpret_cast<const uint4*>(xp);
            x1 = *reinterpret_cast<const uint4*>(xp + 8);
        }
    };
    fetch(0);
    for (int64_t it = 0; it < rounds; ++it) {
        __syncthreads();   // every wave has read the previous chunk's fragments
        *reinterpret_cast<uint4*>(&gt[wave][lane * 16]) = g0;
        *reinterpret_cast<uint4*>(&gt[wave][lane * 16 + 8]) = g1;
        *reinterpret_cast<uint4*>(&xt[wave][lane * 16]) = x0;
        *reinterpret_cast<uint4*>(&xt[wave][lane * 16 + 8]) = x1;
        __syncthreads();
        if (it + 1 < rounds) fetch(it + 1);
#pragma unroll
        for (int kk = 0; kk < 64; kk += 32) {
            const bf16x8 af = read_tr8(&gt[wave][kk * 16 + lv]);
            const bf16x8 bf = read_tr8(&xt[wave][kk * 16 + lv]);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, bf, acc, 0, 0, 0);
        }
    }
    asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" : "+a"(acc));
    // lane (li, g) holds dW rows co = 4 g .. 4 g + 3 of column ci = li
#pragma unroll
    for (int e = 0; e < 4; ++e) red[wave][(4 * g + e) * 16 + li] = acc[e];
    __syncthreads();
    const int t = threadIdx.x, co_l = t >> 4, ci_l = t & 15;
    const float sum = ((red[0][t] + red[1][t]) + red[2][t]) + red[3][t];
    float* part = partial + (size_t)split * cout * 8 * cin;
    part[((size_t)(cot * 16 + co_l) * 8 + s) * cin + cit * 16 + ci_l] = sum;
}

// residual head: out[v] = x_in[v] + hb + sum_c hw[c] a[v][c] (FP32)
__global__ void k_head(const float* __restrict__ xin, const u16* __restrict__ act, int lda, int c,
                       const u16* __restrict__ hw, const float* __restrict__ hb, int64_t nvox, float* __restrict__ out)
{
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= nvox) return;
    float s = 0.0f;
    for (int c8 = 0; c8 < c; c8 += 8) {
        float fa[8];
        unpack8(*reinterpret_cast<const uint4*>(act + v * lda + c8), fa);
#pragma unroll
        for (int k = 0; k < 8; ++k) s = fmaf(fa[k], bf2f(hw[c8 + k]), s);
    }
    out[v] = xin[v] + (hb[0] + s);
}

// MSE loss through the head (16 channels): g = 2 (out - t) / M; dz[v][c] =
// bf16(g hw[c] mask(a[v][c])); per-block FP64 partial sums of g a[v][c]
// (16 columns), of g, and of (out - t)^2 -> partial[block][18]
constexpr int HEAD_C = 16;

__global__ __launch_bounds__(256) void k_head_loss_bwd(const float* __restrict__ out, const float* __restrict__ tgt,
                                                       const u16* __restrict__ act, int lda,
                                                       const u16* __restrict__ hw, int64_t nvox, double inv_m,
                                                       u16* __restrict__ dz, int ldz, double* __restrict__ partial)
{
    __shared__ double red[256];
    const int tid = threadIdx.x;
    float hwf[HEAD_C];
#pragma unroll
    for (int k = 0; k < HEAD_C; ++k) hwf[k] = bf2f(hw[k]);
    double s[HEAD_C + 2];
#pragma unroll
    for (int k = 0; k < HEAD_C + 2; ++k) s[k] = 0.0;
    for (int64_t v = (int64_t)blockIdx.x * 256 + tid; v < nvox; v += (int64_t)gridDim.x * 256) {
        const float diff = out[v] - tgt[v];
        const float gv = (float)(2.0 * inv_m) * diff;
#pragma unroll
        for (int c8 = 0; c8 < HEAD_C; c8 += 8) {
            float fa[8], o[8];
            unpack8(*reinterpret_cast<const uint4*>(act + v * lda + c8), fa);
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                s[c8 + k] += (double)gv * fa[k];
                o[k] = fa[k] > 0.0f ? gv * hwf[c8 + k] : 0.0f;
            }
            *reinterpret_cast<uint4*>(dz + v * ldz + c8) = pack8(o);
        }
        s[HEAD_C] += gv;
        s[HEAD_C + 1] += (double)diff * diff;
    }
#pragma unroll
    for (int k = 0; k < HEAD_C + 2; ++k) {
        red[tid] = s[k];
        __syncthreads();
        for (int st = 128; st > 0; st >>= 1) {
            if (tid < st) red[tid] += red[tid + st];
            __syncthreads();
        }
        if (tid == 0) partial[(size_t)blockIdx.x * (HEAD_C + 2) + k] = red[0];
        __syncthreads();
    }
}

// out[i] = sum_k partial[k][i] in FP64, one block per column i (lane l sums the
// terms l mod 256 in order, then a tree: a fixed order); the first nf sums also
// go to outf as FP32 when outf is given
__global__ __launch_bounds__(256) void k_sum_partials64(const double* __restrict__ partial, int nsplit, int n,
                                                        double* __restrict__ out, float* __restrict__ outf, int nf)
{
    __shared__ double red[256];
    const int i = blockIdx.x, tid = threadIdx.x;
    double s = 0.0;
    for (int k = tid; k < nsplit; k += 256) s += partial[(size_t)k * n + i];
    red[tid] = s;
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if (tid < st) red[tid] += red[tid + st];
        __syncthreads();
    }
    if (tid == 0) {
        out[i] = red[0];
        if (outf && i < nf) outf[i] = (float)red[0];
    }
}

// Adam on FP32 master weights (bias-corrected step sizes from the host):
// m = b1 m + (1 - b1) g; v = b2 v + (1 - b2) g^2;
// w -= lr_t m / (sqrt(v) / sqrt(1 - b2^t) + eps), lr_t = lr / (1 - b1^t)
__global__ void k_adam(float* __restrict__ w, float* __restrict__ m, float* __restrict__ v,
                       const float* __restrict__ gr, int64_t n, float b1, float b2, float lr_t, float inv_sqrt_bc2,
                       float eps)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float g = gr[i];
    const float mi = fmaf(b1, m[i], (1.0f - b1) * g);
    const float vi = fmaf(b2, v[i], (1.0f - b2) * g * g);
    m[i] = mi;
    v[i] = vi;
    w[i] -= lr_t * mi / (sqrtf(vi) * inv_sqrt_bc2 + eps);
}

// FP32 [cout][27][cin] -> BF16 forward weights (same layout) and, if wd is
// given, BF16 data-gradient weights wd[ci][26 - t][co]
__global__ void k_pack_conv3(const float* __restrict__ w, int cout, int cin, u16* __restrict__ wf, u16* __restrict__ wd)
{
    const int64_t n = (int64_t)cout * 27 * cin;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int ci = (int)(i % cin);
    const int t = (int)((i / cin) % 27);
    const int co = (int)(i / ((int64_t)27 * cin));
    const u16 q = f2bf(w[i]);
    wf[i] = q;
    if (wd) wd[((size_t)ci * 27 + (26 - t)) * cout + co] = q;
}

__global__ void k_to_bf16(const float* __restrict__ a, int64_t n, u16* __restrict__ out)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = f2bf(a[i]);
}

inline unsigned blocks_for(int64_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }

}  // namespace

// k_conv3z marches over zc planes: 32 where the volume gives the 256 CUs a
// few workgroups each that way, fewer where it does not (each march stages two
// planes more than it computes)
template <int NCH, int NTW, bool FIRST = false, bool HEAD = false>
static hipError_t launch_conv3z(const UnetConv3& a, hipStream_t s)
{
    constexpr int YT = march_rows<NCH>();
    const int64_t cols = (int64_t)((a.w + CX - 1) / CX) * ((a.h + YT - 1) / YT) * (a.cout / (16 * NTW));
    int zc = 32;
    while (zc > 2 && cols * a.n * ((a.d + zc - 1) / zc) < 1024) zc >>= 1;
    const dim3 grid((unsigned)cols, (a.d + zc - 1) / zc, a.n);
    if (!FIRST && !HEAD && a.mask)
        k_conv3z<NCH, NTW, false, false, true><<<grid, 256, 0, s>>>(a, zc);
    else
        k_conv3z<NCH, NTW, FIRST, HEAD, false><<<grid, 256, 0, s>>>(a, zc);
    return hipGetLastError();
}

hipError_t launch_unet_conv3(const UnetConv3& a, hipStream_t s)
{
    const int cin = a.c0 + a.c1;
    const int64_t plane = (int64_t)a.h * a.w;
    // up to 32 input channels: the z march (its lane offsets are 32-bit, and
    // a chunk of 16 channels comes from one tensor)
    if (cin <= 32 && a.c0 % 16 == 0 && plane * std::max(a.ld0, a.ld1) < (int64_t)1 << 30 && a.d <= 65535 * 2) {
        if (cin == 16) return a.cout == 16 ? launch_conv3z<1, 1>(a, s) : launch_conv3z<1, 2>(a, s);
        return a.cout == 16 ? launch_conv3z<2, 1>(a, s) : launch_conv3z<2, 2>(a, s);
    }
    const int tiles = ((a.w + CX - 1) / CX) * ((a.h + CY - 1) / CY), tiles_z = (a.d + CZ - 1) / CZ;
    // output channels per workgroup: all of them (the halo is then read once), or
    // fewer (down to 16) where the tiles alone leave most of the 256 CUs idle (the
    // deep levels of four 64^3 crops: 38 to 101 us per layer with all, 19 us with 16)
    int nt = a.cout / 16;
    while (nt > 1 && (int64_t)tiles * tiles_z * a.n * (a.cout / (16 * nt)) < 512) nt >>= 1;
    const dim3 grid(tiles * (a.cout / (16 * nt)), tiles_z, a.n);
    switch (nt) {
    case 1: k_conv3<1><<<grid, 256, 0, s>>>(a); break;
    case 2: k_conv3<2><<<grid, 256, 0, s>>>(a); break;
    case 4: k_conv3<4><<<grid, 256, 0, s>>>(a); break;
    case 8: k_conv3<8><<<grid, 256, 0, s>>>(a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_unet_conv3_first(const UnetConv3& a, hipStream_t s) { return launch_conv3z<1, 1, true>(a, s); }

hipError_t launch_unet_conv3_head(const UnetConv3& a, hipStream_t s) { return launch_conv3z<1, 1, false, true>(a, s); }

int unet_wgrad_splits(int n, int d, int h, int w, int cin, int cout)
{
    const int64_t tiles = (int64_t)n * ((d + CZ - 1) / CZ) * ((h + CY - 1) / CY) * ((w + CX - 1) / CX);
    const int pairs = (cin / 16) * (cout / 16);
    int64_t sp = 1024 / pairs;
    if (sp < 1) sp = 1;
    if (sp > tiles) sp = tiles;
    return (int)sp;
}

// Blocks of a bias gradient's channel sums over nvox voxels
static int bias_blocks(int64_t nvox) { return (int)std::min<int64_t>(1024, std::max<int64_t>(1, nvox / 1024)); }

size_t unet_wgrad_ws_bytes(int n, int d, int h, int w, int cin, int cout)
{
    return ((size_t)unet_wgrad_splits(n, d, h, w, cin, cout) * cout * 27 * cin +
            (size_t)bias_blocks((int64_t)n * d * h * w) * cout) *
           sizeof(float);
}

static hipError_t launch_sum_partials(const float* partial, int nsplit, int64_t nw, const float* bias, int nbias, int nb,
                                      float* dw, float* db, int accumulate, hipStream_t s)
{
    const unsigned blocks = blocks_for(nw, SUM_E) + (db ? blocks_for(nb, SUM_E) : 0);
    k_sum_partials<<<blocks, 256, 0, s>>>(partial, nsplit, nw, bias, nbias, nb, dw, db, accumulate);
    return hipGetLastError();
}

hipError_t launch_unet_conv3_wgrad(const UnetWgrad& a, float* dw, float* db, int accumulate, hipStream_t s)
{
    const int cin = a.c0 + a.c1;
    const int nsplit = unet_wgrad_splits(a.n, a.d, a.h, a.w, cin, a.cout);
    const int64_t nw = (int64_t)a.cout * 27 * cin;
    const int nbias = db ? bias_blocks((int64_t)a.n * a.d * a.h * a.w) : 0;
    float* bias = a.partial + nsplit * nw;
    k_conv3_wgrad<<<(cin / 16) * (a.cout / 16) * nsplit + nbias, WG_T, 0, s>>>(a, nsplit, nbias, bias);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_sum_partials(a.partial, nsplit, nw, bias, nbias, a.cout, dw, db, accumulate, s);
}

hipError_t launch_unet_pack_input(const float* x, int64_t nvox, uint16_t* out, hipStream_t s)
{
    k_pack_input<<<blocks_for(nvox, 256), 256, 0, s>>>(x, nvox, out);
    return hipGetLastError();
}

hipError_t launch_unet_pool2(const uint16_t* in, int ldi, int n, int d, int h, int w, int c, uint16_t* out, int ldo,
                             hipStream_t s)
{
    const int64_t total = (int64_t)n * d * h * w * (c / 8);
    k_pool2<<<blocks_for(total, 256), 256, 0, s>>>(in, ldi, n, d, h, w, c, out, ldo);
    return hipGetLastError();
}

hipError_t launch_unet_skip_grad(const uint16_t* e, int lde, const uint16_t* dp, int ldp, const uint16_t* dcat,
                                 int ldc, int n, int d, int h, int w, int c, uint16_t* out, int ldo, hipStream_t s)
{
    const int64_t total = (int64_t)n * d * h * w * (c / 8);
    k_skip_grad<<<blocks_for(total, 256), 256, 0, s>>>(e, lde, dp, ldp, dcat, ldc, n, d, h, w, c, out, ldo);
    return hipGetLastError();
}

hipError_t launch_unet_up2(const uint16_t* x, int ldx, int cin, const uint16_t* wt, const float* bias, int cout,
                           int n, int d, int h, int w, uint16_t* out, int ldo, hipStream_t s)
{
    const int64_t nvox = (int64_t)n * d * h * w;
    if (cin % 32 == 0 && (cout == 16 || cout == 32 || cout == 64)) {
        // one wave per 16 coarse voxels, four waves per workgroup, all output
        // channels and sub-positions (the input is then read once), or, where
        // that leaves most of the 256 CUs idle, 16 channels and two
        // sub-positions (four crops of 8^3, 128 -> 64 channels: 32 us in 32
        // workgroups, 13 us in 512)
        const unsigned blocks = (unsigned)((nvox + 63) / 64);
        if (cout == 16 || blocks < 256) {
            const dim3 grid(blocks, cout / 16, blocks < 256 ? 4 : 1);
            k_up2_mfma<1><<<grid, 256, 0, s>>>(x, ldx, cin, wt, bias, n, d, h, w, out, ldo);
        } else {   // (64 channels in two halves: 47 us against 66 at once, 32^3 coarse voxels)
            k_up2_mfma<2><<<dim3(blocks, cout / 32), 256, 0, s>>>(x, ldx, cin, wt, bias, n, d, h, w, out, ldo);
        }
        return hipGetLastError();
    }
    const int64_t total = nvox * 8 * (cout / 8);
    k_up2<<<blocks_for(total, 256), 256, 0, s>>>(x, ldx, cin, wt, bias, cout, n, d, h, w, out, ldo);
    return hipGetLastError();
}

hipError_t launch_unet_up2_dgrad(const uint16_t* g, int ldg, int cout, const uint16_t* wt, int cin,
                                 const uint16_t* below, int ldb, int n, int d, int h, int w, uint16_t* out, int ldo,
                                 hipStream_t s)
{
    const int64_t nvox = (int64_t)n * d * h * w;
    if (cout % 16 == 0 && (cin == 32 || cin == 64 || cin == 128)) {
        // all input channels per workgroup, or 16 where the voxels alone leave
        // most of the 256 CUs idle (four crops of 8^3, 128 channels: 44 us in 16
        // workgroups, 21 us in 128)
        const unsigned blocks = (unsigned)((nvox + 4 * 16 * UPD_VG - 1) / (4 * 16 * UPD_VG));
        const int nt = blocks < 256 ? 1 : cin / 16;
        const dim3 grid(blocks, cin / (16 * nt));
        auto run = [&](auto kernel) { kernel<<<grid, 256, 0, s>>>(g, ldg, cout, wt, cin, below, ldb, n, d, h, w, out, ldo); };
        if (nt == 1) run(k_up2_dgrad_mfma<1>);
        else if (nt == 2) run(k_up2_dgrad_mfma<2>);
        else if (nt == 4) run(k_up2_dgrad_mfma<4>);
        else run(k_up2_dgrad_mfma<8>);
        return hipGetLastError();
    }
    const int64_t total = nvox * (cin / 8);
    k_up2_dgrad<<<blocks_for(total, 256), 256, 0, s>>>(g, ldg, cout, wt, cin, below, ldb, n, d, h, w, out, ldo);
    return hipGetLastError();
}

int unet_up2_wgrad_splits(int n, int d, int h, int w, int cin, int cout)
{
    const int64_t chunks = ((int64_t)n * d * h * w + 63) / 64;
    const int blocks = 8 * (cin / 16) * (cout / 16);
    int64_t sp = 2048 / blocks;
    if (sp < 1) sp = 1;
    if (sp > chunks) sp = chunks;
    return (int)sp;
}

size_t unet_up2_wgrad_ws_bytes(int n, int d, int h, int w, int cin, int cout)
{
    return ((size_t)unet_up2_wgrad_splits(n, d, h, w, cin, cout) * cout * 8 * cin +
            (size_t)bias_blocks((int64_t)n * 8 * d * h * w) * cout) *
           sizeof(float);
}

hipError_t launch_unet_up2_wgrad(const uint16_t* x, int ldx, int cin, const uint16_t* g, int ldg, int cout, int n,
                                 int d, int h, int w, float* ws, float* dw, float* db, int accumulate, hipStream_t s)
{
    const int nsplit = unet_up2_wgrad_splits(n, d, h, w, cin, cout);
    const int64_t nw = (int64_t)cout * 8 * cin;
    const int nbias = db ? bias_blocks((int64_t)n * 8 * d * h * w) : 0;
    float* bias = ws + nsplit * nw;
    k_up2_wgrad_mfma<<<8 * (cin / 16) * (cout / 16) * nsplit + nbias, 256, 0, s>>>(x, ldx, cin, g, ldg, cout, n, d, h, w,
                                                                                   ws, nsplit, nbias, bias);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_sum_partials(ws, nsplit, nw, bias, nbias, cout, dw, db, accumulate, s);
}

hipError_t launch_unet_head(const float* xin, const uint16_t* act, int lda, int c, const uint16_t* hw,
                            const float* hb, int64_t nvox, float* out, hipStream_t s)
{
    k_head<<<blocks_for(nvox, 256), 256, 0, s>>>(xin, act, lda, c, hw, hb, nvox, out);
    return hipGetLastError();
}

size_t unet_head_ws_bytes() { return (size_t)512 * (HEAD_C + 2) * sizeof(double); }

hipError_t launch_unet_head_loss_bwd(const float* out, const float* tgt, const uint16_t* act, int lda,
                                     const uint16_t* hw, int64_t nvox, uint16_t* dz, int ldz, double* ws,
                                     double* sums, float* dhead, hipStream_t s)
{
    const int nb = (int)std::min<int64_t>(512, std::max<int64_t>(1, (nvox + 255) / 256));
    k_head_loss_bwd<<<nb, 256, 0, s>>>(out, tgt, act, lda, hw, nvox, 1.0 / (double)nvox, dz, ldz, ws);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    k_sum_partials64<<<HEAD_C + 2, 256, 0, s>>>(ws, nb, HEAD_C + 2, sums, dhead, HEAD_C + 1);
    return hipGetLastError();
}

hipError_t launch_unet_adam(float* w, float* m, float* v, const float* g, int64_t n, float b1, float b2, float lr_t,
                            float inv_sqrt_bc2, float eps, hipStream_t s)
{
    k_adam<<<blocks_for(n, 256), 256, 0, s>>>(w, m, v, g, n, b1, b2, lr_t, inv_sqrt_bc2, eps);
    return hipGetLastError();
}

hipError_t launch_unet_pack_conv3(const float* w, int cout, int cin, uint16_t* wf, uint16_t* wd, hipStream_t s)
{
    k_pack_conv3<<<blocks_for((int64_t)cout * 27 * cin, 256), 256, 0, s>>>(w, cout, cin, wf, wd);
    return hipGetLastError();
}

hipError_t launch_unet_to_bf16(const float* a, int64_t n, uint16_t* out, hipStream_t s)
{
    k_to_bf16<<<blocks_for(n, 256), 256, 0, s>>>(a, n, out);
    return hipGetLastError();
}

}  // namespace ctmi
