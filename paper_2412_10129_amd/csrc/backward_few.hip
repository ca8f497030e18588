// The interpolated adjoint for calls of few views (FEW_VIEWS; the blocks of
// ordered-subset methods), with fixed-point units per round of 512 rays.
//
// Those methods divide A_s^T r by A_s^T 1, and a voxel at the edge of a few
// views' cones is reached by a handful of samples of small weight: there the
// unit of the fixed point shows in the quotient (with a unit per group of
// views, single-view updates of a 256^3 volume moved by up to 6 % of an update
// in such voxels, 5e-5 over the volume).  So the unit stays a round's: its rays'
// summed |y| times the most one ray adds to a cell, at 2^30, whatever the other
// rays of the brick hold, and A_s^T 1 and A_s^T r of a block are rounded alike.
//
// For a group of 8 views, the brick's detector footprints (bounding boxes of
// its projected corners) are enumerated in rounds of 512 pixels: each thread
// re-traces two pixels' rays inside the brick, with the same FP32 arithmetic
// as the forward kernel (shared helpers in ctmi_internal.h), and records them
// in an LDS ray table; the rays' work is cut into items of bounded size (6
// samples), numbered by a block scan, and processed round-robin so rays of
// different lengths keep every lane busy.  32-bit cells hold the round's exact
// integer sum and are flushed after every round, in a fixed order, so the
// result is bit-reproducible.
#include "adjoint_bricks.h"

namespace ctmi {

namespace {

#ifndef CTMI_BWD_INT_SAMPLES
#define CTMI_BWD_INT_SAMPLES 6
#endif
constexpr int BZ = CTMI_BWD_BZ;                   // planes per brick
constexpr int NB = BX * BY * BZ;
constexpr int OWN = NB / 256;                     // voxels owned per thread

// Pixel range whose rays may cross the voxel-centre-coordinate box [lo, hi] (per
// axis x, y, z).  Returns false if empty.
__device__ __forceinline__ bool footprint(const ViewGeo& g, const float lo[3], const float hi[3],
                                          const DetDims& det, int& u0, int& u1, int& v0, int& v1)
{
    float umin = CTMI_INF, umax = -CTMI_INF, vmin = CTMI_INF, vmax = -CTMI_INF;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const float cx = (q & 1) ? hi[0] : lo[0];
        const float cy = (q & 2) ? hi[1] : lo[1];
        const float cz = (q & 4) ? hi[2] : lo[2];
        const float W = __builtin_fmaf(g.MW[0], cx, __builtin_fmaf(g.MW[1], cy, __builtin_fmaf(g.MW[2], cz, g.MW[3])));
        const float U = __builtin_fmaf(g.MU[0], cx, __builtin_fmaf(g.MU[1], cy, __builtin_fmaf(g.MU[2], cz, g.MU[3])));
        const float V = __builtin_fmaf(g.MV[0], cx, __builtin_fmaf(g.MV[1], cy, __builtin_fmaf(g.MV[2], cz, g.MV[3])));
        const float rw = 1.0f / W;
        umin = fminf(umin, U * rw);
        umax = fmaxf(umax, U * rw);
        vmin = fminf(vmin, V * rw);
        vmax = fmaxf(vmax, V * rw);
    }
    foot_pixels(umin, umax, vmin, vmax, det, u0, u1, v0, v1);
    return u0 <= u1 && v0 <= v1;
}

// Views are processed in groups of GV, the ray-setup rounds running over the
// group's combined footprint candidates.  The group's footprints live in LDS.
#ifndef CTMI_BWD_GV
#define CTMI_BWD_GV 8
#endif
constexpr int GV = CTMI_BWD_GV;

struct GroupLds {
    int u0[GV], v0[GV], w[GV], pre[GV + 1];
    float rw[GV];   // 1 / w
};

// Footprints of views [k, k + n) (threads 0..n-1, one view each) and their
// candidate prefix; returns the candidate total (uniform).
__device__ __forceinline__ int make_group(GroupLds& G, const ViewGeo* __restrict__ tab, int view0, int k, int n,
                                          const float lo[3], const float hi[3], const DetDims& det)
{
    if ((int)threadIdx.x < GV) {
        const int g = threadIdx.x;
        int u0 = 0, u1 = -1, v0 = 0, v1 = -1;
        const bool ok = g < n && footprint(tab[view0 + k + g], lo, hi, det, u0, u1, v0, v1);
        G.u0[g] = u0;
        G.v0[g] = v0;
        G.w[g] = ok ? u1 - u0 + 1 : 1;
        G.rw[g] = 1.0f / (float)(ok ? u1 - u0 + 1 : 1);
        G.pre[g + 1] = ok ? (u1 - u0 + 1) * (v1 - v0 + 1) : 0;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        G.pre[0] = 0;
        for (int g = 0; g < GV; ++g) G.pre[g + 1] += G.pre[g];
    }
    __syncthreads();
    return G.pre[GV];
}

// Candidate c of the group -> view g and pixel (iu, iv).  The row p / w is
// estimated in FP32 (p / w <= nv <= 2^20, so the estimate is within 1/4 of
// the quotient and its truncation off by at most one) and corrected with
// the exact remainder (w <= nu <= 4096 and the row fit __umul24).
__device__ __forceinline__ void group_pixel(const GroupLds& G, int c, int& g, int& iu, int& iv)
{
    g = 0;
#pragma unroll
    for (int i = 1; i < GV; ++i) g += c >= G.pre[i] ? 1 : 0;
    const int p = c - G.pre[g];
    const int w = G.w[g];
    int r = (int)((float)p * G.rw[g]);
    int rem = p - (int)__umul24((unsigned)r, (unsigned)w);
    if (rem < 0) {
        --r;
        rem += w;
    } else if (rem >= w) {
        ++r;
        rem -= w;
    }
    iv = G.v0[g] + r;
    iu = G.u0[g] + rem;
}

// Add the round's fixed-point sums into the owned FP32 registers and clear
// those cells (voxel (lx, ly, lz) of the brick sits at
// ((lz + pad) * py + ly + pad) * px + lx + pad).  Each cell is read and
// cleared by the same thread; cells outside the brick that no flush reads
// are never cleared (they only collect discarded contributions).
template <typename Acc>
__device__ __forceinline__ void flush_view(Acc* acc, int px, int py, int pad, int e, float own[OWN])
{
#pragma unroll
    for (int m = 0; m < OWN; ++m) {
        const int i = threadIdx.x + 256 * m;
        const int lx = i % BX, ly = (i / BX) % BY, lz = i / (BX * BY);
        Acc* c = acc + ((lz + pad) * py + (ly + pad)) * px + (lx + pad);
        const Acc a = *c;
        *c = 0;
        own[m] += __builtin_ldexpf((float)(long long)a, -e);
    }
}

__device__ __forceinline__ void acc_add(int* a, float q) { atomicAdd(a, round_int(q)); }

constexpr int HX = BX + 2, HY = BY + 2, HZ = BZ + 2;   // interpolated accumulator: brick plus a one-voxel halo
constexpr int INT_SAMPLES = CTMI_BWD_INT_SAMPLES;  // samples per interpolated item

// Each interpolation sample is processed once, by the brick that holds its
// lower corner (the first brick of an axis also takes corners at -1, whose
// cell lies outside the volume).  Its upper corners may fall one voxel past
// the brick: those cells form the brick's upper shell, 553 cells in three
// faces (x = BX with y, z in [0, BY] x [0, BZ]; y = BY with x < BX; z = BZ
// with x < BX, y < BY), written to the plan's halo buffer and added to the
// neighbouring bricks' voxels by k_halo_add in a fixed order.
constexpr int HALO_SLOTS = Shell<BZ>::N;
constexpr int NH = (HALO_SLOTS + 255) / 256;   // shell cells per thread
// shell cells -> per-thread FP32 registers, clearing them (accumulator
// origin at the brick corner minus one voxel)
template <typename Acc>
__device__ __forceinline__ void flush_shell(Acc* acc, int e, float hown[NH])
{
#pragma unroll
    for (int m = 0; m < NH; ++m) {
        const int h = threadIdx.x + 256 * m;
        if (h < HALO_SLOTS) {
            int lx, ly, lz;
            Shell<BZ>::cell(h, lx, ly, lz);
            Acc* c = acc + ((lz + 1) * HY + (ly + 1)) * HX + (lx + 1);
            const Acc a = *c;
            *c = 0;
            hown[m] += __builtin_ldexpf((float)(long long)a, -e);
        }
    }
}

// Rounds of the interpolated adjoint: RPT rays per thread, RAYS per round.
// Ray-table slot s = tid + 256 h (h < RPT) holds footprint pixel
// p0 + bitrev9(s), so slots next to each other (whose items run on
// neighbouring lanes) hold pixels far apart on the detector.  Item -> slot
// lookups go through a 16-bit map for the first IMAPCAP items of a round.
constexpr int RPT = 2, RAYS = 256 * RPT;
#ifndef CTMI_BWD_IMAPCAP
#define CTMI_BWD_IMAPCAP 4096
#endif
constexpr int IMAPCAP = CTMI_BWD_IMAPCAP;
static_assert(RAYS == 512, "slot permutation is a 9-bit reversal");

// Ray-table slots hold footprint pixels in bit-reversed order: slots that sit
// next to each other (whose items run on neighbouring lanes) then hold pixels
// far apart on the detector.  The rays of adjacent pixels cross the same cells
// at the same steps, and LDS atomics of one instruction from several lanes to
// one address serialise (about 3x the cost of distinct addresses when 4 lanes
// share one).
__device__ __forceinline__ int slot_pixel(int s)
{
    return (int)(__builtin_bitreverse32((unsigned)s) >> 23);
}

// Largest slot r in [0, RAYS) with pre[r] <= it (pre non-decreasing).
__device__ __forceinline__ int owner_slot(const int* pre, int it)
{
    int lo = 0, hi = RAYS - 1;
#pragma unroll
    for (int st = 0; st < 9; ++st) {
        const int mid = (lo + hi + 1) >> 1;
        if (pre[mid] <= it) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Inclusive scan of one int over a wave.
__device__ __forceinline__ int wave_scan(int x)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    return x;
}

#ifndef CTMI_BWD_WAVES
#define CTMI_BWD_WAVES 4
#endif
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(CTMI_BWD_WAVES, 8))) k_backward_interp_few(const float* __restrict__ proj, float* __restrict__ vol,
                                                         const ViewGeo* __restrict__ tab,
                                                         const ViewGeo64* __restrict__ tab64, int view0, int nviews,
                                                         VolDims v, DetDims det, BrickMap m, float beta, float ds,
                                                         float cmax, float* __restrict__ shell)
{
    // accumulator over voxels [b0 - 1, b1] per axis, so every sample scatters
    // to 8 fixed offsets without per-corner tests; the lower face only
    // receives corners outside the volume (first brick of an axis), the
    // upper shell goes to the neighbours
    __shared__ int acc[HX * HY * HZ];
    // ray table: (base, y) and (st, first sample | sample count << 16)
    __shared__ float4 t_a[RAYS], t_b[RAYS];
    __shared__ int t_pre[RAYS];
    __shared__ unsigned short imap[IMAPCAP];
    __shared__ int wsum[RPT][4];
    __shared__ float wsumf[4];
    __shared__ GroupLds G;
    for (int i = threadIdx.x; i < HX * HY * HZ; i += blockDim.x) acc[i] = 0;
    float own[OWN], hown[NH];
#pragma unroll
    for (int i = 0; i < OWN; ++i) own[i] = 0.0f;
#pragma unroll
    for (int i = 0; i < NH; ++i) hown[i] = 0.0f;
    int bx, by, bz;
    brick_origin(m, (int)blockIdx.x, bx, by, bz);
    const int x0 = bx * BX, y0 = by * BY, z0 = bz * BZ;
    const int x1 = min(x0 + BX, v.nx), y1 = min(y0 + BY, v.ny), z1 = min(z0 + BZ, v.nz);
    // the brick takes samples whose lower corner lies in [x0, x1) (from -1
    // for the first brick of an axis); their positions lie in [lo, hi)
    // (voxel-centre coordinates)
    const float lo[3] = {x0 > 0 ? (float)x0 : -1.0f, y0 > 0 ? (float)y0 : -1.0f, z0 > 0 ? (float)z0 : -1.0f};
    const float hi[3] = {(float)x1, (float)y1, (float)z1};
    // a sample's lower corner (floor of its position) must lie in
    // [lo, hi - 1] per axis; the accumulator's byte offset of corner c is
    // 4 ((c_z - z0 + 1) HX HY + (c_y - y0 + 1) HX + (c_x - x0 + 1)), formed
    // in FP32 (integers below 2^24)
    const float cmx = hi[0] - 1.0f, cmy = hi[1] - 1.0f, cmz = hi[2] - 1.0f;
    constexpr float AB = (float)sizeof(int);   // accumulator bytes per cell
    const float aoff =
        -AB * ((float)(z0 - 1) * (float)(HX * HY) + (float)(y0 - 1) * (float)HX + (float)(x0 - 1));
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    char* const accb = reinterpret_cast<char*>(acc);
    const float inv_ds = 1.0f / ds;

    for (int k = 0; k < nviews; k += GV) {
        const int ng = min(GV, nviews - k);
        __syncthreads();
        const int npx = make_group(G, tab, view0, k, ng, lo, hi, det);
        for (int p0 = 0; p0 < npx; p0 += RAYS) {
            // --- ray setup: RPT rays per thread
            int cnt[RPT];
            float ya = 0.0f;   // sum of |y| over this thread's rays
            float yr[RPT];
#pragma unroll
            for (int h = 0; h < RPT; ++h) {
                const int sl = tid + 256 * h;
                const int p = p0 + slot_pixel(sl);
                cnt[h] = 0;
                yr[h] = 0.0f;
                if (p < npx) {
                    int gv, iu, iv;
                    group_pixel(G, p, gv, iu, iv);
                    InterpRay ray;
                    if (interp_ray(tab64[view0 + k + gv], iu, iv, v, ds, inv_ds, ray)) {
                        // samples (relative to the anchor kc) inside the brick's
                        // box, widened by 1e-3 of a sample against the
                        // reciprocal's rounding, and by the samples within
                        // 2^-22 |face| of a face (|face| <= wface): a position
                        // that close may round onto either side of it, and for
                        // a ray nearly parallel to the face that span holds
                        // many samples (the smallest nonzero step bounds it on
                        // every axis).  A sample outside the box adds nothing
                        // (its weights are zeroed below), so widening only
                        // costs work, while a sample missed here would be lost.
                        float kmin = -CTMI_INF, kmax = CTMI_INF, imax = 0.0f;
                        bool inside = true;
#pragma unroll
                        for (int a = 0; a < 3; ++a) {
                            if (ray.st[a] != 0.0f) {
                                const float ia = ray.inv[a];
                                const float ka = (lo[a] - ray.base[a]) * ia, kb = (hi[a] - ray.base[a]) * ia;
                                kmin = fmaxf(kmin, fminf(ka, kb));
                                kmax = fminf(kmax, fmaxf(ka, kb));
                                imax = fmaxf(imax, fabsf(ia));
                            } else {
                                // constant coordinate: the loop's own test
                                const float f = __builtin_floorf(ray.base[a]);
                                inside &= f >= lo[a] && f <= hi[a] - 1.0f;
                            }
                        }
                        // (capped at 2^16 samples, more than a ray holds, so
                        // that the sample indices below stay in int range)
                        const float wface = 0x1p-22f * fmaxf(hi[0], fmaxf(hi[1], hi[2]));
                        const float wk = fminf(__builtin_fmaf(wface, imax, 1e-3f), 65536.0f);
                        if (inside && kmin < kmax + 2.0f * wk) {
                            const int ks = max(ray.k0, ray.kc + (int)__builtin_ceilf(kmin - wk));
                            const int ke = min(ray.k1, ray.kc + (int)__builtin_floorf(kmax + wk));
                            const int n = ke - ks + 1;
                            if (n > 0 && n < 65536) {
                                cnt[h] = (n + INT_SAMPLES - 1) / INT_SAMPLES;
                                // first sample relative to the anchor: |ks - kc| < 2^15
                                // because a ray has fewer than 2^15 samples in the
                                // volume (checked at plan creation)
                                const int jn = ((ks - ray.kc) & 0xFFFF) | (n << 16);
                                const float* pk = proj + (int64_t)(k + gv) * det.nv * det.nu;
                                yr[h] = pk[(int64_t)iv * det.nu + iu];
                                ya += fabsf(yr[h]);
                                t_a[sl] = make_float4(ray.base[0], ray.base[1], ray.base[2], 0.0f);
                                t_b[sl] = make_float4(ray.st[0], ray.st[1], ray.st[2], __int_as_float(jn));
                            }
                        }
                    }
                }
            }
            // --- one block pass: item offsets (exclusive scan over slots in
            // slot order) and the round's sum of |y| (fixed order)
            int inc[RPT];
#pragma unroll
            for (int h = 0; h < RPT; ++h) inc[h] = wave_scan(cnt[h]);
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) ya += __shfl_xor(ya, o, 64);
            if (lane == 63) {
#pragma unroll
                for (int h = 0; h < RPT; ++h) wsum[h][wid] = inc[h];
            }
            if (lane == 0) wsumf[wid] = ya;
            __syncthreads();
            float ysum = (wsumf[0] + wsumf[1]) + (wsumf[2] + wsumf[3]);
            if (!(ysum <= 0x1.fffffep127f)) {
                // a NaN or an infinity among the round's values (those rays
                // add nothing here; k_nonfinite marks their voxels), or a
                // finite sum past FLT_MAX: sum again over the finite values
                // (block-uniform branch)
                float yb = 0.0f;
#pragma unroll
                for (int h = 0; h < RPT; ++h) {
                    yr[h] = finite_or_zero(yr[h]);
                    yb += fabsf(yr[h]);
                }
#pragma unroll
                for (int o = 32; o > 0; o >>= 1) yb += __shfl_xor(yb, o, 64);
                __syncthreads();
                if (lane == 0) wsumf[wid] = yb;
                __syncthreads();
                ysum = (wsumf[0] + wsumf[1]) + (wsumf[2] + wsumf[3]);
            }
            if (!(ysum > 0.0f)) {
                // nothing to add: keep the LDS sums of this pass alive until
                // every thread has read them
                __syncthreads();
                continue;
            }
            int base = 0, off[RPT];
#pragma unroll
            for (int h = 0; h < RPT; ++h) {
                int before = 0, tot = 0;
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    const int t = wsum[h][w];
                    before += w < wid ? t : 0;
                    tot += t;
                }
                off[h] = base + before + inc[h] - cnt[h];
                base += tot;
            }
            const int total = base;
            // one cell's round sum is at most cmax sum_r |y_r| (cmax: K
            // samples of ds, K the most samples of one ray inside a
            // 2x2x2-voxel support)
            // (a sum of finite values can only overflow when some |y| is
            // near FLT_MAX; 512 values of at most 2^128 bound it by 2^137)
            const int ex = ysum <= 0x1.fffffep127f ? fixed_exp(cmax, ysum) : fixed_exp(cmax, 0x1p127f) - 10;
#pragma unroll
            for (int h = 0; h < RPT; ++h) {
                const int sl = tid + 256 * h;
                t_pre[sl] = off[h];
                if (cnt[h] > 0) {
                    // scaled before ds: |y 2^e| <= 2^30 / cmax and cmax >= ds
                    t_a[sl].w = __builtin_ldexpf(yr[h], ex) * ds;
                    const int e = min(off[h] + cnt[h], IMAPCAP);
                    for (int i = off[h]; i < e; ++i) imap[i] = (unsigned short)sl;
                }
            }
            __syncthreads();
            // --- items, taken round-robin: every lane runs at most
            // INT_SAMPLES samples per item, so the wave stays converged
            for (int it = tid; it < total; it += 256) {
                const int r = it < IMAPCAP ? (int)imap[it] : owner_slot(t_pre, it);
                const int q = it - t_pre[r];
                const float4 ta = t_a[r], tb = t_b[r];
                const int jn = __float_as_int(tb.w);
                const int j0 = (int)(int16_t)(uint16_t)(jn & 0xFFFF) + q * INT_SAMPLES;  // first sample
                const int cntq = min(INT_SAMPLES, (int)((unsigned)jn >> 16) - q * INT_SAMPLES);
                const float bxr = ta.x, byr = ta.y, bzr = ta.z, yv = ta.w;
                const float sxr = tb.x, syr = tb.y, szr = tb.z;
                // the ray's values must be in registers before the sample
                // loop, so that the loop never waits on its own atomics
                asm volatile("" ::"v"(bxr), "v"(byr), "v"(bzr), "v"(sxr), "v"(syr), "v"(szr), "v"(yv), "v"(j0),
                             "v"(cntq));
                // j runs over the item's samples as an exact FP32 integer
                const float jend = (float)(j0 + cntq);
                for (float j = (float)j0; j < jend; j += 1.0f) {
                    // same FP32 position as the forward kernel's sample k
                    const float px = __builtin_fmaf(j, sxr, bxr);
                    const float py = __builtin_fmaf(j, syr, byr);
                    const float pz = __builtin_fmaf(j, szr, bzr);
                    const float fx = __builtin_floorf(px), fy = __builtin_floorf(py), fz = __builtin_floorf(pz);
                    // corner clamped into the accumulator; a sample whose
                    // corner moved lies outside the box and adds 0
                    const float cx = __builtin_amdgcn_fmed3f(fx, lo[0], cmx);
                    const float cy = __builtin_amdgcn_fmed3f(fy, lo[1], cmy);
                    const float cz = __builtin_amdgcn_fmed3f(fz, lo[2], cmz);
                    const bool ok = cx == fx && cy == fy && cz == fz;
                    const int boff = (int)__builtin_fmaf(cz, AB * (float)(HX * HY),
                                                         __builtin_fmaf(cy, AB * (float)HX,
                                                                        __builtin_fmaf(cx, AB, aoff)));
                    const float ax_ = px - fx, ay_ = py - fy, az_ = pz - fz;
                    // trilinear weights times y, each pair split as (w - a w, a w)
                    const float yo = ok ? yv : 0.0f;
                    const float yz1 = az_ * yo, yz0 = yo - yz1;
                    const float w10 = ay_ * yz0, w00 = yz0 - w10;
                    const float w11 = ay_ * yz1, w01 = yz1 - w11;
                    const float u00 = ax_ * w00, u10 = ax_ * w10, u01 = ax_ * w01, u11 = ax_ * w11;
                    int* a0 = reinterpret_cast<int*>(accb + boff);
                    acc_add(a0, w00 - u00);
                    acc_add(a0 + 1, u00);
                    acc_add(a0 + HX, w10 - u10);
                    acc_add(a0 + HX + 1, u10);
                    acc_add(a0 + HX * HY, w01 - u01);
                    acc_add(a0 + HX * HY + 1, u01);
                    acc_add(a0 + HX * HY + HX, w11 - u11);
                    acc_add(a0 + HX * HY + HX + 1, u11);
                }
            }
            __syncthreads();
            // --- flush: 32-bit cells hold one round's sums (bounded by the
            // scale).  No barrier is needed after it: the next round's
            // atomics come after two more barriers, and nothing before them
            // touches the accumulator.
            flush_shell(acc, ex, hown);
            flush_view(acc, HX, HY, 1, ex, own);
        }
    }
    store_owned<BZ, 256>(vol, own, v, x0, y0, z0, beta);
    float* out = shell + (size_t)blockIdx.x * HALO_SLOTS;
#pragma unroll
    for (int m2 = 0; m2 < NH; ++m2) {
        const int h = threadIdx.x + 256 * m2;
        if (h < HALO_SLOTS) out[h] = hown[m2];
    }
}

}  // namespace

hipError_t launch_backward_interp_few_bricks(const Plan& p, const float* proj, float* vol, int64_t view0,
                                             int64_t nviews, float beta, float* shell, hipStream_t s)
{
    const BrickMap m = brick_map(p, BZ);
    const unsigned blocks = (unsigned)m.nbx * m.nby * m.nbz;
    hipLaunchKernelGGL(k_backward_interp_few, dim3(blocks), dim3(256), 0, s, proj, vol, p.d_views, p.d_views64,
                       (int)view0, (int)nviews, p.vol, p.det, m, beta, p.ds, p.round_interp, shell);
    return hipGetLastError();
}

}  // namespace ctmi
