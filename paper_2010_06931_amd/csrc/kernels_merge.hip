// Output kernels (Sec. 2.1 "merging", Sec. 2.5): sampling density, merge
// weights and the weighted average of the two resampled scans.
//
//   k_density       every output A-scan splats its (clamped) sample position
//                   bilinearly into a per-scan h x w grid; fixed-point 64-bit
//                   integer atomics keep the sums independent of order
//   k_merge_weights density read back at the sample position -> weight
//                   exp(-kappa max(0, rho - 1)), clipped below tau, normalised;
//                   the OCTA weights are further multiplied by the resampled
//                   validity (Eq. 5); where both vanish, OCT keeps the scan with
//                   the lower density and OCTA is 0
//   k_merge_quads   resample both scans with their fields (Eq. 2 interpolator,
//                   value only) and write the weighted sum (float32 volumes);
//   k_merge_volume  the same of 16-bit and of shallow float32 volumes;
//   k_merge_tile    the same of 16-bit volumes of many A-scans, on the matrix cores
#include <hip/hip_runtime.h>

#include "octmc_internal.h"
#include "tile_blend.h"

namespace octmc {
namespace {

constexpr double kFix = 4294967296.0;  // 2^32

__device__ __forceinline__ void bilin(float x, float y, int w, int h, int& x0, int& y0, int& x1, int& y1, float& fx,
                                      float& fy)
{
    x = fminf(fmaxf(x, 0.f), (float)(w - 1));
    y = fminf(fmaxf(y, 0.f), (float)(h - 1));
    x0 = (int)floorf(x);
    y0 = (int)floorf(y);
    x1 = min(x0 + 1, w - 1);
    y1 = min(y0 + 1, h - 1);
    fx = x - x0;
    fy = y - y0;
}

__global__ void k_density(const float* __restrict__ disp, int w, int h, unsigned long long* __restrict__ grid,
                          int nvol)
{
    const int na = w * h;
    for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < nvol * na; q += gridDim.x * blockDim.x) {
        const int V = q / na, a = q % na;
        const int i = a % w, j = a / w;
        int x0, y0, x1, y1;
        float fx, fy;
        bilin(i + disp[(size_t)q * 3], j + disp[(size_t)q * 3 + 1], w, h, x0, y0, x1, y1, fx, fy);
        unsigned long long* G = grid + (size_t)V * na;
        atomicAdd(G + (size_t)y0 * w + x0, (unsigned long long)llrint((1.0 - fx) * (1.0 - fy) * kFix));
        atomicAdd(G + (size_t)y0 * w + x1, (unsigned long long)llrint((double)fx * (1.0 - fy) * kFix));
        atomicAdd(G + (size_t)y1 * w + x0, (unsigned long long)llrint((1.0 - fx) * (double)fy * kFix));
        atomicAdd(G + (size_t)y1 * w + x1, (unsigned long long)llrint((double)fx * (double)fy * kFix));
    }
}

__device__ __forceinline__ void cr_w(float t, float w[4])
{
    const float t2 = t * t, t3 = t2 * t;
    w[0] = 0.5f * (-t3 + 2.f * t2 - t);
    w[1] = 0.5f * (3.f * t3 - 5.f * t2 + 2.f);
    w[2] = 0.5f * (-3.f * t3 + 4.f * t2 + t);
    w[3] = 0.5f * (t3 - t2);
}

__device__ __forceinline__ float valid_at(const float* v, int n, int idx, float dv)
{
    const float f = floorf(dv);
    const int nx = idx + (int)f;
    float w[4];
    cr_w(dv - f, w);
    float s = 0.f;
    for (int a = 0; a < 4; ++a) s = fmaf(w[a], v[clampi(nx - 1 + a, 0, n - 1)], s);
    return fminf(fmaxf(s, 0.f), 1.f);
}

__global__ void k_merge_weights(const float* __restrict__ disp, int w, int h,
                                const unsigned long long* __restrict__ grid, const float* __restrict__ vx,
                                const float* __restrict__ vy, double kappa, double tau, float4* __restrict__ wts)
{
    const int na = w * h;
    for (int a = blockIdx.x * blockDim.x + threadIdx.x; a < na; a += gridDim.x * blockDim.x) {
        const int i = a % w, j = a / w;
        double rho[2];
        for (int V = 0; V < 2; ++V) {
            const float* dv = disp + ((size_t)V * na + a) * 3;
            int x0, y0, x1, y1;
            float fx, fy;
            bilin(i + dv[0], j + dv[1], w, h, x0, y0, x1, y1, fx, fy);
            const unsigned long long* G = grid + (size_t)V * na;
            rho[V] = ((1.0 - fx) * (1.0 - fy) * (double)G[(size_t)y0 * w + x0] +
                      (double)fx * (1.0 - fy) * (double)G[(size_t)y0 * w + x1] +
                      (1.0 - fx) * (double)fy * (double)G[(size_t)y1 * w + x0] +
                      (double)fx * (double)fy * (double)G[(size_t)y1 * w + x1]) / kFix;
        }
        double wx = exp(-kappa * fmax(0.0, rho[0] - 1.0)), wy = exp(-kappa * fmax(0.0, rho[1] - 1.0));
        if (wx < tau) wx = 0.0;
        if (wy < tau) wy = 0.0;
        double ax, ay;
        if (wx + wy > 0) {
            ax = wx / (wx + wy);
            ay = wy / (wx + wy);
        } else if (rho[0] <= rho[1]) {
            ax = 1.0;
            ay = 0.0;
        } else {
            ax = 0.0;
            ay = 1.0;
        }
        double ox = 0.0, oy = 0.0;
        if (vx && vy) {
            ox = wx * valid_at(vx, h, j, disp[(size_t)a * 3 + 1]);
            oy = wy * valid_at(vy, w, i, disp[((size_t)na + a) * 3]);
            const double s = ox + oy;
            if (s > 0) {
                ox /= s;
                oy /= s;
            }
        }
        wts[a] = make_float4((float)ax, (float)ay, (float)ox, (float)oy);
    }
}

template <typename T>
__device__ __forceinline__ float ld(const void* p, size_t q);
template <>
__device__ __forceinline__ float ld<float>(const void* p, size_t q) { return static_cast<const float*>(p)[q]; }
template <>
__device__ __forceinline__ float ld<bf16_t>(const void* p, size_t q)
{
    return __builtin_bit_cast(float, (uint32_t) static_cast<const unsigned short*>(p)[q] << 16);
}
template <>
__device__ __forceinline__ float ld<f16_t>(const void* p, size_t q)
{
    return (float)__builtin_bit_cast(_Float16, static_cast<const unsigned short*>(p)[q]);
}

// 32-bit buffer loads of one sample (wave-uniform column offset in soff)
template <typename T>
__device__ __forceinline__ float ldb(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff);
template <>
__device__ __forceinline__ float ldb<float>(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
}
template <>
__device__ __forceinline__ float ldb<bf16_t>(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff)
{
    return __builtin_bit_cast(float, (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(r, voff, soff, 0) << 16);
}
template <>
__device__ __forceinline__ float ldb<f16_t>(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff)
{
    return (float)__builtin_bit_cast(_Float16, __builtin_amdgcn_raw_buffer_load_b16(r, voff, soff, 0));
}

// value of the next lane (DPP whole-wave shift; lane 63 reads 0 by bound control)
__device__ __forceinline__ float next_lane(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x130, 0xF, 0xF, true));
}

// Depth steps of 61 output samples on 64 lanes: lane l holds source sample
// base + 61 n + l (clamped to the A-scan), and output lane l < 61 reads the
// blended values of lanes l .. l + 3.
constexpr int kMergeStep = 61;

// One output A-scan (a at i, j) by one wave, lanes along depth, from volumes of dp
// samples a column (the first d are the A-scan); wgt: the weights of the two scans.
// The 16 lateral columns of each scan are read with 32-bit buffer offsets (their
// offsets and weights wave-uniform), each source sample once per step.
template <typename T>
__device__ __forceinline__ void merge_ascan(const __amdgpu_buffer_rsrc_t (&rs)[2], const float* __restrict__ disp, int a,
                                            int i, int j, const float (&wgt)[2], int w, int h, int d, int dp, int lane,
                                            float* __restrict__ out)
{
    const int na = w * h;
    uint32_t off[2][16];
    float wl[2][16], wz[2][4];
    int base[2];
#pragma unroll
    for (int V = 0; V < 2; ++V) {
        const float* dv = disp + ((size_t)V * na + a) * 3;
        const float fxf = floorf(dv[0]), fyf = floorf(dv[1]), fzf = floorf(dv[2]);
        const int nx = i + (int)fxf, ny = j + (int)fyf, nz = (int)fzf;
        float wx[4], wy[4];
        cr_w(dv[0] - fxf, wx);
        cr_w(dv[1] - fyf, wy);
        cr_w(dv[2] - fzf, wz[V]);
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                off[V][b * 4 + c] = (uint32_t)__builtin_amdgcn_readfirstlane(
                    (int)((uint32_t)(clampi(ny - 1 + b, 0, h - 1) * w + clampi(nx - 1 + c, 0, w - 1)) * (uint32_t)dp *
                          esize<T>::v));
                wl[V][b * 4 + c] = wx[c] * wy[b];
            }
        base[V] = min(max(nz, -kMxLimit), kMxLimit) - 1;
    }
    const int nsteps = (d + kMergeStep - 1) / kMergeStep;
    for (int n = 0; n < nsteps; ++n) {
        float res = 0.f;
#pragma unroll
        for (int V = 0; V < 2; ++V) {
            const uint32_t voff = (uint32_t)clampi(base[V] + kMergeStep * n + lane, 0, d - 1) * esize<T>::v;
            float c = 0.f;
#pragma unroll
            for (int q = 0; q < 16; ++q) c = fmaf(wl[V][q], ldb<T>(rs[V], voff, off[V][q]), c);
            const float c1 = next_lane(c), c2 = next_lane(c1), c3 = next_lane(c2);
            float iv = 0.f;
            iv = fmaf(wz[V][0], c, iv);
            iv = fmaf(wz[V][1], c1, iv);
            iv = fmaf(wz[V][2], c2, iv);
            iv = fmaf(wz[V][3], c3, iv);
            res = fmaf(wgt[V], iv, res);
        }
        const int k = kMergeStep * n + lane;
        if (lane < kMergeStep && k < d) out[(size_t)a * d + k] = res;
    }
}

// one wavefront per output A-scan; which = 0 uses the OCT weights (wts.x, wts.y),
// which = 1 the OCTA weights (wts.z, wts.w)
template <typename T>
__global__ __launch_bounds__(256) void k_merge_volume(const void* __restrict__ sx, const void* __restrict__ sy,
                                                      const float* __restrict__ disp, const float4* __restrict__ wts,
                                                      int which, int w, int h, int d, int dp, uint32_t vol_bytes,
                                                      float* __restrict__ out)
{
    const int a = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
    if (a >= w * h) return;
    const float4 wt = wts[a];
    const float wgt[2] = {which ? wt.z : wt.x, which ? wt.w : wt.y};
    const __amdgpu_buffer_rsrc_t rs[2] = {
        __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(sx), (short)0, (int)vol_bytes, kRsrcWord3),
        __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(sy), (short)0, (int)vol_bytes, kRsrcWord3)};
    merge_ascan<T>(rs, disp, a, a % w, a / w, wgt, w, h, d, dp, threadIdx.x & 63, out);
}

// k_merge_volume on the matrix cores: one wave per 2 x 2 tile of A-scans
// (tile_blend.h), L depths per lane.  k_merge_volume loads every column of a
// tile up to four times, one sample per lane and load, and keeps the texture
// path busy with that; here a tile's columns are loaded once, 16 bytes per lane.
// 500 x 500 x 465: 1.50 -> 0.46 ms from BF16 volumes.
// Outputs that are not finite are formed again by merge_ascan, each A-scan for
// itself: a sample that is not finite reaches the whole tile through the weights
// 0, and the three parts of a weight make a NaN of an infinity.
template <typename T, int L>
__global__ __launch_bounds__(256, 3) void k_merge_tile(const void* __restrict__ sx, const void* __restrict__ sy,
                                                       const float* __restrict__ disp, const float4* __restrict__ wts,
                                                       int which, int w, int h, int d, int dp, uint32_t vol_bytes,
                                                       float* __restrict__ out)
{
    constexpr int es = (int)esize<T>::v;
    typedef MxGeo<es, L> Geo;
    __shared__ MxLds<es, 2, L> lds[4];
    const int wv = uni((int)(threadIdx.x >> 6));
    MxLds<es, 2, L>& M = lds[wv];
    int i0, j0;
    if (!mx_tile(w, h, xcd_block(blockIdx.x, gridDim.x), wv, i0, j0)) return;
    const __amdgpu_buffer_rsrc_t rx =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(sx), (short)0, (int)vol_bytes, kRsrcWord3);
    const __amdgpu_buffer_rsrc_t ry =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(sy), (short)0, (int)vol_bytes, kRsrcWord3);
    const size_t na = (size_t)w * h;
    int groups = 15;  // the tile's A-scans of a round: all, or two where they need too many slots
    for (;;) {
        int lane = threadIdx.x & 63;
        asm volatile("" : "+v"(lane));
        const int g = lane >> 4, p0 = L * (lane & 15);
        const int2 pg = make_int2(min(i0 + (g & 1), w - 1), min(j0 + (g >> 1), h - 1));
        const int ag = pg.y * w + pg.x;
        const bool write = i0 + (g & 1) < w && j0 + (g >> 1) < h && (groups >> g & 1);
        MxScan SX, SY;
        int nrest = 0;
        if (!mx_setup<T, 1>(SX, M, 0, disp, ag, pg, 0, w, h, dp, lane, groups, nrest) ||
            !mx_setup<T, 1>(SY, M, 1, disp + na * 3, ag, pg, SX.sh, w, h, dp, lane, groups, nrest)) {
            groups = 3;
            continue;
        }
        const float4 wt = wts[ag];
        const float wx = which ? wt.z : wt.x, wy = which ? wt.w : wt.y;
        float* const o = out + (size_t)ag * d;
        float bad = 0.f;  // not a number once an output was not finite
        const int nsteps = (d + SX.any + Geo::kOut - 1) / Geo::kOut;
        for (int s = 0; s < nsteps; ++s) {
            typename MxDwords<Geo::kDw>::type qx[8], qy[8];
            mx_load(qx, SX, M, 0, rx, s, dp, lane);
            mx_load(qy, SY, M, 1, ry, s, dp, lane);
            float x[L + 3], y[L + 3], v[1][L];
            f32x4 D[L] = {};
            mx_blend<T>(D, qx, M, 0, lane);
            if (SX.ns > 32) mx_rest<T>(D, SX, M, 0, rx, s, dp, lane);
            mx_rows<false>(v, D, SX, M, s, dp, lane);
#pragma unroll
            for (int i = 0; i < L; ++i) x[i] = v[0][i];
            f32x4 E[L] = {};
            mx_blend<T>(E, qy, M, 1, lane);
            if (SY.ns > 32) mx_rest<T>(E, SY, M, 1, ry, s, dp, lane);
            mx_rows<true>(v, E, SY, M, s, dp, lane);
#pragma unroll
            for (int i = 0; i < L; ++i) y[i] = v[0][i];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                x[L + i] = row_next(x[i]);
                y[L + i] = row_next(y[i]);
            }
            float r[L];
#pragma unroll
            for (int i = 0; i < L; ++i) {
                r[i] = fmaf(wy, mx_fir(SY.wz, y, i), wx * mx_fir(SX.wz, x, i));
                bad = fmaf(r[i], 0.f, bad);
            }
            const int k0 = Geo::kOut * s + p0 - SX.sh;  // output of position 0
            if (write) {
                if (p0 + L <= Geo::kOut && k0 >= 0 && k0 + L <= d) {
                    typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
#pragma unroll
                    for (int i = 0; i < L; i += 4)
                        *reinterpret_cast<f32x4u*>(o + k0 + i) = f32x4u{r[i], r[i + 1], r[i + 2], r[i + 3]};
                } else {
#pragma unroll
                    for (int i = 0; i < L; ++i)
                        if (p0 + i < Geo::kOut && (unsigned)(k0 + i) < (unsigned)d) o[k0 + i] = r[i];
                }
            }
        }
        if (__ballot(bad != 0.f)) {
            __threadfence();  // the stores above come first
            const __amdgpu_buffer_rsrc_t rs[2] = {rx, ry};
            for (int q = 0; q < 4; ++q) {
                const int i = i0 + (q & 1), j = j0 + (q >> 1), a = uni(j * w + i);
                if (!(groups >> q & 1) || i >= w || j >= h) continue;  // wave-uniform
                const float4 wq = wts[a];
                const float wgt[2] = {which ? wq.z : wq.x, which ? wq.w : wq.y};
                merge_ascan<T>(rs, disp, a, i, j, wgt, w, h, d, dp, lane, out);
            }
        }
        groups = mx_next(groups, false);
        if (!groups) return;
    }
}

// float32 volumes, four samples a lane: k_merge_volume is bound by its loads, one of
// 8.6 cycles of the CU's vector memory path per column and 61 outputs; a 16-byte one
// takes 16.7 and serves 252.  A wave takes an A-scan and a workgroup four in a row,
// step by step together, so that the columns they share are still in the L1 when
// the others read them; that takes all 16 loads of a scan in flight and no more than
// four waves a SIMD, which the registers see to (500 x 500 x 465, 2 x 2 A-scans a
// workgroup: 0.77 ms so, 0.93 with six, 1.15 with five, whose workgroups drift apart;
// four in a row 0.74, 4 x 2 0.75, 4 x 4 0.84).  Lane l holds samples
// base + 252 n + 4 l .. + 3; those outside the A-scan take the edge's value after the
// blend (the loads stay inside).  Arithmetic and order are k_merge_volume's.  200 x
// 200 x 300, both volumes: 367 us by k_merge_volume, 262 in a tile's distinct columns
// on the matrix cores (where float32 runs at the vector rate), 231 so; 64 x 64 x 128
// 51, -, 42.
constexpr int kQuadStep = 252;

__global__ __launch_bounds__(256, 4) void k_merge_quads(const float* __restrict__ sx, const float* __restrict__ sy,
                                                     const float* __restrict__ disp, const float4* __restrict__ wts,
                                                     int which, int w, int h, int d, uint32_t vol_bytes,
                                                     float* __restrict__ out)
{
    typedef float quad_t __attribute__((ext_vector_type(4), aligned(4)));
    const int wv = uni((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    // 8 bands of rows (one per XCD), swept column by column
    const int rpb = (h + 7) >> 3, per = rpb * ((w + 3) >> 2);
    const int t = xcd_block(blockIdx.x, gridDim.x), band = t / per, tb = t - band * per;
    const int i = 4 * (tb / rpb) + wv, j = band * rpb + tb % rpb;
    if (j >= h) return;           // whole block
    const bool active = i < w;  // wave-uniform
    const int na = w * h, a = uni(active ? j * w + i : 0);
    const float4 wt = wts[a];
    const float wgt[2] = {which ? wt.z : wt.x, which ? wt.w : wt.y};
    const float* vol[2] = {sx, sy};
    __amdgpu_buffer_rsrc_t rs[2];
    uint32_t off[2][16];
    float wl[2][16], wz[2][4];
    int base[2];
#pragma unroll
    for (int V = 0; V < 2; ++V) {
        rs[V] = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(vol[V]), (short)0, (int)vol_bytes, kRsrcWord3);
        const float* dv = disp + ((size_t)V * na + a) * 3;
        const float fxf = floorf(dv[0]), fyf = floorf(dv[1]), fzf = floorf(dv[2]);
        const int nx = i + (int)fxf, ny = j + (int)fyf, nz = (int)fzf;
        float wx[4], wy[4];
        cr_w(dv[0] - fxf, wx);
        cr_w(dv[1] - fyf, wy);
        cr_w(dv[2] - fzf, wz[V]);
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                off[V][b * 4 + c] = (uint32_t)uni((int)((uint32_t)(clampi(ny - 1 + b, 0, h - 1) * w +
                                                                   clampi(nx - 1 + c, 0, w - 1)) * (uint32_t)d * 4u));
                wl[V][b * 4 + c] = wx[c] * wy[b];
            }
        base[V] = uni(min(max(nz, -kMxLimit), kMxLimit) - 1);
    }
    const int nsteps = (d + kQuadStep - 1) / kQuadStep;
    for (int n = 0; n < nsteps; ++n) {
        float res[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int V = 0; V < 2; ++V) {
            const int m = base[V] + kQuadStep * n + 4 * lane, at = clampi(m, 0, d - 4);
            quad_t x[16];
#pragma unroll
            for (int q = 0; q < 16; ++q)
                x[q] = __builtin_bit_cast(quad_t, __builtin_amdgcn_raw_buffer_load_b128(rs[V], 4u * (uint32_t)at, off[V][q], 0));
            float c[7] = {};
#pragma unroll
            for (int q = 0; q < 16; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e) c[e] = fmaf(wl[V][q], x[q][e], c[e]);
            if (base[V] + kQuadStep * n < 0 || base[V] + kQuadStep * n + 256 > d) {  // uniform
                const float b0 = c[0], b1 = c[1], b2 = c[2], b3 = c[3];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int q = clampi(m + e, 0, d - 1) - at;
                    c[e] = q <= 0 ? b0 : (q == 1 ? b1 : (q == 2 ? b2 : b3));
                }
            }
#pragma unroll
            for (int e = 0; e < 3; ++e) c[4 + e] = next_lane(c[e]);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float iv = 0.f;
#pragma unroll
                for (int q = 0; q < 4; ++q) iv = fmaf(wz[V][q], c[e + q], iv);
                res[e] = fmaf(wgt[V], iv, res[e]);
            }
        }
        const int k = kQuadStep * n + 4 * lane;
        if (active && 4 * lane < kQuadStep && k < d) {
            float* const o = out + (size_t)a * d + k;
            if (k + 4 <= d) {
                *reinterpret_cast<quad_t*>(o) = quad_t{res[0], res[1], res[2], res[3]};
            } else {
#pragma unroll
                for (int e = 0; e < 3; ++e)
                    if (k + e < d) o[e] = res[e];
            }
        }
        __builtin_amdgcn_s_barrier();
    }
}

// n-volume merge weights: OCT weights wo[V][a] normalised over the volumes
// (the lowest-density volume where all vanish; the first on a tie) and OCTA
// weights wa[V][a] = OCT weight before normalisation times the resampled
// validity along the volume's slow axis, normalised (0 where all vanish)
__global__ void k_merge_weights_multi(const float* __restrict__ disp, int w, int h,
                                      const unsigned long long* __restrict__ grid, const MultiVols mv, double kappa,
                                      double tau, float* __restrict__ wo, float* __restrict__ wa)
{
    const int na = w * h;
    for (int a = blockIdx.x * blockDim.x + threadIdx.x; a < na; a += gridDim.x * blockDim.x) {
        const int i = a % w, j = a / w;
        double rho[kMaxVol], wt[kMaxVol], ow[kMaxVol];
        double sw = 0.0, so = 0.0;
        int lowest = 0;
        for (int V = 0; V < mv.n; ++V) {
            const float* dv = disp + ((size_t)V * na + a) * 3;
            int x0, y0, x1, y1;
            float fx, fy;
            bilin(i + dv[0], j + dv[1], w, h, x0, y0, x1, y1, fx, fy);
            const unsigned long long* G = grid + (size_t)V * na;
            rho[V] = ((1.0 - fx) * (1.0 - fy) * (double)G[(size_t)y0 * w + x0] +
                      (double)fx * (1.0 - fy) * (double)G[(size_t)y0 * w + x1] +
                      (1.0 - fx) * (double)fy * (double)G[(size_t)y1 * w + x0] +
                      (double)fx * (double)fy * (double)G[(size_t)y1 * w + x1]) / kFix;
            wt[V] = exp(-kappa * fmax(0.0, rho[V] - 1.0));
            if (wt[V] < tau) wt[V] = 0.0;
            sw += wt[V];
            if (rho[V] < rho[lowest]) lowest = V;
            ow[V] = 0.0;
            if (mv.valid[V])
                ow[V] = wt[V] * (mv.orient[V] == 0 ? valid_at(mv.valid[V], h, j, dv[1])
                                                    : valid_at(mv.valid[V], w, i, dv[0]));
            so += ow[V];
        }
        for (int V = 0; V < mv.n; ++V) {
            const double o = sw > 0 ? wt[V] / sw : (V == lowest ? 1.0 : 0.0);
            wo[(size_t)V * na + a] = (float)o;
            wa[(size_t)V * na + a] = (float)(so > 0 ? ow[V] / so : 0.0);
        }
    }
}

// one thread per output sample: the weighted sum over the volumes of the
// Eq. 2 interpolator's value at each volume's sample position
template <typename T>
__global__ __launch_bounds__(256) void k_merge_volume_multi(const MultiVols mv, const float* __restrict__ disp,
                                                            const float* __restrict__ wts, int w, int h, int d,
                                                            int dp, float* __restrict__ out)
{
    const int na = w * h;
    const size_t total = (size_t)na * d;
    for (size_t q = (size_t)blockIdx.x * blockDim.x + threadIdx.x; q < total;
         q += (size_t)gridDim.x * blockDim.x) {
        const int a = (int)(q / d), k = (int)(q - (size_t)a * d);
        const int i = a % w, j = a / w;
        float res = 0.f;
        for (int V = 0; V < mv.n; ++V) {
            const float wgt = wts[(size_t)V * na + a];
            if (wgt == 0.f) continue;
            const float* dv = disp + ((size_t)V * na + a) * 3;
            const float fxf = floorf(dv[0]), fyf = floorf(dv[1]), fzf = floorf(dv[2]);
            const int nx = i + (int)fxf, ny = j + (int)fyf, nz = k + (int)fzf;
            float wx[4], wy[4], wz[4];
            cr_w(dv[0] - fxf, wx);
            cr_w(dv[1] - fyf, wy);
            cr_w(dv[2] - fzf, wz);
            float v = 0.f;
            for (int b = 0; b < 4; ++b) {
                const size_t row = (size_t)clampi(ny - 1 + b, 0, h - 1) * w;
                for (int c = 0; c < 4; ++c) {
                    const size_t col = (row + clampi(nx - 1 + c, 0, w - 1)) * dp;  // volumes [h][w][dp]
                    float z = 0.f;
                    for (int e = 0; e < 4; ++e) z = fmaf(wz[e], ld<T>(mv.vol[V], col + clampi(nz - 1 + e, 0, d - 1)), z);
                    v = fmaf(wx[c] * wy[b], z, v);
                }
            }
            res = fmaf(wgt, v, res);
        }
        out[q] = res;
    }
}

inline int grid_for(size_t n, int cap = 65536)
{
    size_t g = (n + 255) / 256;
    if (g > (size_t)cap) g = cap;
    return g < 1 ? 1 : (int)g;
}

}  // namespace

hipError_t launch_density(const float* disp, int w, int h, unsigned long long* grid, hipStream_t s, int nvol)
{
    hipLaunchKernelGGL(k_density, dim3(grid_for((size_t)nvol * w * h)), dim3(256), 0, s, disp, w, h, grid, nvol);
    return hipGetLastError();
}
hipError_t launch_merge_weights_multi(const float* disp, int w, int h, const unsigned long long* grid,
                                      const MultiVols& mv, double kappa, double tau, float* wo, float* wa,
                                      hipStream_t s)
{
    hipLaunchKernelGGL(k_merge_weights_multi, dim3(grid_for((size_t)w * h)), dim3(256), 0, s, disp, w, h, grid, mv,
                       kappa, tau, wo, wa);
    return hipGetLastError();
}
hipError_t launch_merge_volume_multi(const MultiVols& mv, octmc_dtype dt, const float* disp, const float* wts, int w,
                                     int h, int d, int dp, float* out, hipStream_t s)
{
    const size_t n = (size_t)w * h * d;
    switch (dt) {
    case OCTMC_F32:
        hipLaunchKernelGGL(k_merge_volume_multi<float>, dim3(grid_for(n)), dim3(256), 0, s, mv, disp, wts, w, h, d,
                           dp, out);
        break;
    case OCTMC_BF16:
        hipLaunchKernelGGL(k_merge_volume_multi<bf16_t>, dim3(grid_for(n)), dim3(256), 0, s, mv, disp, wts, w, h, d,
                           dp, out);
        break;
    case OCTMC_F16:
        hipLaunchKernelGGL(k_merge_volume_multi<f16_t>, dim3(grid_for(n)), dim3(256), 0, s, mv, disp, wts, w, h, d,
                           dp, out);
        break;
    default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}
hipError_t launch_merge_weights(const float* disp, int w, int h, const unsigned long long* grid, const float* vx,
                                const float* vy, double kappa, double tau, float4* wts, hipStream_t s)
{
    hipLaunchKernelGGL(k_merge_weights, dim3(grid_for((size_t)w * h)), dim3(256), 0, s, disp, w, h, grid, vx, vy,
                       kappa, tau, wts);
    return hipGetLastError();
}
// With fewer A-scans the tiles do not fill the device and the merge takes
// k_merge_volume.  Merges of a structural volume, k_merge_volume / k_merge_tile: 91 x
// 91 x 400 82 / 42 us, 128 x 128 x 128 52 / 43; below the line 64 x 64 x 128 35 / 33,
// 64 x 64 x 400 44 / 38, 90 x 90 x 400 66 / 42, so it could lie lower.
constexpr int kMergeTileMinAscans = 8192;

template <typename T, int L>
static hipError_t launch_merge_t(const void* vx, const void* vy, const float* disp, const float4* wts, int which, int w,
                                 int h, int d, int dp, float* out, hipStream_t s)
{
    const size_t bytes = (size_t)w * h * dp * esize<T>::v;
    if (bytes >= (1ull << 31)) return hipErrorInvalidValue;  // 32-bit buffer offsets
    if (w * h >= kMergeTileMinAscans)
        hipLaunchKernelGGL((k_merge_tile<T, L>), dim3(struct_mx_blocks(w, h)), dim3(256), 0, s, vx, vy, disp, wts, which,
                           w, h, d, dp, (uint32_t)bytes, out);
    else
        hipLaunchKernelGGL(k_merge_volume<T>, dim3((w * h + 3) / 4), dim3(256), 0, s, vx, vy, disp, wts, which, w, h, d,
                           dp, (uint32_t)bytes, out);
    return hipGetLastError();
}

// Up to kMergeStep samples are one step of k_merge_volume, whose loads are shorter:
// both volumes of 300 x 300 x 61 203 us by it, 234 by k_merge_quads, x 4 164 and 211
// (x 62, two steps, 286 and 236); 128 x 128 x 61 60 and 67, x 62 75 and 67.
static hipError_t launch_merge_f32(const float* vx, const float* vy, const float* disp, const float4* wts, int which,
                                   int w, int h, int d, int dp, float* out, hipStream_t s)
{
    const size_t bytes = (size_t)w * h * d * 4;
    if (bytes >= (1ull << 31) || dp != d) return hipErrorInvalidValue;
    if (d <= kMergeStep)
        hipLaunchKernelGGL(k_merge_volume<float>, dim3((w * h + 3) / 4), dim3(256), 0, s, vx, vy, disp, wts, which, w, h, d,
                           dp, (uint32_t)bytes, out);
    else
        hipLaunchKernelGGL(k_merge_quads, dim3(8 * ((h + 7) / 8) * ((w + 3) / 4)), dim3(256), 0, s, vx, vy, disp, wts,
                           which, w, h, d, (uint32_t)bytes, out);
    return hipGetLastError();
}

hipError_t launch_merge_volume(const void* vx, const void* vy, octmc_dtype dt, const float* disp, const float4* wts,
                               int which, int w, int h, int d, int dp, float* out, hipStream_t s)
{
    const bool eight = mx_eight(d, dp);
    switch (dt) {
    case OCTMC_F32:
        return launch_merge_f32(static_cast<const float*>(vx), static_cast<const float*>(vy), disp, wts, which, w, h, d, dp,
                                out, s);
    case OCTMC_BF16:
        return eight ? launch_merge_t<bf16_t, 8>(vx, vy, disp, wts, which, w, h, d, dp, out, s)
                     : launch_merge_t<bf16_t, 4>(vx, vy, disp, wts, which, w, h, d, dp, out, s);
    case OCTMC_F16:
        return eight ? launch_merge_t<f16_t, 8>(vx, vy, disp, wts, which, w, h, d, dp, out, s)
                     : launch_merge_t<f16_t, 4>(vx, vy, disp, wts, which, w, h, d, dp, out, s);
    default:
        return hipErrorInvalidValue;
    }
}

}  // namespace octmc
