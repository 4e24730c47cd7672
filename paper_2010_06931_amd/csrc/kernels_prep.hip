// Ingest and pyramid kernels (run once per pair) and the level transition.
//
//   k_level       float32 -> storage type (round to nearest even), and the next
//                 level of the factor-2 pyramid (Sec. 2.1): coarse sample I is the
//                 mean of fine samples 2I and min(2I + 1, n - 1) along every axis
//   k_take_octa   OCTA volume with nearest-valid replacement of invalid B-scans
//                 (Sec. 2.5), and its depth mean (stand-in for the projection of
//                 Sec. 2.3)
//   k_upsample    level transition: twice the bilinear interpolation of the
//                 coarse field at ((i - 1/2) / 2, (j - 1/2) / 2)
#include <hip/hip_runtime.h>

#include "octmc_internal.h"
#include "row_quads.h"

namespace octmc {
namespace {

__device__ __forceinline__ unsigned short f32_to_bf16_rne(float f)
{
    uint32_t u = __builtin_bit_cast(uint32_t, f);
    if ((u & 0x7f800000u) == 0x7f800000u) return (unsigned short)((u >> 16) | ((u & 0xffffu) ? 0x40u : 0u));
    u += 0x7fffu + ((u >> 16) & 1u);
    return (unsigned short)(u >> 16);
}

template <int DT>
__device__ __forceinline__ unsigned short to_half(float v)
{
    if constexpr (DT == OCTMC_BF16) return f32_to_bf16_rne(v);
    return __builtin_bit_cast(unsigned short, (_Float16)v);
}

typedef unsigned short halves_t __attribute__((ext_vector_type(4), aligned(4)));
typedef float pair_t __attribute__((ext_vector_type(2), aligned(4)));

// Four samples of an A-scan in the storage type, from sample k; an odd depth of
// 16-bit storage is followed by a copy of its last sample (dp = d + 1).
template <int DT>
__device__ __forceinline__ void store_quad(void* __restrict__ st, size_t column, int k, int d, int dp, const float (&v)[4])
{
    if constexpr (DT == OCTMC_F32) {
        float* o = static_cast<float*>(st) + column * dp + k;
        if (k + 4 <= d) {
            *reinterpret_cast<quad_t*>(o) = quad_t{v[0], v[1], v[2], v[3]};
        } else {
            for (int e = 0; e < 4 && k + e < d; ++e) o[e] = v[e];
        }
    } else {
        unsigned short* o = static_cast<unsigned short*>(st) + column * dp + k;
        if (k + 4 <= dp) {
            *reinterpret_cast<halves_t*>(o) = halves_t{to_half<DT>(v[0]), to_half<DT>(v[1]), to_half<DT>(v[2]), to_half<DT>(v[3])};
        } else {
            for (int e = 0; e < 4 && k + e < dp; ++e) o[e] = to_half<DT>(v[e]);
        }
    }
}

// One level of the pyramid of one or two volumes (blockIdx.y), and, by the last
// blockIdx.y, of their images and validity: the level in the storage type and the
// next one in float32, from one reading.  A thread takes four samples of the 2 x 2
// A-scans of one coarse A-scan with 16-byte loads.  Bound by the memory: 300 x
// 300 x 640 float32, both volumes, 980 MB written and read: 178 us, 5.5 TB/s
// (storage and pyramid as kernels of their own, 4 bytes a load: 370 us).
template <int DT>
__global__ __launch_bounds__(256) void k_level(const LevelJob J)
{
    const int w = J.w, h = J.h, d = J.d, w2 = (w + 1) / 2, h2 = (h + 1) / 2, d2 = (d + 1) / 2;
    if ((int)blockIdx.y == J.nvol) {
        for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < J.nvol * w2 * h2; t += gridDim.x * blockDim.x) {
            const int V = t >= w2 * h2, q = t - V * w2 * h2;
            const float* __restrict__ in = J.image[V];
            const int I = q % w2, Y = q / w2;
            const int y1 = min(2 * Y + 1, h - 1), x1 = min(2 * I + 1, w - 1);
            J.next_image[V][q] = 0.25f * ((in[(size_t)2 * Y * w + 2 * I] + in[(size_t)2 * Y * w + x1]) +
                                          (in[(size_t)y1 * w + 2 * I] + in[(size_t)y1 * w + x1]));
        }
        if (blockIdx.x == 0) {
#pragma unroll
            for (int V = 0; V < 2; ++V) {
                if (V >= J.nvol) break;
                const int n = J.nvalid[V], n2 = (n + 1) / 2;
                for (int q = threadIdx.x; q < n2; q += blockDim.x)
                    J.next_valid[V][q] = 0.5f * (J.valid[V][2 * q] + J.valid[V][min(2 * q + 1, n - 1)]);
            }
        }
        return;
    }
    const unsigned quads = (unsigned)(d + 3) / 4;
    const unsigned q = blockIdx.x * blockDim.x + threadIdx.x, c = q / quads;
    if (c >= (unsigned)w2 * (unsigned)h2) return;
    const int k = 4 * (int)(q - c * quads);
    const int Y = (int)(c / (unsigned)w2), I = (int)(c - (unsigned)Y * (unsigned)w2);
    const float* __restrict__ in = J.in[blockIdx.y];
    void* __restrict__ st = J.store[blockIdx.y];
    float* __restrict__ next = J.next[blockIdx.y];
    float v[4][4];
    size_t column[4];
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        const int x = min(2 * I + (a & 1), w - 1), y = min(2 * Y + (a >> 1), h - 1);
        column[a] = (size_t)y * w + x;
        const float* __restrict__ col = in + column[a] * d;
        if (k + 4 <= d) {
            const quad_t t = *reinterpret_cast<const quad_t*>(col + k);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[a][e] = t[e];
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[a][e] = col[min(k + e, d - 1)];
        }
    }
    if (st) {
#pragma unroll
        for (int a = 0; a < 4; ++a)
            if (2 * I + (a & 1) < w && 2 * Y + (a >> 1) < h) store_quad<DT>(st, column[a], k, d, J.dp, v[a]);
    }
    if (next) {
        float m[2];
#pragma unroll
        for (int e = 0; e < 2; ++e)
            m[e] = 0.125f * (((v[0][2 * e] + v[0][2 * e + 1]) + (v[1][2 * e] + v[1][2 * e + 1])) +
                             ((v[2][2 * e] + v[2][2 * e + 1]) + (v[3][2 * e] + v[3][2 * e + 1])));
        float* o = next + (size_t)c * d2 + k / 2;
        if (k / 2 + 2 <= d2) *reinterpret_cast<pair_t*>(o) = pair_t{m[0], m[1]};
        else o[0] = m[0];
    }
}

// The OCTA volume as it is kept for the merge, invalid B-scans replaced by the
// B-scan that `from` names (null: none are), and the depth means of its A-scans
// (null: not wanted).  The two volumes may be one: a replacement is a B-scan that
// stays.  300 x 300 x 640, 461 MB: 85 us, 5.4 TB/s (copy, replacement and mean as
// launches of their own: 260 us).
__global__ __launch_bounds__(256) void k_take_octa(const float* in, float* out, int w, int na, int d,
                                                   const int* __restrict__ from, int V, float* __restrict__ mean)
{
    const int part = threadIdx.x & (kRowLanes - 1);
    const int a = blockIdx.x * (blockDim.x / kRowLanes) + threadIdx.x / kRowLanes;
    if (a >= na) return;  // whole rows; the sum below stays within one
    const int j = a / w, i = a - j * w;
    int src = a;
    if (from) src = V == 0 ? from[j] * w + i : j * w + from[i];
    const float* col = in + (size_t)src * d;
    float* o = out + (size_t)a * d;
    const bool keep = src == a && in == out;
    double s = 0.0;
    for (int k0 = 0; k0 < d; k0 += kRowLoads * kRowStep) {
        Quad q[kRowLoads];
#pragma unroll
        for (int g = 0; g < kRowLoads; ++g) {
            if (k0 + g * kRowStep >= d) break;
            q[g] = load_quad(col, k0 + g * kRowStep + 4 * part, d);
        }
#pragma unroll
        for (int g = 0; g < kRowLoads; ++g) {
            const int k = k0 + g * kRowStep + 4 * part;
            if (k0 + g * kRowStep >= d) break;
            if (k < d) {
                if (keep) {
                } else if (k + 4 <= d) {
                    *reinterpret_cast<quad_t*>(o + k) = q[g].v;
                } else {
                    for (int e = q[g].first; e < 4; ++e) o[k + e - q[g].first] = q[g].v[e];
                }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) s += e >= q[g].first ? (double)q[g].v[e] : 0.0;
        }
    }
    if (!mean) return;
    s = row_sum(s);
    if (part == 0) mean[a] = (float)(s / d);
}

// The B-scan whose data each B-scan takes: itself if it is valid or none is, or
// the nearest valid one (the lower index on a tie).  One block.
__global__ __launch_bounds__(256) void k_nearest_valid(const float* __restrict__ valid, int nb, int* __restrict__ from)
{
    __shared__ int any;
    if (threadIdx.x == 0) any = 0;
    __syncthreads();
    for (int b = threadIdx.x; b < nb; b += blockDim.x)
        if (valid[b] > 0.5f) any = 1;  // every writer stores 1
    __syncthreads();
    for (int b = threadIdx.x; b < nb; b += blockDim.x) {
        int src = b;
        if (any && !(valid[b] > 0.5f)) {
            src = -1;
            for (int dist = 1; dist < nb && src < 0; ++dist) {
                if (b - dist >= 0 && valid[b - dist] > 0.5f) src = b - dist;
                else if (b + dist < nb && valid[b + dist] > 0.5f) src = b + dist;
            }
        }
        from[b] = src;
    }
}

__global__ void k_count_nonfinite(const float* __restrict__ v, size_t n, unsigned* counter)
{
    unsigned bad = 0;
    for (size_t q = (size_t)blockIdx.x * blockDim.x + threadIdx.x; q < n; q += (size_t)gridDim.x * blockDim.x)
        bad += !isfinite(v[q]);
    for (int off = 32; off > 0; off >>= 1) bad += __shfl_xor(bad, off, 64);
    if ((threadIdx.x & 63) == 0 && bad) atomicAdd(counter, bad);
}

__global__ void k_upsample(const double* __restrict__ C, int wc, int hc, double* __restrict__ Fo, int wf, int hf,
                           int nvol)
{
    const int total = nvol * wf * hf;
    for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < total; q += gridDim.x * blockDim.x) {
        const int V = q / (wf * hf);
        const int r = q % (wf * hf);
        const int i = r % wf, j = r / wf;
        double x = (i - 0.5) * 0.5, y = (j - 0.5) * 0.5;
        x = fmin(fmax(x, 0.0), (double)(wc - 1));
        y = fmin(fmax(y, 0.0), (double)(hc - 1));
        const int x0 = (int)floor(x), y0 = (int)floor(y);
        const int x1 = min(x0 + 1, wc - 1), y1 = min(y0 + 1, hc - 1);
        const double fx = x - x0, fy = y - y0;
        const double* CV = C + (size_t)V * wc * hc * 3;
        for (int c = 0; c < 3; ++c) {
            const double v00 = CV[((size_t)y0 * wc + x0) * 3 + c], v10 = CV[((size_t)y0 * wc + x1) * 3 + c];
            const double v01 = CV[((size_t)y1 * wc + x0) * 3 + c], v11 = CV[((size_t)y1 * wc + x1) * 3 + c];
            const double v = (1 - fy) * ((1 - fx) * v00 + fx * v10) + fy * ((1 - fx) * v01 + fx * v11);
            Fo[(size_t)q * 3 + c] = 2.0 * v;
        }
    }
}

inline int grid_for(size_t n, int block = 256, int cap = 65536)
{
    size_t g = (n + block - 1) / block;
    if (g > (size_t)cap) g = cap;
    return g < 1 ? 1 : (int)g;
}

// Input validity of an OCTA volume (Sec. 2.2).  Step 1: mean decorrelation
// of every B-scan (one block per B-scan, float64, fixed-order sum): rows j
// of the X-fast scan (V = 0), columns i of the Y-fast scan (V = 1).
constexpr int kVB = 256;

__device__ __forceinline__ double block_sum_d(double v, double* sh)
{
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int s = kVB / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
        __syncthreads();
    }
    const double r = sh[0];
    __syncthreads();
    return r;
}

__global__ __launch_bounds__(kVB) void k_bscan_mean(const float* __restrict__ vol, int w, int h, int d, int V,
                                                    double* __restrict__ m)
{
    __shared__ double sh[kVB];
    const int b = blockIdx.x;
    const int na = V == 0 ? w : h;
    double s = 0.0;
    if (V == 0) {  // one contiguous run of w * d samples
        const float* p = vol + (size_t)b * w * d;
        const size_t n = (size_t)w * d;
        for (size_t q = threadIdx.x; q < n; q += kVB) s += (double)p[q];
    } else {  // h A-scans of d samples, w * d apart
        for (int o = 0; o < h; ++o) {
            const float* p = vol + ((size_t)o * w + b) * d;
            for (int k = threadIdx.x; k < d; k += kVB) s += (double)p[k];
        }
    }
    s = block_sum_d(s, sh);
    if (threadIdx.x == 0) m[b] = s / ((double)na * (double)d);
}

// Step 2 (one block): mean mu and population standard deviation sigma of the
// B-scan means; B-scan b is flagged if m_b > mu + 3 sigma, and valid (1) if
// none of b - 2 .. b + 2 is flagged.
__global__ __launch_bounds__(kVB) void k_validity(const double* __restrict__ m, int nb, float* __restrict__ v)
{
    __shared__ double sh[kVB];
    double s = 0.0;
    for (int b = threadIdx.x; b < nb; b += kVB) s += m[b];
    const double mu = block_sum_d(s, sh) / nb;
    double q = 0.0;
    for (int b = threadIdx.x; b < nb; b += kVB) q += (m[b] - mu) * (m[b] - mu);
    const double thr = mu + 3.0 * sqrt(block_sum_d(q, sh) / nb);
    for (int b = threadIdx.x; b < nb; b += kVB) {
        bool bad = false;
        for (int o = b - 2; o <= b + 2; ++o)
            if (o >= 0 && o < nb && m[o] > thr) bad = true;
        v[b] = bad ? 0.f : 1.f;
    }
}

}  // namespace

hipError_t launch_validity(const float* vol, int w, int h, int d, int V, double* means, float* valid,
                           hipStream_t s)
{
    const int nb = V == 0 ? h : w;
    hipLaunchKernelGGL(k_bscan_mean, dim3(nb), dim3(kVB), 0, s, vol, w, h, d, V, means);
    hipLaunchKernelGGL(k_validity, dim3(1), dim3(kVB), 0, s, means, nb, valid);
    return hipGetLastError();
}

hipError_t launch_level(const LevelJob& J, octmc_dtype dt, hipStream_t s)
{
    // only 16-bit storage is padded, to a whole number of sample pairs
    if (J.dp < J.d || (dt == OCTMC_F32 ? J.dp != J.d : J.dp % 2 != 0)) return hipErrorInvalidValue;
    const unsigned quads = (unsigned)((J.w + 1) / 2) * (unsigned)((J.h + 1) / 2) * ((unsigned)(J.d + 3) / 4);
    const dim3 grid((quads + 255) / 256, J.nvol + (J.next_image[0] ? 1 : 0));
    switch (dt) {
    case OCTMC_F32: hipLaunchKernelGGL(k_level<OCTMC_F32>, grid, dim3(256), 0, s, J); break;
    case OCTMC_BF16: hipLaunchKernelGGL(k_level<OCTMC_BF16>, grid, dim3(256), 0, s, J); break;
    case OCTMC_F16: hipLaunchKernelGGL(k_level<OCTMC_F16>, grid, dim3(256), 0, s, J); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}
hipError_t launch_take_octa(const float* in, float* out, int w, int h, int d, const int* from, int V, float* mean,
                            hipStream_t s)
{
    const int na = w * h, rows = 256 / kRowLanes;
    hipLaunchKernelGGL(k_take_octa, dim3((na + rows - 1) / rows), dim3(256), 0, s, in, out, w, na, d, from, V, mean);
    return hipGetLastError();
}
hipError_t launch_nearest_valid(const float* valid, int nb, int* from, hipStream_t s)
{
    hipLaunchKernelGGL(k_nearest_valid, dim3(1), dim3(256), 0, s, valid, nb, from);
    return hipGetLastError();
}
hipError_t launch_count_nonfinite(const float* v, size_t n, unsigned* counter, hipStream_t s)
{
    hipLaunchKernelGGL(k_count_nonfinite, dim3(grid_for(n)), dim3(256), 0, s, v, n, counter);
    return hipGetLastError();
}
hipError_t launch_upsample(const double* coarse, int wc, int hc, double* fine, int wf, int hf, hipStream_t s,
                           int nvol)
{
    hipLaunchKernelGGL(k_upsample, dim3(grid_for((size_t)nvol * wf * hf)), dim3(256), 0, s, coarse, wc, hc, fine, wf,
                       hf, nvol);
    return hipGetLastError();
}

}  // namespace octmc
