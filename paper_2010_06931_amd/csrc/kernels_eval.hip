// Hot-path kernels: one evaluation of the registration objective and its
// gradient (Eqs. 1-10 of Ploner et al., without the stage-1 tilt term).
//
//   k_sum     sum of the displacements of both scans (mean term M); part of
//             the launches of k_struct, k_struct2 and k_struct_mx otherwise
//   k_struct  per output A-scan: resample both structural volumes with
//             their displacement (Eq. 2), residual, pseudo-Huber loss (Eq. 4)
//             and the depth sums of the loss and of its gradient with respect
//             to the A-scan's displacement; one depth sample per lane (float32
//             storage, and 16-bit volumes of odd depth in the caller's layout; fewer A-scans)
//   k_struct2 the same with two 16-bit samples per lane (small levels: an odd
//             depth is stored with one padding sample)
//   k_struct_mx the same for volumes of many A-scans, the lateral
//             resampling on the matrix cores
//   k_struct_multi, k_struct_multi1, k_multi_mx  the structural partials of
//             every volume pair of n = 3 or 4 volumes, each volume resampled
//             once (16-bit, float32, many A-scans; the last not for three of float32)
//   k_combine per output A-scan: en face residual (Eq. 7), resampled
//             validity (Eq. 5), weight delta (Eq. 8), combination with eta
//             (Eq. 9), scan-order regulariser, mean term, gradient; float64
//             block partials (k_combine_few: few A-scans, with the sums of the
//             displacements and the final sums in the same launch)
//   k_finalize the float64 global sums in a fixed order (one block per job;
//             a kernel boundary, not a device-scope fence per block, makes
//             the partials visible)
#include <hip/hip_runtime.h>

#include "octmc_internal.h"
#include "tile_blend.h"

namespace octmc {

namespace {

template <typename T>
__device__ __forceinline__ float ldv(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff);
template <>
__device__ __forceinline__ float ldv<float>(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
}
template <>
__device__ __forceinline__ float ldv<bf16_t>(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff)
{
    const unsigned short b = __builtin_amdgcn_raw_buffer_load_b16(r, voff, soff, 0);
    return __builtin_bit_cast(float, (uint32_t)b << 16);
}
template <>
__device__ __forceinline__ float ldv<f16_t>(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff)
{
    const unsigned short b = __builtin_amdgcn_raw_buffer_load_b16(r, voff, soff, 0);
    return (float)__builtin_bit_cast(_Float16, b);
}
// Stage 1 (rough axial prealignment) evaluates at dx = dy = 0, where the
// lateral weights are (0, 1, 0, 0) in x and y: the blend of the 16 columns
// is exactly the centre column (index 5; every other product is an exact 0),
// so the axial kernels load that column alone and skip the lateral adjoint.
constexpr int kCentre = 5;

// Per-scan stencil of one output A-scan: 16 lateral columns with their
// (wave-uniform) byte offsets and blend weights, and the depth taps.  The
// lateral derivative taps are recomputed after the depth loop (from tx, ty,
// or from make_stencils' per-lane taps), so they do not occupy registers
// during it.
struct Stencil {
    float w[16];
    uint32_t off[16];
    float wz[4], dwz[4];
    float tx, ty;
    int base;  // source sample of the first depth tap of output sample 0
};

// One scan's stencil, every tap and product computed on wave-uniform values
// (the two-samples-per-lane kernel's form: with the per-lane form below its
// register allocation changed and the BF16 kernel ran 21 % slower).
template <typename T>
__device__ __forceinline__ void make_stencil(Stencil& s, int i, int j, float dx, float dy, float dz, int w,
                                             int h, int d)
{
    int nx, ny, nz;
    float tx, ty, tz;
    split(i, uni(dx), nx, tx);
    split(j, uni(dy), ny, ty);
    split(0, uni(dz), nz, tz);
    nx = uni(nx);
    ny = uni(ny);
    nz = uni(nz);
    float wx[4], dwx[4], wy[4], dwy[4];
    cr_taps(uni(tx), wx, dwx);
    cr_taps(uni(ty), wy, dwy);
    cr_taps(uni(tz), s.wz, s.dwz);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        s.wz[c] = uni(s.wz[c]);
        s.dwz[c] = uni(s.dwz[c]);
    }
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const int row = clampi(ny - 1 + b, 0, h - 1);
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            const int col = clampi(nx - 1 + a, 0, w - 1);
            s.off[b * 4 + a] = (uint32_t)uni((int)((uint32_t)(row * w + col) * (uint32_t)d * esize<T>::v));
            s.w[b * 4 + a] = uni(wx[a] * wy[b]);
        }
    }
    s.tx = uni(tx);
    s.ty = uni(ty);
    s.base = uni(nz - 1);
}

// The stencil of the axial kernels (every displacement has dx = dy = 0, so
// the lateral weights are (0, 1, 0, 0) along x and y and the blend is the
// centre column): the depth taps, the centre column's offset and the base;
// the other offsets and weights are left unset (the axial kernels read
// neither).
template <typename T>
__device__ __forceinline__ void make_stencil_axial(Stencil& s, int i, int j, float dz, int w, int d)
{
    int nz;
    float tz;
    split(0, uni(dz), nz, tz);
    cr_taps(uni(tz), s.wz, s.dwz);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        s.wz[c] = uni(s.wz[c]);
        s.dwz[c] = uni(s.dwz[c]);
    }
    s.off[kCentre] = (uint32_t)((uint32_t)(j * w + i) * (uint32_t)d * esize<T>::v);
    s.tx = s.ty = 0.f;
    s.base = uni(nz) - 1;
}

// Both scans' stencils of one output A-scan.  The taps are computed one per
// lane, lane 12 V + 4 p + c holding tap c of scan V's coordinate p (0: x,
// 1: y, 2: z), and the lateral weights w_ab = wx_a wy_b one per lane (lane
// 32 + 16 V + 4 b + a); each is then read out as a wave-uniform value.  That
// takes a few dozen instructions per wave instead of computing every tap and
// product on uniform operands one after another.  tw and tdw keep each
// lane's tap and tap derivative for the lateral gradient after the depth
// loop (tap_x/tap_y read them).
template <typename T>
__device__ __forceinline__ void make_stencils(Stencil& SX, Stencil& SY, float& tw, float& tdw, int i, int j,
                                              const float* dX, const float* dY, int w, int h, int d, int lane)
{
    float t[6];
    int n[6];
    split(i, uni(dX[0]), n[0], t[0]);
    split(j, uni(dX[1]), n[1], t[1]);
    split(0, uni(dX[2]), n[2], t[2]);
    split(i, uni(dY[0]), n[3], t[3]);
    split(j, uni(dY[1]), n[4], t[4]);
    split(0, uni(dY[2]), n[5], t[5]);
#pragma unroll
    for (int k = 0; k < 6; ++k) n[k] = uni(n[k]);
    const int p = lane >> 2, c = lane & 3;
    float tl = t[0];
#pragma unroll
    for (int k = 1; k < 6; ++k) tl = p == k ? t[k] : tl;
    float wv[4], dv[4];
    cr_taps(tl, wv, dv);
    float wl = wv[0], dl = dv[0];
#pragma unroll
    for (int k = 1; k < 4; ++k) {
        wl = c == k ? wv[k] : wl;
        dl = c == k ? dv[k] : dl;
    }
    tw = wl;
    tdw = dl;
    // lanes 32 + 16 V + 4 b + a: wx_a wy_b of scan V
    const int V = (lane >> 4) & 1, b = (lane >> 2) & 3, a = lane & 3;
    const float prod = __shfl(wl, 12 * V + a) * __shfl(wl, 12 * V + 4 + b);
    const int pb = __builtin_bit_cast(int, prod), wb = __builtin_bit_cast(int, wl), db = __builtin_bit_cast(int, dl);
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        SX.w[q] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(pb, 32 + q));
        SY.w[q] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(pb, 48 + q));
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        SX.wz[k] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(wb, 8 + k));
        SX.dwz[k] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(db, 8 + k));
        SY.wz[k] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(wb, 20 + k));
        SY.dwz[k] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(db, 20 + k));
    }
    Stencil* S[2] = {&SX, &SY};
#pragma unroll
    for (int v = 0; v < 2; ++v) {
        const int nx = n[3 * v], ny = n[3 * v + 1];
#pragma unroll
        for (int bb = 0; bb < 4; ++bb) {
            const int row = clampi(ny - 1 + bb, 0, h - 1);
#pragma unroll
            for (int aa = 0; aa < 4; ++aa) {
                const int col = clampi(nx - 1 + aa, 0, w - 1);
                S[v]->off[bb * 4 + aa] = (uint32_t)uni((int)((uint32_t)(row * w + col) * (uint32_t)d * esize<T>::v));
            }
        }
        S[v]->base = n[3 * v + 2] - 1;
    }
}

// The lateral taps and their derivatives of scan V (x: p = 0, y: p = 1),
// read back from make_stencils' per-lane values.
__device__ __forceinline__ void lateral_taps(float tw, float tdw, int V, int p, float w[4], float dw[4])
{
    const int wb = __builtin_bit_cast(int, tw), db = __builtin_bit_cast(int, tdw);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        w[k] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(wb, 12 * V + 4 * p + k));
        dw[k] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(db, 12 * V + 4 * p + k));
    }
}

// Depth is processed in steps of 61 output samples on 64 lanes: lane l holds
// source sample base + 61 n + l, output lane l (< 61) reads source lanes
// l .. l+3, and the adjoint of output lane l goes to the same source lanes.
// Every step is therefore self-contained (a source sample shared by two
// steps receives each step's part of the adjoint separately).
constexpr int kOutPerStep = 61;

template <typename T>
__device__ __forceinline__ void load_cols(float (&v)[16], __amdgpu_buffer_rsrc_t r, const Stencil& s, int step,
                                          int lane, int d)
{
    const int m = clampi(s.base + step * kOutPerStep + lane, 0, d - 1);
    const uint32_t voff = (uint32_t)m * esize<T>::v;
#pragma unroll
    for (int q = 0; q < 16; ++q) v[q] = ldv<T>(r, voff, s.off[q]);
}


__device__ __forceinline__ float blend(const float (&v)[16], const Stencil& s)
{
    float c = 0.f;
#pragma unroll
    for (int q = 0; q < 16; ++q) c = fmaf(s.w[q], v[q], c);
    return c;
}

// Whole-wave lane shifts (DPP): shl1 gives lane l the value of lane l + 1,
// shr1 that of lane l - 1; a lane whose source lies outside the wave reads 0
// (bound control), so the shift can fold into the instruction that uses it.
__device__ __forceinline__ float shl1(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x130, 0xF, 0xF, true));
}
__device__ __forceinline__ float shr1(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x138, 0xF, 0xF, true));
}

// Sum over the wave in float32, left in lane 63: within each row of 16 lanes
// (DPP row shifts; the last lane of a row ends with the row's sum), then two
// row broadcasts (rows 1 and 3 add the last lane of the row before them, then
// rows 2 and 3 add lane 31): (r3 + r2) + (r1 + r0).  Six DPP additions, no
// lane reads.
__device__ __forceinline__ float wave_sum_last(float x)
{
    float v = row_shr_add<1>(x);
    v = row_shr_add<2>(v);
    v = row_shr_add<4>(v);
    v = row_shr_add<8>(v);
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x142, 0xA, 0xF, false));
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x143, 0xC, 0xF, false));
    return v;
}
// the same sum, wave-uniform (lane 63's)
__device__ __forceinline__ float wave_sum(float x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, wave_sum_last(x)), 63));
}

// Sums of N (4 or 8) values over a wave by halving: at each step a lane keeps
// half of its values and gives the other half to its partner, so N - 1 + log2(64
// / N) exchanges do.  Lane l is left with the sum of value l / (64 / N).
template <int N>
__device__ __forceinline__ double wave_sums(const double (&in)[N], int lane)
{
    double v[N];
#pragma unroll
    for (int q = 0; q < N; ++q) v[q] = in[q];
    int m = 32;
#pragma unroll
    for (int half = N / 2; half > 0; half >>= 1, m >>= 1) {
#pragma unroll
        for (int q = 0; q < half; ++q) {
            const bool up = lane & m;
            const double give = up ? v[q] : v[q + half], keep = up ? v[q + half] : v[q];
            v[q] = keep + __shfl_xor(give, m);
        }
    }
    for (; m > 0; m >>= 1) v[0] += __shfl_xor(v[0], m);
    return v[0];
}

// The waves' sums, one row per wave; after the next barrier wave_rows adds them
// in order.
template <int N>
__device__ __forceinline__ void store_wave_sums(const double (&v)[N], double (&sh)[kRedBlock / 64][N])
{
    const int lane = threadIdx.x & 63;
    const double s = wave_sums<N>(v, lane);
    if (lane % (64 / N) == 0) sh[threadIdx.x >> 6][lane / (64 / N)] = s;
}
template <int N>
__device__ __forceinline__ double wave_rows(const double (&sh)[kRedBlock / 64][N], int q)
{
    double s = sh[0][q];
#pragma unroll
    for (int r = 1; r < kRedBlock / 64; ++r) s += sh[r][q];
    return s;
}

template <int N>
__device__ __forceinline__ void block_reduce_store(const double (&v)[N], double* blk_row)
{
    __shared__ double sh[kRedBlock / 64][N];
    store_wave_sums<N>(v, sh);
    __syncthreads();
    if ((int)threadIdx.x < N) blk_row[threadIdx.x] = wave_rows<N>(sh, threadIdx.x);
}

// Block b of nblk of the sum of the displacements of both slots.
__device__ __forceinline__ void sum_block(const float* __restrict__ dx, const float* __restrict__ dy, int na, int nblk,
                                          int b, double* blk)
{
    double v[4] = {0, 0, 0, 0};
    for (int q = b * kRedBlock + threadIdx.x; q < 2 * na; q += nblk * kRedBlock) {
        const float* dq = q < na ? dx + (size_t)q * 3 : dy + (size_t)(q - na) * 3;
        v[0] += (double)dq[0];
        v[1] += (double)dq[1];
        v[2] += (double)dq[2];
    }
    block_reduce_store<4>(v, blk + (size_t)b * 4);
}

// The first blocks of a structural launch sum the displacements of its jobs (a
// multiple of the 8 XCDs, so that the others stay where they were): a launch less,
// 4.8 of 81 us for 251 x 251 x 233 BF16.
__device__ __forceinline__ bool struct_sums(const StructJobs& jobs)
{
    const int b = blockIdx.x;
    if (b >= jobs.sum_blocks) return false;
    for (int q = 0; q < jobs.n; ++q) {  // block-uniform
        const StructJob& J = jobs.j[q];
        if (b >= J.sum_begin && b < J.sum_begin + J.nsum)
            sum_block(J.disp, J.disp + (size_t)J.na * 3, J.na, J.nsum, b - J.sum_begin, J.sum_blk);
    }
    return true;
}

// The count of finished blocks of a combination of few A-scans is cleared by the
// structural launch before it (for the fused pass of several volumes by the launch of
// their field sums), so that no evaluation depends on how an earlier one ended
// (evaluations that overlapped on one object may leave any count).  The lane
// that stores A-scan 0 does it, at the end: at the start every wave would wait for
// one more load of its arguments (64 x 64 x 128 21.1 -> 21.6 us).
__device__ __forceinline__ void clear_ticket(unsigned* ticket, int a)
{
    if (a == 0 && ticket) *ticket = 0u;
}

template <typename T, bool AXIAL>
__global__ __launch_bounds__(256) void k_struct(const StructJobs jobs)
{
    if (jobs.skip && *jobs.skip) return;
    if (!AXIAL && struct_sums(jobs)) return;
    const int wv = uni((int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    const int lb = xcd_block((int)blockIdx.x - jobs.sum_blocks, (int)gridDim.x - jobs.sum_blocks);
    int jid = -1;
    for (int q = 0; q < jobs.n; ++q)
        if (lb >= jobs.j[q].blk_begin) jid = q;
    if (jid < 0) return;  // whole block
    const StructJob& J = jobs.j[jid];
    const int w = J.w, h = J.h, d = J.d;
    const int dp = J.dp;  // storage pitch: d, or d + 1 (a padding sample) for an odd depth in 16-bit storage
    // 2 x 2 tile of output A-scans per workgroup, one per wave.  The tile
    // rows form 8 bands (one per XCD when the job fills the grid); a band is
    // swept column by column, so the rows a tile reads are still in that
    // XCD's L2 when the neighbouring column of tiles reads them again.
    const int tpr = (w + 1) >> 1;
    const int trows = (h + 1) >> 1;
    const int rpb = (trows + 7) >> 3;
    const int t = lb - J.blk_begin;
    const int band = t / (rpb * tpr), tb = t - band * (rpb * tpr);
    const int trow = band * rpb + tb % rpb;
    if (t >= 8 * rpb * tpr || trow >= trows) return;  // whole block
    const int i = 2 * (tb / rpb) + (wv & 1);
    const int j = 2 * trow + (wv >> 1);
    // With float32 storage the waves of a tile step through depth together
    // (one barrier per step), so the columns they share are still in the L1
    // cache when the others read them (measured: no gain for 16-bit
    // storage).  A wave outside the scan only takes part in the barriers.
    const bool active = i < w && j < h;  // wave-uniform
    const int a = uni(active ? j * w + i : 0);
    const float* dX = J.disp + (size_t)a * 3;
    const float* dY = J.disp + ((size_t)J.na + a) * 3;
    Stencil SX, SY;
    float tw = 0.f, tdw = 0.f;
    if constexpr (AXIAL) {
        make_stencil_axial<T>(SX, i, j, dX[2], w, dp);
        make_stencil_axial<T>(SY, i, j, dY[2], w, dp);
    } else {
        make_stencils<T>(SX, SY, tw, tdw, i, j, dX, dY, w, h, dp, lane);
    }
    const __amdgpu_buffer_rsrc_t rx =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(J.sx), (short)0, (int)J.vol_bytes, kRsrcWord3);
    const __amdgpu_buffer_rsrc_t ry =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(J.sy), (short)0, (int)J.vol_bytes, kRsrcWord3);
    const float eps = J.eps_h;
    const float inv_eps = 1.0f / J.eps_h;

    float sx[16], sy[16];
    float PX[16], PY[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) PX[q] = PY[q] = 0.f;
    float lam = 0.f, gzx = 0.f, gzy = 0.f;
    const int nsteps = (d + kOutPerStep - 1) / kOutPerStep;
    for (int n = 0; n < nsteps; ++n) {
        if (active) {
            float vx, vy;
            if constexpr (AXIAL) {
                const int m = clampi(SX.base + n * kOutPerStep + lane, 0, d - 1);
                const int my = clampi(SY.base + n * kOutPerStep + lane, 0, d - 1);
                vx = ldv<T>(rx, (uint32_t)m * esize<T>::v, SX.off[kCentre]);
                vy = ldv<T>(ry, (uint32_t)my * esize<T>::v, SY.off[kCentre]);
            } else {
                load_cols<T>(sx, rx, SX, n, lane, d);
                load_cols<T>(sy, ry, SY, n, lane, d);
                vx = blend(sx, SX);
                vy = blend(sy, SY);
            }
            // blended columns, then the depth interpolation of Eq. 2 and its
            // depth derivative: output lane l reads source lanes l .. l + 3
            float ix = 0.f, izx = 0.f, iy = 0.f, izy = 0.f;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                ix = fmaf(SX.wz[c], vx, ix);
                izx = fmaf(SX.dwz[c], vx, izx);
                iy = fmaf(SY.wz[c], vy, iy);
                izy = fmaf(SY.dwz[c], vy, izy);
                if (c < 3) {
                    vx = shl1(vx);
                    vy = shl1(vy);
                }
            }
            // residual (Eq. 2) and pseudo-Huber loss (Eq. 4) in the form
            // eps u^2 / (sqrt(1 + u^2) + 1), u = r / eps, and its derivative u / sqrt(1 + u^2)
            const float r = ix - iy;
            const float u = r * inv_eps;
            const float q = u * u;
            const float rs = __builtin_amdgcn_rsqf(1.f + q);
            const float sq = (1.f + q) * rs;
            const bool valid = lane < kOutPerStep && (n * kOutPerStep + lane) < d;
            const float L = valid ? eps * q * __builtin_amdgcn_rcpf(sq + 1.f) : 0.f;
            const float G = valid ? u * rs : 0.f;
            lam += L;
            gzx += valid ? G * izx : 0.f;
            gzy += valid ? G * izy : 0.f;
            if constexpr (!AXIAL) {
                // adjoint of the depth interpolation: source lane l collects the
                // derivatives of output lanes l - 3 .. l (invalid lanes carry 0)
                float hx = 0.f, hy = 0.f, g = G;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    hx = fmaf(SX.wz[c], g, hx);
                    hy = fmaf(SY.wz[c], g, hy);
                    if (c < 3) g = shr1(g);
                }
#pragma unroll
                for (int q2 = 0; q2 < 16; ++q2) {
                    PX[q2] = fmaf(sx[q2], hx, PX[q2]);
                    PY[q2] = fmaf(sy[q2], hy, PY[q2]);
                }
            }
        }
        if constexpr (esize<T>::v == 4) __builtin_amdgcn_s_barrier();
    }
    if (!active) return;
    // Gamma_x = sum_b wy_b sum_a dwx_a P_ab, Gamma_y = sum_b dwy_b sum_a wx_a P_ab
    // (left at 0 by the axial kernel: stage 1 uses only the z components)
    float wx[4], dwx[4], wy[4], dwy[4];
    float gxx = 0.f, gyx = 0.f, gxy = 0.f, gyy = 0.f;
    if constexpr (!AXIAL) {
        lateral_taps(tw, tdw, 0, 0, wx, dwx);
        lateral_taps(tw, tdw, 0, 1, wy, dwy);
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            float rv = 0.f, rd = 0.f;
#pragma unroll
            for (int a2 = 0; a2 < 4; ++a2) {
                rv = fmaf(wx[a2], PX[b * 4 + a2], rv);
                rd = fmaf(dwx[a2], PX[b * 4 + a2], rd);
            }
            gxx = fmaf(wy[b], rd, gxx);
            gyx = fmaf(dwy[b], rv, gyx);
        }
        lateral_taps(tw, tdw, 1, 0, wx, dwx);
        lateral_taps(tw, tdw, 1, 1, wy, dwy);
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            float rv = 0.f, rd = 0.f;
#pragma unroll
            for (int a2 = 0; a2 < 4; ++a2) {
                rv = fmaf(wx[a2], PY[b * 4 + a2], rv);
                rd = fmaf(dwx[a2], PY[b * 4 + a2], rd);
            }
            gxy = fmaf(wy[b], rd, gxy);
            gyy = fmaf(dwy[b], rv, gyy);
        }
    }
    lam = wave_sum(lam);
    gxx = wave_sum(gxx);
    gyx = wave_sum(gyx);
    gzx = wave_sum(gzx);
    gxy = wave_sum(gxy);
    gyy = wave_sum(gyy);
    gzy = wave_sum(gzy);
    if (lane == 0) {
        float4* o = reinterpret_cast<float4*>(J.part + (size_t)a * 8);
        o[0] = make_float4(lam, gxx, gyx, gzx);
        o[1] = make_float4(gxy, gyy, gzy, 0.f);
        clear_ticket(J.ticket, a);
    }
}

// Two depth samples per lane (16-bit storage).  A step covers outputs o = 122 n + p - sx,
// p = 2 l + e in [sx, 121 + sx] (lane l, e in {0, 1}), sx = parity of the
// X-fast scan's first depth tap.  Pair position p of scan V holds the
// sample base_V + o of output o's first tap, so the depth interpolation of
// output p reads positions p .. p + 3 (this lane and the next one or two, by
// DPP).  Each scan loads even-aligned pairs (q0, q1) = samples (E + 2l,
// E + 2l + 1) with one 32-bit load per column; a
// scan whose positions start one sample after an even boundary (r = 1) uses
// c0 = q1 and c1 = the next lane's q0 (so the taps of every output, up to
// position 125, lie inside the 128 loaded samples).  Samples outside the A-scan take the
// edge value (clamp), applied to the blended columns and, for the adjoint, to
// the weights of q0 and q1.  Every step is self-contained as in k_struct.
constexpr int kOutPerStep2 = 122;

// A pair of 16-bit samples is one 32-bit load.  (Float32 storage keeps one
// sample per lane: 64-bit loads measured slower per byte than 32-bit ones on
// this path, so pairs would not pay.)
template <typename T>
__device__ __forceinline__ void ld2(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff, float& a, float& b);
template <>
__device__ __forceinline__ void ld2<bf16_t>(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff, float& a, float& b)
{
    const uint32_t v = __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0);
    a = __builtin_bit_cast(float, v << 16);
    b = __builtin_bit_cast(float, v & 0xFFFF0000u);
}
template <>
__device__ __forceinline__ void ld2<f16_t>(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff, float& a, float& b)
{
    const uint32_t v = __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0);
    a = (float)__builtin_bit_cast(_Float16, (unsigned short)(v & 0xFFFFu));
    b = (float)__builtin_bit_cast(_Float16, (unsigned short)(v >> 16));
}

template <typename T>
__device__ __forceinline__ void load_pairs(float (&q0)[16], float (&q1)[16], __amdgpu_buffer_rsrc_t rs,
                                           const Stencil& S, int m, int dp)
{
    const int mc = clampi(m, 0, dp - 2);
    const uint32_t voff = (uint32_t)mc * esize<T>::v;
#pragma unroll
    for (int q = 0; q < 16; ++q) ld2<T>(rs, voff, S.off[q], q0[q], q1[q]);
}

template <typename T, bool AXIAL>
__global__ __launch_bounds__(256) void k_struct2(const StructJobs jobs)
{
    if (jobs.skip && *jobs.skip) return;
    if (!AXIAL && struct_sums(jobs)) return;
    const int wv = uni((int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    const int lb = xcd_block((int)blockIdx.x - jobs.sum_blocks, (int)gridDim.x - jobs.sum_blocks);
    int jid = -1;
    for (int q = 0; q < jobs.n; ++q)
        if (lb >= jobs.j[q].blk_begin) jid = q;
    if (jid < 0) return;  // whole block
    const StructJob& J = jobs.j[jid];
    const int w = J.w, h = J.h, d = J.d;
    const int dp = J.dp;  // storage pitch: d, or d + 1 (a padding sample) for an odd depth in 16-bit storage
    // 2 x 2 tiles in 8 bands of tile rows, swept column by column (as k_struct)
    const int tpr = (w + 1) >> 1;
    const int trows = (h + 1) >> 1;
    const int rpb = (trows + 7) >> 3;
    const int t = lb - J.blk_begin;
    const int band = t / (rpb * tpr), tb = t - band * (rpb * tpr);
    const int trow = band * rpb + tb % rpb;
    if (t >= 8 * rpb * tpr || trow >= trows) return;  // whole block
    const int i = 2 * (tb / rpb) + (wv & 1);
    const int j = 2 * trow + (wv >> 1);
    const bool active = i < w && j < h;  // wave-uniform
    const int a = uni(active ? j * w + i : 0);
    const float* dX = J.disp + (size_t)a * 3;
    const float* dY = J.disp + ((size_t)J.na + a) * 3;
    Stencil SX, SY;
    if constexpr (AXIAL) {
        make_stencil_axial<T>(SX, i, j, dX[2], w, dp);
        make_stencil_axial<T>(SY, i, j, dY[2], w, dp);
    } else {
        make_stencil<T>(SX, i, j, dX[0], dX[1], dX[2], w, h, dp);
        make_stencil<T>(SY, i, j, dY[0], dY[1], dY[2], w, h, dp);
    }
    const __amdgpu_buffer_rsrc_t rx =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(J.sx), (short)0, (int)J.vol_bytes, kRsrcWord3);
    const __amdgpu_buffer_rsrc_t ry =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(J.sy), (short)0, (int)J.vol_bytes, kRsrcWord3);
    const float eps = J.eps_h;
    const float inv_eps = 1.0f / J.eps_h;
    // position 0 of step 0 holds sample base_V - sx of scan V
    const int sx = SX.base & 1;
    const int rY = uni((SY.base - sx) & 1);
    const int EX = SX.base - sx, EY = SY.base - sx - rY;  // even

    float x0[16], x1[16], y0[16], y1[16];
    float PX[16], PY[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) PX[q] = PY[q] = 0.f;
    float lam = 0.f, gzx = 0.f, gzy = 0.f;
    const int nsteps = (d + kOutPerStep2 - 1) / kOutPerStep2;
    for (int n = 0; n < nsteps; ++n) {
        if (active) {
            const int mX = EX + kOutPerStep2 * n + 2 * lane;
            const int mY = EY + kOutPerStep2 * n + 2 * lane;
            float bx0, bx1, by0, by1;
            if constexpr (AXIAL) {
                ld2<T>(rx, (uint32_t)clampi(mX, 0, dp - 2) * esize<T>::v, SX.off[kCentre], bx0, bx1);
                ld2<T>(ry, (uint32_t)clampi(mY, 0, dp - 2) * esize<T>::v, SY.off[kCentre], by0, by1);
            } else {
                load_pairs<T>(x0, x1, rx, SX, mX, dp);
                load_pairs<T>(y0, y1, ry, SY, mY, dp);
                bx0 = blend(x0, SX);
                bx1 = blend(x1, SX);
                by0 = blend(y0, SY);
                by1 = blend(y1, SY);
            }
            // clamp: a pair below the A-scan holds sample 0 twice, one above it sample d - 1 twice
            // (with an odd depth the last stored pair is sample d - 1 and its padding copy)
            const bool loX = mX < 0, hiX = mX > dp - 2, loY = mY < 0, hiY = mY > dp - 2;
            const float cx0 = hiX ? bx1 : bx0, cx1 = loX ? bx0 : bx1;
            const float ty0 = hiY ? by1 : by0, ty1 = loY ? by0 : by1;
            // Y positions start one sample after the pair boundary when rY = 1
            const float ty0n = shl1(ty0);
            const float cy0 = rY ? ty1 : ty0, cy1 = rY ? ty0n : ty1;
            // depth interpolation (Eq. 2) of outputs at positions 2l and 2l + 1
            const float cx0n = shl1(cx0), cx1n = shl1(cx1), cx0nn = shl1(cx0n);
            const float cy0n = shl1(cy0), cy1n = shl1(cy1), cy0nn = shl1(cy0n);
            const float ix0 = SX.wz[0] * cx0 + SX.wz[1] * cx1 + SX.wz[2] * cx0n + SX.wz[3] * cx1n;
            const float ix1 = SX.wz[0] * cx1 + SX.wz[1] * cx0n + SX.wz[2] * cx1n + SX.wz[3] * cx0nn;
            const float zx0 = SX.dwz[0] * cx0 + SX.dwz[1] * cx1 + SX.dwz[2] * cx0n + SX.dwz[3] * cx1n;
            const float zx1 = SX.dwz[0] * cx1 + SX.dwz[1] * cx0n + SX.dwz[2] * cx1n + SX.dwz[3] * cx0nn;
            const float iy0 = SY.wz[0] * cy0 + SY.wz[1] * cy1 + SY.wz[2] * cy0n + SY.wz[3] * cy1n;
            const float iy1 = SY.wz[0] * cy1 + SY.wz[1] * cy0n + SY.wz[2] * cy1n + SY.wz[3] * cy0nn;
            const float zy0 = SY.dwz[0] * cy0 + SY.dwz[1] * cy1 + SY.dwz[2] * cy0n + SY.dwz[3] * cy1n;
            const float zy1 = SY.dwz[0] * cy1 + SY.dwz[1] * cy0n + SY.dwz[2] * cy1n + SY.dwz[3] * cy0nn;
            // residual and pseudo-Huber loss (Eq. 4), eps u^2 / (sqrt(1 + u^2) + 1), and u / sqrt(1 + u^2)
            const int p0 = 2 * lane;
            const int o0 = kOutPerStep2 * n + p0 - sx;
            const bool v0 = p0 >= sx && p0 <= 121 + sx && o0 < d;
            const bool v1 = p0 + 1 <= 121 + sx && o0 + 1 < d;
            float L0, G0, L1, G1;
            {
                const float u = (ix0 - iy0) * inv_eps, q = u * u;
                const float rs = __builtin_amdgcn_rsqf(1.f + q), sq = (1.f + q) * rs;
                L0 = v0 ? eps * q * __builtin_amdgcn_rcpf(sq + 1.f) : 0.f;
                G0 = v0 ? u * rs : 0.f;
            }
            {
                const float u = (ix1 - iy1) * inv_eps, q = u * u;
                const float rs = __builtin_amdgcn_rsqf(1.f + q), sq = (1.f + q) * rs;
                L1 = v1 ? eps * q * __builtin_amdgcn_rcpf(sq + 1.f) : 0.f;
                G1 = v1 ? u * rs : 0.f;
            }
            lam += L0 + L1;
            gzx += G0 * zx0 + G1 * zx1;
            gzy += G0 * zy0 + G1 * zy1;
            if constexpr (!AXIAL) {
                // adjoint of the depth interpolation: position q collects the
                // derivatives of the outputs at q, q - 1, q - 2, q - 3
                const float G0p = shr1(G0), G1p = shr1(G1), G1pp = shr1(G1p);
                const float hx0 = SX.wz[0] * G0 + SX.wz[1] * G1p + SX.wz[2] * G0p + SX.wz[3] * G1pp;
                const float hx1 = SX.wz[0] * G1 + SX.wz[1] * G0 + SX.wz[2] * G1p + SX.wz[3] * G0p;
                const float hy0 = SY.wz[0] * G0 + SY.wz[1] * G1p + SY.wz[2] * G0p + SY.wz[3] * G1pp;
                const float hy1 = SY.wz[0] * G1 + SY.wz[1] * G0 + SY.wz[2] * G1p + SY.wz[3] * G0p;
                // back to the loaded samples q0, q1: alignment shift, then clamp
                const float hy1p = shr1(hy1);
                const float uy0 = rY ? hy1p : hy0, uy1 = rY ? hy0 : hy1;
                const float wx0 = loX ? hx0 + hx1 : (hiX ? 0.f : hx0);
                const float wx1 = hiX ? hx0 + hx1 : (loX ? 0.f : hx1);
                const float wy0 = loY ? uy0 + uy1 : (hiY ? 0.f : uy0);
                const float wy1 = hiY ? uy0 + uy1 : (loY ? 0.f : uy1);
#pragma unroll
                for (int q2 = 0; q2 < 16; ++q2) {
                    PX[q2] = fmaf(x0[q2], wx0, fmaf(x1[q2], wx1, PX[q2]));
                    PY[q2] = fmaf(y0[q2], wy0, fmaf(y1[q2], wy1, PY[q2]));
                }
            }
        }
    }
    if (!active) return;
    float wx[4], dwx[4], wy[4], dwy[4];
    float gxx = 0.f, gyx = 0.f, gxy = 0.f, gyy = 0.f;
    if constexpr (!AXIAL) {
        cr_taps(SX.tx, wx, dwx);
        cr_taps(SX.ty, wy, dwy);
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            float rv = 0.f, rd = 0.f;
#pragma unroll
            for (int a2 = 0; a2 < 4; ++a2) {
                rv = fmaf(wx[a2], PX[b * 4 + a2], rv);
                rd = fmaf(dwx[a2], PX[b * 4 + a2], rd);
            }
            gxx = fmaf(wy[b], rd, gxx);
            gyx = fmaf(dwy[b], rv, gyx);
        }
        cr_taps(SY.tx, wx, dwx);
        cr_taps(SY.ty, wy, dwy);
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            float rv = 0.f, rd = 0.f;
#pragma unroll
            for (int a2 = 0; a2 < 4; ++a2) {
                rv = fmaf(wx[a2], PY[b * 4 + a2], rv);
                rd = fmaf(dwx[a2], PY[b * 4 + a2], rd);
            }
            gxy = fmaf(wy[b], rd, gxy);
            gyy = fmaf(dwy[b], rv, gyy);
        }
    }
    lam = wave_sum(lam);
    gxx = wave_sum(gxx);
    gyx = wave_sum(gyx);
    gzx = wave_sum(gzx);
    gxy = wave_sum(gxy);
    gyy = wave_sum(gyy);
    gzy = wave_sum(gzy);
    if (lane == 0) {
        float4* o = reinterpret_cast<float4*>(J.part + (size_t)a * 8);
        o[0] = make_float4(lam, gxx, gyx, gzx);
        o[1] = make_float4(gxy, gyy, gzy, 0.f);
        clear_ticket(J.ticket, a);
    }
}

// ---------------------------------------------------------------------------
// k_struct_mx: the structural data term on the matrix cores.
//
// One wave evaluates a 2 x 2 tile of output A-scans (tile_blend.h).  Lane 16 g +
// n holds the lateral blends (value, x and y derivative) of A-scan g at L
// consecutive source depths, and everything along depth (interpolation of Eq. 2,
// residual, loss of Eq. 4, its adjoint) runs on the vector units in that layout,
// the neighbouring depths coming from the next lane of the row (DPP).

// The seven sums of an A-scan, one part of them per lane of its row.
struct MxSums {
    float lam = 0.f, gxx = 0.f, gyx = 0.f, gzx = 0.f, gxy = 0.f, gyy = 0.f, gzy = 0.f;
    __device__ __forceinline__ void reduce()  // to the row's last lane
    {
        lam = row_sum_last(lam);
        gxx = row_sum_last(gxx);
        gyx = row_sum_last(gyx);
        gzx = row_sum_last(gzx);
        gxy = row_sum_last(gxy);
        gyy = row_sum_last(gyy);
        gzy = row_sum_last(gzy);
    }
    __device__ __forceinline__ bool finite() const
    {
        return __builtin_isfinite(((lam + gxx) + (gyx + gzx)) + ((gxy + gyy) + gzy));
    }
    __device__ __forceinline__ void store(float* p) const
    {
        float4* o = reinterpret_cast<float4*>(p);
        o[0] = make_float4(lam, gxx, gyx, gzx);
        o[1] = make_float4(gxy, gyy, gzy, 0.f);
    }
};

// The depth work of one step on the lateral blends of both scans (value x, y
// with three positions of the next lane; x and y derivatives xx, xy, yx, yy).
// ie_lo, ie_hi: 1 / eps for the first two positions and the others, or 0.
// ends (wave-uniform): only those of the outputs o0 + i that are 0 .. d - 1 count.
template <int L>
__device__ __forceinline__ void mx_depth(MxSums& A, const float (&x)[L + 3], const float (&xx)[L], const float (&xy)[L],
                                         const float (&y)[L + 3], const float (&yx)[L], const float (&yy)[L],
                                         const float (&wx)[4], const float (&dwx)[4], const float (&wy)[4],
                                         const float (&dwy)[4], float ie_lo, float ie_hi, bool ends, int o0,
                                         int d)
{
    // depth interpolation (Eq. 2) and residual over eps
    float u[L];
#pragma unroll
    for (int i = 0; i < L; ++i) u[i] = (mx_fir(wx, x, i) - mx_fir(wy, y, i)) * (i < 2 ? ie_lo : ie_hi);
    if (ends) {
#pragma unroll
        for (int i = 0; i < L; ++i) u[i] = (unsigned)(o0 + i) < (unsigned)d ? u[i] : 0.f;
    }
    // pseudo-Huber loss (Eq. 4) eps u^2 / (sqrt(1 + u^2) + 1) and its derivative u / sqrt(1 + u^2)
    float G[L + 3];  // G[3 + i]: this lane's position i; G[0 .. 2]: the lane before
#pragma unroll
    for (int i = 0; i < L; ++i) {
        const float q = u[i] * u[i];
        const float rs = __builtin_amdgcn_rsqf(1.f + q), sq = (1.f + q) * rs;
        A.lam = fmaf(q, __builtin_amdgcn_rcpf(sq + 1.f), A.lam);
        G[3 + i] = u[i] * rs;
        A.gzx = fmaf(G[3 + i], mx_fir(dwx, x, i), A.gzx);
        A.gzy = fmaf(G[3 + i], mx_fir(dwy, y, i), A.gzy);
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) G[i] = row_prev(G[L + i]);
    // adjoint of the depth interpolation: position p collects the outputs p - 3 .. p
#pragma unroll
    for (int i = 0; i < L; ++i) {
        float hx = wx[0] * G[3 + i], hy = wy[0] * G[3 + i];
#pragma unroll
        for (int c = 1; c < 4; ++c) {
            hx = fmaf(wx[c], G[3 + i - c], hx);
            hy = fmaf(wy[c], G[3 + i - c], hy);
        }
        A.gxx = fmaf(hx, xx[i], A.gxx);
        A.gyx = fmaf(hx, xy[i], A.gyx);
        A.gxy = fmaf(hy, yx[i], A.gxy);
        A.gyy = fmaf(hy, yy[i], A.gyy);
    }
}

// Bound by vector issue: a step of eight depths per lane takes some 440 vector
// and 48 matrix instructions (16 cycles each, partly overlapped), of which the
// depth work is 46 per sample pair and the operand packing 8.  Three waves per
// SIMD: 168 registers; two waves with the next step's samples loaded ahead
// measured 25 % slower, and so did one workgroup barrier per step to share L1
// lines; the column offsets are read from the LDS at each step, which saves
// 16 registers and with them the spills.  The lateral blends and their adjoint took k_struct2 128 FMAs and 64
// conversions per 122 outputs of one A-scan, and its 64 loads of 256 bytes per
// step of a tile are 16 of 1 KB here.  500 x 500 x 800 in BF16: 1.058 -> 0.563
// ms (68 TFLOP/s of the method's operations), 500 x 500 x 465 in FP16: 0.645 ->
// 0.367, 300 x 300 x 233 in BF16 0.160 -> 0.092 ms.
// float32 (four depths a lane): bound by its matrix products, 56 to 64 of 32 cycles
// a step, and some 290 vector instructions, which do not overlap; four waves per
// SIMD.  500 x 500 x 800 1.60 -> 1.19 ms (32 TFLOP/s), 300 x 300 x 640 0.464 -> 0.418
// (with the fours of slots without a column multiplied too 0.434).
template <typename T, int L>
__global__ __launch_bounds__(256, 3) void k_struct_mx(const StructJobs jobs)
{
    if (jobs.skip && *jobs.skip) return;
    if (struct_sums(jobs)) return;
    constexpr int kEs = (int)esize<T>::v;
    __shared__ MxLds<kEs, 2, L> lds[4];
    const int wv = uni((int)(threadIdx.x >> 6));
    MxLds<kEs, 2, L>& M = lds[wv];
    const int lb = xcd_block((int)blockIdx.x - jobs.sum_blocks, (int)gridDim.x - jobs.sum_blocks);
    int jid = -1;
    for (int q = 0; q < jobs.n; ++q)
        if (lb >= jobs.j[q].blk_begin) jid = q;
    if (jid < 0) return;  // whole block
    const StructJob& J = jobs.j[jid];
    const int w = J.w, h = J.h, d = J.d, dp = J.dp;
    int i0, j0;
    if (!mx_tile(w, h, lb - J.blk_begin, wv, i0, j0)) return;
    const __amdgpu_buffer_rsrc_t rx =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(J.sx), (short)0, (int)J.vol_bytes, kRsrcWord3);
    const __amdgpu_buffer_rsrc_t ry =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(J.sy), (short)0, (int)J.vol_bytes, kRsrcWord3);
    typedef MxGeo<kEs, L> Geo;
    const float eps = J.eps_h;
    const float inv_eps = 1.0f / J.eps_h;
    // The groups of the tile evaluated together: all four; two where the four
    // need too many slots; one at a time where a sample is not finite, since
    // it reaches every A-scan of the tile through the weights 0.
    int groups = 15;
    for (;;) {
        // opaque to the compiler, which otherwise keeps the set-up's addresses
        // for a second round in registers it does not have
        int lane = threadIdx.x & 63;
        asm volatile("" : "+v"(lane));
        const int g = lane >> 4;
        const bool last = (lane & 15) == 15;
        const int p0 = L * (lane & 15);  // this lane's first position
        // an A-scan outside the scan repeats its neighbour and is not written
        const int2 pg = make_int2(min(i0 + (g & 1), w - 1), min(j0 + (g >> 1), h - 1));
        const bool inscan = i0 + (g & 1) < w && j0 + (g >> 1) < h;
        const int ag = pg.y * w + pg.x;
        // 1 / eps for this lane's first two positions and the others, 0 where they
        // are no outputs: no residual, loss or derivative there
        static_assert(Geo::kOut % L == 0 || Geo::kOut % L == 2, "two classes of positions");
        const float ie_lo = p0 < Geo::kOut ? inv_eps : 0.f, ie_hi = p0 + 2 < Geo::kOut ? inv_eps : 0.f;
        MxScan SX, SY;
        int nrest = 0;
        if (!mx_setup<T, 3>(SX, M, 0, J.disp, ag, pg, 0, w, h, dp, lane, groups, nrest) ||
            !mx_setup<T, 3>(SY, M, 1, J.disp + (size_t)J.na * 3, ag, pg, SX.sh, w, h, dp, lane, groups, nrest)) {
            groups = 3;  // two groups never need more than 32 slots
            continue;
        }
        MxSums A;
        const int nsteps = (d + SX.any + Geo::kOut - 1) / Geo::kOut;  // the last output's position: at most d - 1 + any
        for (int s = 0; s < nsteps; ++s) {
            float x[L + 3], xx[L], xy[L], y[L + 3], yx[L], yy[L];
            {
                typename MxDwords<Geo::kDw>::type qx[8], qy[8];
                mx_load(qx, SX, M, 0, rx, s, dp, lane);
                mx_load(qy, SY, M, 1, ry, s, dp, lane);
                float v[3][L];
                f32x4 D[L] = {};
                mx_blend<T>(D, qx, M, 0, lane, SX.ns);
                if (SX.ns > 32) mx_rest<T>(D, SX, M, 0, rx, s, dp, lane);
                mx_rows<false>(v, D, SX, M, s, dp, lane);
#pragma unroll
                for (int i = 0; i < L; ++i) {
                    x[i] = v[0][i];
                    xx[i] = v[1][i];
                    xy[i] = v[2][i];
                }
                f32x4 E[L] = {};
                mx_blend<T>(E, qy, M, 1, lane, SY.ns);
                if (SY.ns > 32) mx_rest<T>(E, SY, M, 1, ry, s, dp, lane);
                mx_rows<true>(v, E, SY, M, s, dp, lane);
#pragma unroll
                for (int i = 0; i < L; ++i) {
                    y[i] = v[0][i];
                    yx[i] = v[1][i];
                    yy[i] = v[2][i];
                }
            }
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                x[L + i] = row_next(x[i]);
                y[L + i] = row_next(y[i]);
            }
            mx_depth<L>(A, x, xx, xy, y, yx, yy, SX.wz, SX.dwz, SY.wz, SY.dwz, ie_lo, ie_hi,
                        s == 0 || Geo::kOut * (s + 1) > d, Geo::kOut * s + p0 - SX.sh, d);
        }
        A.lam *= eps;
        A.reduce();
        const bool active = groups >> g & 1;
        if (last && inscan && active) A.store(J.part + (size_t)ag * 8);
        const bool bad = __ballot(last && active && !A.finite()) != 0;
        groups = mx_next(groups, bad);
        if (!groups) return;
    }
}

// ---------------------------------------------------------------------------
// deterministic block reduction helpers

// Fixed-order sum of the rows of block partials (strided per thread, then a
// fixed tree); every thread of the block receives the result, and every block
// that sums the same rows gets the same bits.
template <int N>
__device__ __forceinline__ void sum_rows(const double* blk, int nblk, double (&out)[N])
{
    __shared__ double sh[kRedBlock / 64][N];
    double acc[N];
#pragma unroll
    for (int q = 0; q < N; ++q) acc[q] = 0.0;
    for (int r = threadIdx.x; r < nblk; r += kRedBlock) {
#pragma unroll
        for (int q = 0; q < N; ++q) acc[q] += blk[(size_t)r * N + q];
    }
    store_wave_sums<N>(acc, sh);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < N; ++q) out[q] = wave_rows<N>(sh, q);
}

// ---------------------------------------------------------------------------

__global__ __launch_bounds__(kRedBlock) void k_sum(const SumJobs jobs)
{
    if (jobs.skip && *jobs.skip) return;
    int jid = 0;
    for (int q = 1; q < jobs.n; ++q)
        if ((int)blockIdx.x >= jobs.j[q].blk_begin) jid = q;
    const SumJob& J = jobs.j[jid];
    sum_block(J.disp[0], J.disp[1], J.na, J.nblk, blockIdx.x - J.blk_begin, J.blk);
}

// pseudo-Huber in float64 (regulariser and en face terms); ieps = 1 / eps
__device__ __forceinline__ void huber_d(double x, double eps, double ieps, double& L, double& dL)
{
    const double u = x * ieps;
    const double s = sqrt(1.0 + u * u);
    L = eps * u * u / (s + 1.0);
    dL = u / s;
}

// 2-D / 1-D Catmull-Rom samples (value and derivatives) in float32
__device__ __forceinline__ void sample2(const float* img, int w, int h, int i, int j, float dx, float dy,
                                        float out[3])
{
    int nx, ny;
    float tx, ty;
    split(i, dx, nx, tx);
    split(j, dy, ny, ty);
    float wx[4], dwx[4], wy[4], dwy[4];
    cr_taps(tx, wx, dwx);
    cr_taps(ty, wy, dwy);
    float v = 0.f, gx = 0.f, gy = 0.f;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const float* row = img + (size_t)clampi(ny - 1 + b, 0, h - 1) * w;
        float rv = 0.f, rd = 0.f;
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            const float s = row[clampi(nx - 1 + a, 0, w - 1)];
            rv = fmaf(wx[a], s, rv);
            rd = fmaf(dwx[a], s, rd);
        }
        v = fmaf(wy[b], rv, v);
        gx = fmaf(wy[b], rd, gx);
        gy = fmaf(dwy[b], rv, gy);
    }
    out[0] = v;
    out[1] = gx;
    out[2] = gy;
}

__device__ __forceinline__ void sample1(const float* vec, int n, int i, float dv, float out[2])
{
    int nx;
    float t;
    split(i, dv, nx, t);
    float w[4], dw[4];
    cr_taps(t, w, dw);
    float v = 0.f, g = 0.f;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        const float s = vec[clampi(nx - 1 + a, 0, n - 1)];
        v = fmaf(w[a], s, v);
        g = fmaf(dw[a], s, g);
    }
    out[0] = v;
    out[1] = g;
}

// Neighbours of output A-scan (i, j) in scan V's acquisition order (X-fast:
// along rows, then to the next row; Y-fast: along columns).  Returns the
// A-scan index or -1, and the link weight (1 inside a B-scan, wfb across the
// flyback between B-scans).
__device__ __forceinline__ int prev_ascan(int V, int i, int j, int w, int h, double wfb, double& om)
{
    if (V == 0) {
        if (i > 0) { om = 1.0; return j * w + i - 1; }
        if (j > 0) { om = wfb; return (j - 1) * w + (w - 1); }
    } else {
        if (j > 0) { om = 1.0; return (j - 1) * w + i; }
        if (i > 0) { om = wfb; return (h - 1) * w + (i - 1); }
    }
    om = 0.0;
    return -1;
}
__device__ __forceinline__ int next_ascan(int V, int i, int j, int w, int h, double wfb, double& om)
{
    if (V == 0) {
        if (i < w - 1) { om = 1.0; return j * w + i + 1; }
        if (j < h - 1) { om = wfb; return (j + 1) * w; }
    } else {
        if (j < h - 1) { om = 1.0; return (j + 1) * w + i; }
        if (i < w - 1) { om = wfb; return i + 1; }
    }
    om = 0.0;
    return -1;
}

__global__ __launch_bounds__(kRedBlock) void k_combine(const CombineJobs jobs)
{
    if (jobs.skip && *jobs.skip) return;
    int jid = 0;
    for (int q = 1; q < jobs.n; ++q)
        if ((int)blockIdx.x >= jobs.j[q].blk_begin) jid = q;
    const CombineJob& J = jobs.j[jid];
    const int b = blockIdx.x - J.blk_begin;
    const int a = b * kRedBlock + threadIdx.x;
    // sum of all displacements (mean term), from the partials of k_sum
    double sumd[4] = {0, 0, 0, 0};
    if (J.mode == 1) sum_rows<4>(J.sum_blk, J.nsum, sumd);  // block-uniform
    // partial sums: data, str, ang, reg, (unused), str05, ang05, g.p
    double v[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (a < J.na) {
        const int w = J.w, h = J.h, na = J.na;
        const double dd = (double)J.d;
        const int i = a % w, j = a / w;
        const float4 p0 = reinterpret_cast<const float4*>(J.part)[(size_t)a * 2];
        const float4 p1 = reinterpret_cast<const float4*>(J.part)[(size_t)a * 2 + 1];
        const double lam = p0.x;
        const float* dX = J.disp[0] + (size_t)a * 3;
        const float* dY = J.disp[1] + (size_t)a * 3;
        float jx[3], jy[3];
        sample2(J.ax, w, h, i, j, dX[0], dX[1], jx);
        sample2(J.ay, w, h, i, j, dY[0], dY[1], jy);
        double LA, GA;
        huber_d((double)jx[0] - (double)jy[0], J.eps_h, J.ieps_h, LA, GA);
        // validity (Eq. 5) varies along each scan's slow axis: y for an X-fast
        // scan (index j, component dy), x for a Y-fast scan
        const int oX = J.orient & 1, oY = (J.orient >> 1) & 1;
        float rx[2], ry[2];
        if (oX == 0) sample1(J.vx, h, j, dX[1], rx);
        else sample1(J.vx, w, i, dX[0], rx);
        if (oY == 1) sample1(J.vy, w, i, dY[0], ry);
        else sample1(J.vy, h, j, dY[1], ry);
        const double tvx = rx[0] <= 0.f ? 0.0 : (rx[0] >= 1.f ? 1.0 : (double)rx[0]);
        const double dtvx = (rx[0] > 0.f && rx[0] < 1.f) ? (double)rx[1] : 0.0;
        const double tvy = ry[0] <= 0.f ? 0.0 : (ry[0] >= 1.f ? 1.0 : (double)ry[0]);
        const double dtvy = (ry[0] > 0.f && ry[0] < 1.f) ? (double)ry[1] : 0.0;
        v[5] = (1.0 - 0.5 * tvx * tvy) * lam;
        v[6] = 0.5 * tvx * tvy * dd * LA;
        if (J.mode == 1) {
            const double eta = *J.eta;
            const double delta = J.delta0 * tvx * tvy;  // Eq. 8
            const double ws = eta * (1.0 - delta);       // structural weight (Eqs. 6, 9)
            const double wa = dd / eta * delta;          // angiographic weight (Eqs. 7, 9)
            v[1] = (1.0 - delta) * lam;
            v[2] = delta * dd * LA;
            v[0] = eta * v[1] + v[2] / eta;
            const double dpd = -eta * lam + dd / eta * LA;  // d(data)/d(delta)
            double g[6];
            g[0] = ws * p0.y + wa * GA * jx[1];
            g[1] = ws * p0.z + wa * GA * jx[2];
            g[2] = ws * p0.w;
            g[3] = -(ws * p1.x + wa * GA * jy[1]);
            g[4] = -(ws * p1.y + wa * GA * jy[2]);
            g[5] = -(ws * p1.z);
            g[oX == 0 ? 1 : 0] += dpd * J.delta0 * tvy * dtvx;
            g[oY == 1 ? 3 : 4] += dpd * J.delta0 * tvx * dtvy;
            // scan-order regulariser (gather form: this A-scan's two links)
            double reg = 0.0;
            for (int V = 0; V < 2; ++V) {
                const float* DV = J.disp[V];
                const float* da = DV + (size_t)a * 3;
                const int oV = V == 0 ? oX : oY;  // acquisition order of the slot's scan
                double omp, omn;
                const int pa = prev_ascan(oV, i, j, w, h, J.wfb, omp);
                const int nb = next_ascan(oV, i, j, w, h, J.wfb, omn);
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    double Lr, dLr;
                    if (pa >= 0) {
                        huber_d((double)da[c] - (double)DV[(size_t)pa * 3 + c], J.eps_r, J.ieps_r, Lr, dLr);
                        g[V * 3 + c] += J.alpha * dd * omp * dLr;
                    }
                    if (nb >= 0) {
                        huber_d((double)DV[(size_t)nb * 3 + c] - (double)da[c], J.eps_r, J.ieps_r, Lr, dLr);
                        g[V * 3 + c] -= J.alpha * dd * omn * dLr;
                        reg += dd * omn * Lr;
                    }
                }
            }
            v[3] = reg;
            // mean-displacement term: dM/dd_c = gamma d sum_c / N_A
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const double gm = J.gamma * dd * sumd[c] / (double)na;
                g[c] += gm;
                g[3 + c] += gm;
            }
            if (J.grad) {
                float* gX = J.grad + (size_t)a * 3;
                float* gY = J.grad + ((size_t)na + a) * 3;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    gX[c] = (float)g[c];
                    gY[c] = (float)g[3 + c];
                }
            }
            if (J.grad64) {
                double* gX = J.grad64 + (size_t)a * 3;
                double* gY = J.grad64 + ((size_t)na + a) * 3;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    gX[c] = g[c];
                    gY[c] = g[3 + c];
                }
            }
            if (J.p) {  // directional derivative g . p (line search)
                const double* pX = J.p + (size_t)a * 3;
                const double* pY = J.p + ((size_t)na + a) * 3;
                double gp = 0.0;
#pragma unroll
                for (int c = 0; c < 3; ++c) gp += g[c] * pX[c] + g[3 + c] * pY[c];
                v[7] = gp;
            }
        }
    }
    block_reduce_store<8>(v, J.blk + (size_t)b * 8);
}

// Final sums of one evaluation from the rows of its blocks: the objective terms
// (mode 1) or the level's eta (mode 0, Eq. 10).
__device__ __forceinline__ void finalize(const CombineJob& J, const double (&sumd)[4])
{
    double s[8];
    sum_rows<8>(J.blk, J.nblk, s);
    if (threadIdx.x != 0) return;
    if (J.mode == 0) {
        // eta = 1 where a term vanishes (identical inputs)
        *J.eta = (s[5] > 1e-300 && s[6] > 1e-300) ? sqrt(s[6] / s[5]) : 1.0;
        return;
    }
    const double eta = *J.eta;
    double m = 0.0;
    for (int c = 0; c < 3; ++c) m += sumd[c] * sumd[c];
    m *= J.gamma * (double)J.d / (2.0 * (double)J.na);
    double* t = J.terms;
    t[OCTMC_TERM_DATA] = s[0];
    t[OCTMC_TERM_STR] = s[1];
    t[OCTMC_TERM_ANG] = s[2];
    t[OCTMC_TERM_REG] = s[3];
    t[OCTMC_TERM_MEAN] = m;
    t[OCTMC_TERM_STR05] = s[5];
    t[OCTMC_TERM_ANG05] = s[6];
    t[OCTMC_TERM_ETA] = eta;
    t[OCTMC_TERM_GP] = s[7];
    t[OCTMC_TERM_F] = s[0] + J.alpha * s[3] + m;
}

// One block per job, after k_combine.
__global__ __launch_bounds__(kRedBlock) void k_finalize(const CombineJobs jobs)
{
    if (jobs.skip && *jobs.skip) return;
    const CombineJob& J = jobs.j[blockIdx.x];
    double sumd[4] = {0, 0, 0, 0};
    if (J.mode == 1) sum_rows<4>(J.sum_blk, J.nsum, sumd);
    finalize(J, sumd);
}

// sample2 by four lanes, lane b of them taking source row b (the same operations
// in the same order); `first` is the first of the four.
__device__ __forceinline__ void sample2_rows(const float* img, int w, int h, int i, int j, float dx, float dy, int b,
                                        int first, float out[3])
{
    int nx, ny;
    float tx, ty;
    split(i, dx, nx, tx);
    split(j, dy, ny, ty);
    float wx[4], dwx[4], wy[4], dwy[4];
    cr_taps(tx, wx, dwx);
    cr_taps(ty, wy, dwy);
    const float* row = img + (size_t)clampi(ny - 1 + b, 0, h - 1) * w;
    float rv = 0.f, rd = 0.f;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        const float s = row[clampi(nx - 1 + a, 0, w - 1)];
        rv = fmaf(wx[a], s, rv);
        rd = fmaf(dwx[a], s, rd);
    }
    float v = 0.f, gx = 0.f, gy = 0.f;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float qv = __shfl(rv, first + q), qd = __shfl(rd, first + q);
        v = fmaf(wy[q], qv, v);
        gx = fmaf(wy[q], qd, gx);
        gy = fmaf(dwy[q], qv, gy);
    }
    out[0] = v;
    out[1] = gx;
    out[2] = gy;
}

// Sum of the displacements of both slots by every block for itself (few
// A-scans): sixteen-byte loads of four A-scans' twelve floats, four of them in
// flight.
__device__ __forceinline__ void own_sums(const CombineJob& J, double (&v)[4])
{
    typedef float quad_t __attribute__((ext_vector_type(4), aligned(4)));
    const int quads = J.na / 4;
#pragma unroll
    for (int V = 0; V < 2; ++V) {
        const float* __restrict__ D = J.disp[V];
#pragma unroll 4
        for (int q = threadIdx.x; q < quads; q += kRedBlock) {
            const quad_t* p = reinterpret_cast<const quad_t*>(D + (size_t)q * 12);
            const quad_t x = p[0], y = p[1], z = p[2];
            v[0] += ((double)x[0] + (double)x[3]) + ((double)y[2] + (double)z[1]);
            v[1] += ((double)x[1] + (double)y[0]) + ((double)y[3] + (double)z[2]);
            v[2] += ((double)x[2] + (double)y[1]) + ((double)z[0] + (double)z[3]);
        }
        const int a = 4 * quads + threadIdx.x;
        if (a < J.na) {
#pragma unroll
            for (int c = 0; c < 3; ++c) v[c] += (double)D[(size_t)a * 3 + c];
        }
    }
}

// k_combine for few A-scans, which are latency: eight lanes take an A-scan, and
// the launches before and after it go into it.  Lanes 0 - 3 sample the first
// scan's en face image and lanes 4 - 7 the second's, a source row each; every lane
// forms the terms that all components share; lanes 0 - 5 form one component of the
// gradient each, with its two links of the regulariser.  Every block sums the
// displacements for itself and the last one done forms the final sums.  64 x 64
// x 128 float32: displacement sum, combination and final sums 18.5 us in three
// launches, 10.6 in one (the block's count with its release and acquire 1.6 of
// them, and 12 with 1000 blocks, which is why many A-scans keep a launch for the
// final sums).
__global__ __launch_bounds__(kRedBlock) void k_combine_few(const CombineJobs jobs)
{
    __shared__ double shd[kRedBlock / 64][4];
    __shared__ int last;
    if (jobs.skip && *jobs.skip) return;
    int jid = 0;
    for (int q = 1; q < jobs.n; ++q)
        if ((int)blockIdx.x >= jobs.j[q].blk_begin) jid = q;
    const CombineJob& J = jobs.j[jid];
    const int b = blockIdx.x - J.blk_begin;
    const int lane = threadIdx.x & 63, r = lane & 7, V = r >> 2;
    const int w = J.w, h = J.h, na = J.na;
    const double dd = (double)J.d;
    const int oX = J.orient & 1, oY = (J.orient >> 1) & 1, oV = V == 0 ? oX : oY;
    // this lane's component of the gradient: slot S, component c (lanes 6 and 7 none)
    const int S = r >= 3, c = r - 3 * S, oS = S == 0 ? oX : oY;
    const int mine = b * kFewAscans + (int)(threadIdx.x >> 3);
    const bool live = mine < na;
    const int a = live ? mine : na - 1;  // all lanes of a wave exchange: idle ones repeat the last A-scan
    const int i = a % w, j = a / w;
    // sum of all displacements (mean term)
    double sumd[4] = {0, 0, 0, 0};
    if (J.mode == 1) {  // block-uniform
        double own[4] = {0, 0, 0, 0};
        own_sums(J, own);
        store_wave_sums<4>(own, shd);
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 3; ++q) sumd[q] = wave_rows<4>(shd, q);
    }
    const float4 p0 = reinterpret_cast<const float4*>(J.part)[(size_t)a * 2];
    const float4 p1 = reinterpret_cast<const float4*>(J.part)[(size_t)a * 2 + 1];
    const double lam = p0.x;
    const float* dV = J.disp[V] + (size_t)a * 3;
    float mv[3], ov[3];  // en face sample of this lane's scan and of the other
    sample2_rows(V == 0 ? J.ax : J.ay, w, h, i, j, dV[0], dV[1], r & 3, lane & ~3, mv);
#pragma unroll
    for (int q = 0; q < 3; ++q) ov[q] = __shfl_xor(mv[q], 4);
    double LA, GA;
    huber_d(V == 0 ? (double)mv[0] - (double)ov[0] : (double)ov[0] - (double)mv[0], J.eps_h, J.ieps_h, LA, GA);
    // validity (Eq. 5), as in k_combine
    float rv[2];
    sample1(V == 0 ? J.vx : J.vy, oV == 0 ? h : w, oV == 0 ? j : i, oV == 0 ? dV[1] : dV[0], rv);
    const float ro[2] = {__shfl_xor(rv[0], 4), __shfl_xor(rv[1], 4)};
    const float rx0 = V == 0 ? rv[0] : ro[0], ry0 = V == 0 ? ro[0] : rv[0];
    const float rx1 = V == 0 ? rv[1] : ro[1], ry1 = V == 0 ? ro[1] : rv[1];
    const double tvx = rx0 <= 0.f ? 0.0 : (rx0 >= 1.f ? 1.0 : (double)rx0);
    const double dtvx = (rx0 > 0.f && rx0 < 1.f) ? (double)rx1 : 0.0;
    const double tvy = ry0 <= 0.f ? 0.0 : (ry0 >= 1.f ? 1.0 : (double)ry0);
    const double dtvy = (ry0 > 0.f && ry0 < 1.f) ? (double)ry1 : 0.0;
    // partial sums: data, str, ang, reg, (unused), str05, ang05, g.p
    double v[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (live && r == 0) {
        v[5] = (1.0 - 0.5 * tvx * tvy) * lam;
        v[6] = 0.5 * tvx * tvy * dd * LA;
    }
    if (J.mode == 1) {
        const double eta = *J.eta;
        const double delta = J.delta0 * tvx * tvy;  // Eq. 8
        const double ws = eta * (1.0 - delta);       // structural weight (Eqs. 6, 9)
        const double wa = dd / eta * delta;          // angiographic weight (Eqs. 7, 9)
        if (live && r == 0) {
            v[1] = (1.0 - delta) * lam;
            v[2] = delta * dd * LA;
            v[0] = eta * v[1] + v[2] / eta;
        }
        const double dpd = -eta * lam + dd / eta * LA;  // d(data)/d(delta)
        // the component's partial, and the en face derivative of its scan (lane 3's
        // is the other four's)
        const double pc = S == 0 ? (c == 0 ? p0.y : (c == 1 ? p0.z : p0.w)) : (c == 0 ? p1.x : (c == 1 ? p1.y : p1.z));
        const float jc = S == V ? (c == 0 ? mv[1] : mv[2]) : (c == 0 ? ov[1] : ov[2]);
        double g = c == 2 ? ws * pc : ws * pc + wa * GA * jc;
        if (S == 1) g = -g;
        if (S == 0 && c == (oX == 0 ? 1 : 0)) g += dpd * J.delta0 * tvy * dtvx;
        if (S == 1 && c == (oY == 1 ? 0 : 1)) g += dpd * J.delta0 * tvx * dtvy;
        if (live && r < 6) {
            // scan-order regulariser (gather form: this A-scan's two links)
            const float* DS = J.disp[S];
            const double da = DS[(size_t)a * 3 + c];
            double omp, omn, Lr, dLr;
            const int pa = prev_ascan(oS, i, j, w, h, J.wfb, omp);
            const int nb = next_ascan(oS, i, j, w, h, J.wfb, omn);
            if (pa >= 0) {
                huber_d(da - (double)DS[(size_t)pa * 3 + c], J.eps_r, J.ieps_r, Lr, dLr);
                g += J.alpha * dd * omp * dLr;
            }
            if (nb >= 0) {
                huber_d((double)DS[(size_t)nb * 3 + c] - da, J.eps_r, J.ieps_r, Lr, dLr);
                g -= J.alpha * dd * omn * dLr;
                v[3] = dd * omn * Lr;
            }
            // mean-displacement term: dM/dd_c = gamma d sum_c / N_A
            g += J.gamma * dd * (c == 0 ? sumd[0] : (c == 1 ? sumd[1] : sumd[2])) / (double)na;
            const size_t at = ((size_t)S * na + a) * 3 + c;
            if (J.grad) J.grad[at] = (float)g;
            if (J.grad64) J.grad64[at] = g;
            if (J.p) v[7] = g * J.p[at];  // directional derivative g . p (line search)
        }
    }
    block_reduce_store<8>(v, J.blk + (size_t)b * 8);
    __syncthreads();
    // the block that comes last (its count releases its row and acquires the
    // others') forms the sums, and leaves the count at zero for the next launch
    if (threadIdx.x == 0) {
        const unsigned n = __hip_atomic_fetch_add(J.ticket, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
        last = n == (unsigned)J.nblk - 1;
        if (last) __hip_atomic_store(J.ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (last) finalize(J, sumd);
}

// ---------------------------------------------------------------------------
// k_struct_multi: the structural data term of n = 3 or 4 volumes at one
// level (16-bit storage, even depth).  Each output A-scan resamples every
// volume once: the lateral blend of its value and of its x and y derivatives
// (separable: 4 taps along x per source row, then 4 along y), the depth
// interpolation (Eq. 2) of all three, and the depth derivative of the value.
// Every volume pair P < Q then forms the residual I_P - I_Q, the
// pseudo-Huber loss (Eq. 4) and the loss derivative times both volumes'
// derivatives, and writes the eight partial sums per A-scan that k_struct2
// writes for one pair (loss; x, y, z of P; x, y, z of Q; 0).  The pair
// kernels instead resample every volume once per pair it belongs to.
// Lanes hold two samples each, on the output grid of the first volume, as
// in k_struct2.

struct StencilS {
    uint32_t roff[4], coff[4];  // byte offsets of the 4 source rows and the 4 source columns
    float wx[4], dwx[4], wy[4], dwy[4];
    float wz[4], dwz[4];
    int base;  // source sample of the first depth tap of output sample 0
};

template <typename T>
__device__ __forceinline__ void make_stencil_s(StencilS& s, int i, int j, float dx, float dy, float dz, int w, int h,
                                               int d)
{
    int nx, ny, nz;
    float tx, ty, tz;
    split(i, uni(dx), nx, tx);
    split(j, uni(dy), ny, ty);
    split(0, uni(dz), nz, tz);
    nx = uni(nx);
    ny = uni(ny);
    nz = uni(nz);
    cr_taps(uni(tx), s.wx, s.dwx);
    cr_taps(uni(ty), s.wy, s.dwy);
    cr_taps(uni(tz), s.wz, s.dwz);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        s.wz[c] = uni(s.wz[c]);
        s.dwz[c] = uni(s.dwz[c]);
        s.roff[c] = (uint32_t)uni((int)((uint32_t)clampi(ny - 1 + c, 0, h - 1) * (uint32_t)w * (uint32_t)d *
                                        esize<T>::v));
        s.coff[c] = (uint32_t)uni((int)((uint32_t)clampi(nx - 1 + c, 0, w - 1) * (uint32_t)d * esize<T>::v));
    }
    s.base = uni(nz - 1);
}

// value, x derivative and y derivative blends of the 16 columns at one depth
__device__ __forceinline__ void blend3(const float (&c)[16], const StencilS& S, float& v, float& vx, float& vy)
{
    float r[4], dr[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        r[b] = S.wx[0] * c[b * 4];
        dr[b] = S.dwx[0] * c[b * 4];
#pragma unroll
        for (int a = 1; a < 4; ++a) {
            r[b] = fmaf(S.wx[a], c[b * 4 + a], r[b]);
            dr[b] = fmaf(S.dwx[a], c[b * 4 + a], dr[b]);
        }
    }
    v = S.wy[0] * r[0];
    vx = S.wy[0] * dr[0];
    vy = S.dwy[0] * r[0];
#pragma unroll
    for (int b = 1; b < 4; ++b) {
        v = fmaf(S.wy[b], r[b], v);
        vx = fmaf(S.wy[b], dr[b], vx);
        vy = fmaf(S.dwy[b], r[b], vy);
    }
}

// Blended values t0, t1 of the loaded pair (samples m, m + 1) to positions 2l
// and 2l + 1 of the output grid: clamp (a pair below the A-scan holds sample
// 0 twice, one above it sample d - 1 twice), then the shift by one sample
// when the volume's positions start one sample after a pair boundary (r = 1).
__device__ __forceinline__ void grid2(float t0, float t1, bool lo, bool hi, int r, float& c0, float& c1)
{
    const float u0 = hi ? t1 : t0, u1 = lo ? t0 : t1;
    const float u0n = shl1(u0);
    c0 = r ? u1 : u0;
    c1 = r ? u0n : u1;
}

// the resampled value and its x, y, z derivatives at positions 2l, 2l + 1
struct Resampled {
    float i[2], x[2], y[2], z[2];
};

template <typename T>
__device__ __forceinline__ void resample_step(Resampled& o, __amdgpu_buffer_rsrc_t rs, const StencilS& S, int E, int r,
                                              int n, int lane, int dp)
{
    const int m = E + kOutPerStep2 * n + 2 * lane;
    const uint32_t voff = (uint32_t)clampi(m, 0, dp - 2) * esize<T>::v;
    float q0[16], q1[16];
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int a = 0; a < 4; ++a) ld2<T>(rs, voff, S.roff[b] + S.coff[a], q0[b * 4 + a], q1[b * 4 + a]);
    const bool lo = m < 0, hi = m > dp - 2;
    float v0, vx0, vy0, v1, vx1, vy1;
    blend3(q0, S, v0, vx0, vy0);
    blend3(q1, S, v1, vx1, vy1);
    float c0, c1;
    grid2(v0, v1, lo, hi, r, c0, c1);
    {
        const float c0n = shl1(c0), c1n = shl1(c1), c0nn = shl1(c0n);
        o.i[0] = S.wz[0] * c0 + S.wz[1] * c1 + S.wz[2] * c0n + S.wz[3] * c1n;
        o.i[1] = S.wz[0] * c1 + S.wz[1] * c0n + S.wz[2] * c1n + S.wz[3] * c0nn;
        o.z[0] = S.dwz[0] * c0 + S.dwz[1] * c1 + S.dwz[2] * c0n + S.dwz[3] * c1n;
        o.z[1] = S.dwz[0] * c1 + S.dwz[1] * c0n + S.dwz[2] * c1n + S.dwz[3] * c0nn;
    }
    grid2(vx0, vx1, lo, hi, r, c0, c1);
    {
        const float c0n = shl1(c0), c1n = shl1(c1), c0nn = shl1(c0n);
        o.x[0] = S.wz[0] * c0 + S.wz[1] * c1 + S.wz[2] * c0n + S.wz[3] * c1n;
        o.x[1] = S.wz[0] * c1 + S.wz[1] * c0n + S.wz[2] * c1n + S.wz[3] * c0nn;
    }
    grid2(vy0, vy1, lo, hi, r, c0, c1);
    {
        const float c0n = shl1(c0), c1n = shl1(c1), c0nn = shl1(c0n);
        o.y[0] = S.wz[0] * c0 + S.wz[1] * c1 + S.wz[2] * c0n + S.wz[3] * c1n;
        o.y[1] = S.wz[0] * c1 + S.wz[1] * c0n + S.wz[2] * c1n + S.wz[3] * c0nn;
    }
}

template <int N>
struct StructMultiJob {
    const void* vol[N];            // storage-type volumes of this level, [h][w][dp]
    const float* disp;             // [N][h][w][3]
    float* part[N * (N - 1) / 2];  // per pair (P, Q), P < Q in lexicographic order: [na][8]
    int w, h, d, na;
    int dp;                        // storage pitch (d, or d + 1 for an odd depth in 16-bit storage)
    uint32_t vol_bytes;
    float eps_h;
    const int* skip;  // device flag: when nonzero the launch does nothing (may be null)
};

template <typename T, int N>
__global__ __launch_bounds__(256) void k_struct_multi(const StructMultiJob<N> J)
{
    if (J.skip && *J.skip) return;
    constexpr int NP = N * (N - 1) / 2;
    const int wv = uni((int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    const int lb = xcd_block(blockIdx.x, gridDim.x);
    const int w = J.w, h = J.h, d = J.d, dp = J.dp;
    // 2 x 2 tiles in 8 bands of tile rows, swept column by column (as k_struct2)
    const int tpr = (w + 1) >> 1;
    const int trows = (h + 1) >> 1;
    const int rpb = (trows + 7) >> 3;
    const int band = lb / (rpb * tpr), tb = lb - band * (rpb * tpr);
    const int trow = band * rpb + tb % rpb;
    if (lb >= 8 * rpb * tpr || trow >= trows) return;  // whole block
    const int i = 2 * (tb / rpb) + (wv & 1);
    const int j = 2 * trow + (wv >> 1);
    if (i >= w || j >= h) return;  // whole wave
    const int a = uni(j * w + i);
    StencilS S[N];
    __amdgpu_buffer_rsrc_t rs[N];
#pragma unroll
    for (int V = 0; V < N; ++V) {
        const float* dv = J.disp + ((size_t)V * J.na + a) * 3;
        make_stencil_s<T>(S[V], i, j, dv[0], dv[1], dv[2], w, h, dp);
        rs[V] = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(J.vol[V]), (short)0, (int)J.vol_bytes, kRsrcWord3);
    }
    // output grid: position 0 of step 0 holds sample base_0 - s0 of volume 0
    const int s0 = S[0].base & 1;
    int r[N], E[N];
#pragma unroll
    for (int V = 0; V < N; ++V) {
        r[V] = uni((S[V].base - s0) & 1);
        E[V] = S[V].base - s0 - r[V];  // even
    }
    const float eps = J.eps_h;
    const float inv_eps = 1.0f / J.eps_h;
    float acc[NP][7];
#pragma unroll
    for (int q = 0; q < NP; ++q)
#pragma unroll
        for (int c = 0; c < 7; ++c) acc[q][c] = 0.f;
    const int nsteps = (d + kOutPerStep2 - 1) / kOutPerStep2;
    for (int n = 0; n < nsteps; ++n) {
        Resampled R[N];
#pragma unroll
        for (int V = 0; V < N; ++V) resample_step<T>(R[V], rs[V], S[V], E[V], r[V], n, lane, dp);
        const int p0 = 2 * lane;
        const int o0 = kOutPerStep2 * n + p0 - s0;
        const bool ok[2] = {p0 >= s0 && p0 <= 121 + s0 && o0 < d, p0 + 1 <= 121 + s0 && o0 + 1 < d};
        int q = 0;
#pragma unroll
        for (int P = 0; P < N; ++P)
#pragma unroll
            for (int Q = P + 1; Q < N; ++Q, ++q) {
                float L[2], G[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const float u = (R[P].i[e] - R[Q].i[e]) * inv_eps, uu = u * u;
                    const float rsq = __builtin_amdgcn_rsqf(1.f + uu), sq = (1.f + uu) * rsq;
                    L[e] = ok[e] ? eps * uu * __builtin_amdgcn_rcpf(sq + 1.f) : 0.f;
                    G[e] = ok[e] ? u * rsq : 0.f;
                }
                acc[q][0] += L[0] + L[1];
                acc[q][1] += G[0] * R[P].x[0] + G[1] * R[P].x[1];
                acc[q][2] += G[0] * R[P].y[0] + G[1] * R[P].y[1];
                acc[q][3] += G[0] * R[P].z[0] + G[1] * R[P].z[1];
                acc[q][4] += G[0] * R[Q].x[0] + G[1] * R[Q].x[1];
                acc[q][5] += G[0] * R[Q].y[0] + G[1] * R[Q].y[1];
                acc[q][6] += G[0] * R[Q].z[0] + G[1] * R[Q].z[1];
            }
    }
#pragma unroll
    for (int q = 0; q < NP; ++q) {
        float v[7];
#pragma unroll
        for (int c = 0; c < 7; ++c) v[c] = wave_sum_last(acc[q][c]);
        if (lane == 63) {
            float4* o = reinterpret_cast<float4*>(J.part[q] + (size_t)a * 8);
            o[0] = make_float4(v[0], v[1], v[2], v[3]);
            o[1] = make_float4(v[4], v[5], v[6], 0.f);
        }
    }
}

// k_multi_mx: k_struct_multi and k_struct_multi1 on the matrix cores, with the
// tiles, set-up and layout of k_struct_mx.  Every volume's blends are moved to
// the positions of the first volume's; a lane then holds the value and the x, y,
// z derivatives of all N volumes at four depths (four rather than eight, since
// 16 N registers hold them), and the pairs are formed from those.
// Bound by vector issue: with N = 4 a step takes some 900 vector instructions
// for 58 outputs of four A-scans, where k_struct_multi takes 996 for 122 of one.
// Two waves per SIMD (256 registers); the depth taps and the column offsets are
// read from the LDS at each step, which leaves registers to load one volume
// ahead.  Four volumes of 300 x 300 x 640 in BF16: 1230 -> 850 us per
// evaluation (1013 without loading ahead, 880 with the offsets in registers); in
// float32, whose matrix products take the vector units' time, 1521 -> 1318.
template <typename T, int N>
__global__ __launch_bounds__(256, 2) void k_multi_mx(const StructMultiJob<N> J)
{
    if (J.skip && *J.skip) return;
    constexpr int NP = N * (N - 1) / 2, L = 4;
    constexpr int kEs = (int)esize<T>::v;
    typedef MxGeo<kEs, L> Geo;
    __shared__ MxLds<kEs, N, L> lds[4];
    __shared__ f32x4 taps[4][N][4][2];  // per wave, volume and A-scan: the depth taps and their derivatives
    const int wv = uni((int)(threadIdx.x >> 6));
    MxLds<kEs, N, L>& M = lds[wv];
    const int w = J.w, h = J.h, d = J.d, dp = J.dp;
    int i0, j0;
    if (!mx_tile(w, h, xcd_block(blockIdx.x, gridDim.x), wv, i0, j0)) return;
    __amdgpu_buffer_rsrc_t rs[N];
#pragma unroll
    for (int V = 0; V < N; ++V)
        rs[V] = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(J.vol[V]), (short)0, (int)J.vol_bytes, kRsrcWord3);
    const float inv_eps = 1.0f / J.eps_h;
    int groups = 15;  // as k_struct_mx
    for (;;) {
        int lane = threadIdx.x & 63;
        asm volatile("" : "+v"(lane));
        const int g = lane >> 4;
        const bool last = (lane & 15) == 15;
        const int p0 = L * (lane & 15);
        const int2 pg = make_int2(min(i0 + (g & 1), w - 1), min(j0 + (g >> 1), h - 1));
        const bool inscan = i0 + (g & 1) < w && j0 + (g >> 1) < h;
        const int ag = pg.y * w + pg.x;
        const float ie_lo = p0 < Geo::kOut ? inv_eps : 0.f, ie_hi = p0 + 2 < Geo::kOut ? inv_eps : 0.f;
        MxScan S[N];
        int nrest = 0;
        bool fits = true;
#pragma unroll
        for (int V = 0; V < N; ++V) {
            fits = fits && mx_setup<T, 3>(S[V], M, V, J.disp + (size_t)V * J.na * 3, ag, pg, V ? S[0].sh : 0, w, h, dp, lane,
                                       groups, nrest);
            if ((lane & 15) == 0) {
                taps[wv][V][g][0] = f32x4{S[V].wz[0], S[V].wz[1], S[V].wz[2], S[V].wz[3]};
                taps[wv][V][g][1] = f32x4{S[V].dwz[0], S[V].dwz[1], S[V].dwz[2], S[V].dwz[3]};
            }
        }
        mx_lds_fence();
        if (!fits) {
            groups = 3;
            continue;
        }
        float acc[NP][7];
#pragma unroll
        for (int q = 0; q < NP; ++q)
#pragma unroll
            for (int c = 0; c < 7; ++c) acc[q][c] = 0.f;
        const int nsteps = (d + S[0].any + Geo::kOut - 1) / Geo::kOut;
        typename MxDwords<Geo::kDw>::type next[8];
        mx_load(next, S[0], M, 0, rs[0], 0, dp, lane);
        for (int s = 0; s < nsteps; ++s) {
            float I[N][L], X[N][L], Y[N][L], Z[N][L];
#pragma unroll
            for (int V = 0; V < N; ++V) {
                // the next volume's samples are loaded while this one is blended
                typename MxDwords<Geo::kDw>::type q[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) q[k] = next[k];
                if (V + 1 < N) mx_load(next, S[V + 1], M, V + 1, rs[V + 1], s, dp, lane);
                else if (s + 1 < nsteps) mx_load(next, S[0], M, 0, rs[0], s + 1, dp, lane);
                __builtin_amdgcn_sched_barrier(0);
                f32x4 D[L] = {};
                mx_blend<T>(D, q, M, V, lane, S[V].ns);
                if (S[V].ns > 32) mx_rest<T>(D, S[V], M, V, rs[V], s, dp, lane);
                float v[3][L];
                if (V == 0) mx_rows<false>(v, D, S[V], M, s, dp, lane);
                else mx_rows<true>(v, D, S[V], M, s, dp, lane);
                float e[L + 3], ex[L + 3], ey[L + 3];
#pragma unroll
                for (int i = 0; i < L; ++i) {
                    e[i] = v[0][i];
                    ex[i] = v[1][i];
                    ey[i] = v[2][i];
                }
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    e[L + i] = row_next(e[i]);
                    ex[L + i] = row_next(ex[i]);
                    ey[L + i] = row_next(ey[i]);
                }
                const f32x4 t0 = taps[wv][V][g][0], t1 = taps[wv][V][g][1];
                const float wz[4] = {t0[0], t0[1], t0[2], t0[3]}, dwz[4] = {t1[0], t1[1], t1[2], t1[3]};
#pragma unroll
                for (int i = 0; i < L; ++i) {
                    I[V][i] = mx_fir(wz, e, i);
                    Z[V][i] = mx_fir(dwz, e, i);
                    X[V][i] = mx_fir(wz, ex, i);
                    Y[V][i] = mx_fir(wz, ey, i);
                }
                __builtin_amdgcn_sched_barrier(0);  // no volume's loads earlier than that: registers
            }
            const int o0 = Geo::kOut * s + p0 - S[0].sh;
            float ie[L];
#pragma unroll
            for (int i = 0; i < L; ++i) ie[i] = i < 2 ? ie_lo : ie_hi;
            if (s == 0 || Geo::kOut * (s + 1) > d) {
#pragma unroll
                for (int i = 0; i < L; ++i) ie[i] = (unsigned)(o0 + i) < (unsigned)d ? ie[i] : 0.f;
            }
            int q = 0;
#pragma unroll
            for (int P = 0; P < N; ++P)
#pragma unroll
                for (int Q = P + 1; Q < N; ++Q, ++q)
#pragma unroll
                    for (int i = 0; i < L; ++i) {
                        const float u = (I[P][i] - I[Q][i]) * ie[i], uu = u * u;
                        const float rsq = __builtin_amdgcn_rsqf(1.f + uu), sq = (1.f + uu) * rsq;
                        const float G = u * rsq;
                        acc[q][0] = fmaf(uu, __builtin_amdgcn_rcpf(sq + 1.f), acc[q][0]);
                        acc[q][1] = fmaf(G, X[P][i], acc[q][1]);
                        acc[q][2] = fmaf(G, Y[P][i], acc[q][2]);
                        acc[q][3] = fmaf(G, Z[P][i], acc[q][3]);
                        acc[q][4] = fmaf(G, X[Q][i], acc[q][4]);
                        acc[q][5] = fmaf(G, Y[Q][i], acc[q][5]);
                        acc[q][6] = fmaf(G, Z[Q][i], acc[q][6]);
                    }
        }
        const bool active = groups >> g & 1;
        bool finite = true;
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            float v[7];
#pragma unroll
            for (int c = 0; c < 7; ++c) v[c] = row_sum_last(acc[q][c]);
            v[0] *= J.eps_h;
            finite = finite && __builtin_isfinite(((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + v[6]));
            if (last && inscan && active) {
                float4* o = reinterpret_cast<float4*>(J.part[q] + (size_t)ag * 8);
                o[0] = make_float4(v[0], v[1], v[2], v[3]);
                o[1] = make_float4(v[4], v[5], v[6], 0.f);
            }
        }
        groups = mx_next(groups, __ballot(last && active && !finite) != 0);
        if (!groups) return;
    }
}

// The same pass for float32 storage (any depth): one sample per lane, lane l
// holding source sample base_V + 61 n + l of volume V, as in k_struct; the
// depth interpolation of output lane l (< 61) reads source lanes l .. l + 3,
// and taps outside the A-scan take the edge sample (clamped load index).
// Three waves per SIMD (at most 168 registers): for n = 4 that spills a few
// values (six scratch accesses per step) and measured 4 % faster than two.
template <int N>
__global__ __launch_bounds__(256, 3) void k_struct_multi1(const StructMultiJob<N> J)
{
    if (J.skip && *J.skip) return;
    constexpr int NP = N * (N - 1) / 2;
    const int wv = uni((int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    const int lb = xcd_block(blockIdx.x, gridDim.x);
    const int w = J.w, h = J.h, d = J.d;
    const int tpr = (w + 1) >> 1;
    const int trows = (h + 1) >> 1;
    const int rpb = (trows + 7) >> 3;
    const int band = lb / (rpb * tpr), tb = lb - band * (rpb * tpr);
    const int trow = band * rpb + tb % rpb;
    if (lb >= 8 * rpb * tpr || trow >= trows) return;  // whole block
    const int i = 2 * (tb / rpb) + (wv & 1);
    const int j = 2 * trow + (wv >> 1);
    if (i >= w || j >= h) return;  // whole wave
    const int a = uni(j * w + i);
    StencilS S[N];
    __amdgpu_buffer_rsrc_t rs[N];
#pragma unroll
    for (int V = 0; V < N; ++V) {
        const float* dv = J.disp + ((size_t)V * J.na + a) * 3;
        make_stencil_s<float>(S[V], i, j, dv[0], dv[1], dv[2], w, h, d);
        rs[V] = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(J.vol[V]), (short)0, (int)J.vol_bytes, kRsrcWord3);
    }
    const float eps = J.eps_h;
    const float inv_eps = 1.0f / J.eps_h;
    float acc[NP][7];
#pragma unroll
    for (int q = 0; q < NP; ++q)
#pragma unroll
        for (int c = 0; c < 7; ++c) acc[q][c] = 0.f;
    const int nsteps = (d + kOutPerStep - 1) / kOutPerStep;
    for (int n = 0; n < nsteps; ++n) {
        float I[N], X[N], Y[N], Z[N];
#pragma unroll
        for (int V = 0; V < N; ++V) {
            const uint32_t voff = (uint32_t)clampi(S[V].base + kOutPerStep * n + lane, 0, d - 1) * 4u;
            float c[16];
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int a2 = 0; a2 < 4; ++a2) c[b * 4 + a2] = ldv<float>(rs[V], voff, S[V].roff[b] + S[V].coff[a2]);
            float v, vx, vy;
            blend3(c, S[V], v, vx, vy);
            float iv = 0.f, iz = 0.f, ix = 0.f, iy = 0.f;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                iv = fmaf(S[V].wz[e], v, iv);
                iz = fmaf(S[V].dwz[e], v, iz);
                ix = fmaf(S[V].wz[e], vx, ix);
                iy = fmaf(S[V].wz[e], vy, iy);
                if (e < 3) {
                    v = shl1(v);
                    vx = shl1(vx);
                    vy = shl1(vy);
                }
            }
            I[V] = iv;
            X[V] = ix;
            Y[V] = iy;
            Z[V] = iz;
            // one volume's loads in flight at a time: hoisting all of them
            // would take 64 more registers (one wave per SIMD)
            __builtin_amdgcn_sched_barrier(0);
        }
        const bool ok = lane < kOutPerStep && n * kOutPerStep + lane < d;
        int q = 0;
#pragma unroll
        for (int P = 0; P < N; ++P)
#pragma unroll
            for (int Q = P + 1; Q < N; ++Q, ++q) {
                const float u = (I[P] - I[Q]) * inv_eps, uu = u * u;
                const float rsq = __builtin_amdgcn_rsqf(1.f + uu), sq = (1.f + uu) * rsq;
                const float L = ok ? eps * uu * __builtin_amdgcn_rcpf(sq + 1.f) : 0.f;
                const float G = ok ? u * rsq : 0.f;
                acc[q][0] += L;
                acc[q][1] = fmaf(G, X[P], acc[q][1]);
                acc[q][2] = fmaf(G, Y[P], acc[q][2]);
                acc[q][3] = fmaf(G, Z[P], acc[q][3]);
                acc[q][4] = fmaf(G, X[Q], acc[q][4]);
                acc[q][5] = fmaf(G, Y[Q], acc[q][5]);
                acc[q][6] = fmaf(G, Z[Q], acc[q][6]);
            }
    }
#pragma unroll
    for (int q = 0; q < NP; ++q) {
        float v[7];
#pragma unroll
        for (int c = 0; c < 7; ++c) v[c] = wave_sum_last(acc[q][c]);
        if (lane == 63) {
            float4* o = reinterpret_cast<float4*>(J.part[q] + (size_t)a * 8);
            o[0] = make_float4(v[0], v[1], v[2], v[3]);
            o[1] = make_float4(v[4], v[5], v[6], 0.f);
        }
    }
}

}  // namespace

hipError_t launch_sum(const SumJobs& jobs, int total_blocks, hipStream_t s)
{
    hipLaunchKernelGGL(k_sum, dim3(total_blocks), dim3(kRedBlock), 0, s, jobs);
    return hipGetLastError();
}

// The kernel that serves a job of 16-bit volumes (0 .. 3).  The choice is made
// by the job's own sizes, so its result does not depend on the other jobs of
// its launch; each kernel's jobs have their own grid (a multiple of the 8 XCDs).
//   k_struct_mx needs some thousands of tiles to fill the device; with fewer,
//   the one-A-scan kernels, whose waves are shorter, are as fast or faster
//   (64 x 64 x 128: 14 against 18 us, 64 x 64 x 400: 18 against 25, 90 x 90 x
//   400: 31 against 29, 128 x 128 x 256: 43 against 32).
//   k_struct2 loads sample pairs, 32-bit aligned at an even storage pitch
//   (every level of a pair); an odd pitch (volumes in the caller's layout) of
//   fewer A-scans takes one sample per lane.
//   With an odd pitch half the columns start between two 32-bit words, and
//   k_struct_mx's loads of them take longer (tile_blend.h); it is still the faster
//   one, k_struct's being one sample each: 500 x 500 x 465 BF16 916 -> 454 us (406
//   padded), 200 x 200 x 301 FP16 112 -> 75, 91 x 91 x 59 26.0 -> 24.3.
constexpr int kMxMinAscans = kFewMaxAscans + 1;  // it has no count of a combination's blocks to clear
enum { kByMx8, kByMx4, kByPairs, kBySamples };
static int struct_form(const StructJob& J, bool axial)
{
    if (axial || J.na < kMxMinAscans) return J.dp % 2 == 0 ? kByPairs : kBySamples;
    return mx_eight(J.d, J.dp) ? kByMx8 : kByMx4;
}

// Depth steps of the float32 matrix-core kernels, at most (a tile whose A-scans
// start apart needs up to kShift more positions, which costs depths just below a
// multiple of 58 another step), and of the one-A-scan kernels.
static int steps_mx(int d) { return (d + MxGeo<4, 4>::kShift + MxGeo<4, 4>::kOut - 1) / MxGeo<4, 4>::kOut; }
static int steps_one(int d) { return (d + kOutPerStep - 1) / kOutPerStep; }

// float32 jobs likewise.  Its matrix products run at the vector units' expense, so
// k_struct_mx needs more tiles to pay, and depths whose steps are little more than
// those of k_struct (one step costs 0.82 .. 0.92 of k_struct's from 200 x 200 A-scans
// on).  Evaluations by k_struct / k_struct_mx: 200 x 200 x 512 184 / 161 us, 300 x
// 300 x 640 484 / 431, 400 x 400 x 225 323 / 290; another step than k_struct's: 300 x
// 300 x 116 128 / 141, x 174 155 / 172, x 232 190 / 202, x 290 227 / 233; one in
// seven: x 406 312 / 301, 200 x 200 x 406 149 / 152 (156 before the displacement sums
// went with the launch).  Fewer A-scans: 190 x 190 x 512 165 / 136, 160 x 160 x 512
// 121 / 110, so the line could lie lower for depths of whole steps.
constexpr int kMxMinAscansF32 = 40000;
static bool f32_mx(int na, int d, int dp)
{
    return na >= kMxMinAscansF32 && dp >= 4 && 7 * steps_mx(d) <= 8 * steps_one(d);
}

// The jobs of one kernel's launch, and its blocks: first those of the displacement
// sums that the jobs ask for, then the jobs' own.
struct StructLaunch {
    StructJobs jobs{};
    int blocks = 0, sums = 0;
    void add(StructJob J, int n)
    {
        J.blk_begin = blocks;
        J.sum_begin = sums;
        blocks += n;
        sums += J.nsum;
        jobs.j[jobs.n++] = J;
    }
    dim3 grid()
    {
        jobs.sum_blocks = (sums + 7) / 8 * 8;
        return dim3((unsigned)(jobs.sum_blocks + (blocks + 7) / 8 * 8));
    }
};

template <typename T, bool AXIAL>
static hipError_t launch_struct_subsets(const StructJobs& jobs, hipStream_t s)
{
    StructLaunch part[4];
    for (int q = 0; q < jobs.n; ++q) {
        const StructJob& J = jobs.j[q];
        const int k = struct_form(J, AXIAL);
        part[k].add(J, k <= kByMx4 ? struct_mx_blocks(J.w, J.h) : struct_blocks(J.w, J.h));
    }
    for (StructLaunch& P : part) P.jobs.skip = jobs.skip;
    auto launch = [&](int k, void (*kernel)(StructJobs)) {
        const dim3 grid = part[k].grid();
        if (part[k].jobs.n) hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, part[k].jobs);
    };
    if constexpr (!AXIAL) {
        launch(kByMx8, k_struct_mx<T, 8>);
        launch(kByMx4, k_struct_mx<T, 4>);
    }
    launch(kByPairs, k_struct2<T, AXIAL>);
    launch(kBySamples, k_struct<T, AXIAL>);
    return hipGetLastError();
}

template <bool AXIAL>
static hipError_t launch_struct_t(const StructJobs& jobs, octmc_dtype dt, hipStream_t s)
{
    switch (dt) {
    case OCTMC_F32: {
        StructLaunch part[2];
        for (int q = 0; q < jobs.n; ++q) {
            const StructJob& J = jobs.j[q];
            const int k = !AXIAL && f32_mx(J.na, J.d, J.dp);
            part[k].add(J, k ? struct_mx_blocks(J.w, J.h) : struct_blocks(J.w, J.h));
        }
        for (StructLaunch& P : part) P.jobs.skip = jobs.skip;
        if constexpr (!AXIAL) {
            const dim3 grid = part[1].grid();
            if (part[1].jobs.n) hipLaunchKernelGGL((k_struct_mx<float, 4>), grid, dim3(256), 0, s, part[1].jobs);
        }
        const dim3 grid = part[0].grid();
        if (part[0].jobs.n) hipLaunchKernelGGL((k_struct<float, AXIAL>), grid, dim3(256), 0, s, part[0].jobs);
        return hipGetLastError();
    }
    case OCTMC_BF16:
        return launch_struct_subsets<bf16_t, AXIAL>(jobs, s);
    case OCTMC_F16:
        return launch_struct_subsets<f16_t, AXIAL>(jobs, s);
    default:
        return hipErrorInvalidValue;
    }
}

hipError_t launch_struct(const StructJobs& jobs, octmc_dtype dt, hipStream_t s, bool axial)
{
    return axial ? launch_struct_t<true>(jobs, dt, s) : launch_struct_t<false>(jobs, dt, s);
}

// The choice is made by the job's own sizes, as for the structural kernels.
hipError_t launch_combine(const CombineJobs& jobs, hipStream_t s)
{
    CombineJobs few{}, many{};
    few.skip = many.skip = jobs.skip;
    int nb[2] = {0, 0};
    for (int q = 0; q < jobs.n; ++q) {
        CombineJob J = jobs.j[q];
        const bool f = few_ascans(J.na);
        J.blk_begin = nb[f];
        J.nblk = combine_rows(J.na);
        nb[f] += J.nblk;
        CombineJobs& to = f ? few : many;
        to.j[to.n++] = J;
    }
    if (few.n) hipLaunchKernelGGL(k_combine_few, dim3(nb[1]), dim3(kRedBlock), 0, s, few);
    if (many.n) {
        hipLaunchKernelGGL(k_combine, dim3(nb[0]), dim3(kRedBlock), 0, s, many);
        hipLaunchKernelGGL(k_finalize, dim3(many.n), dim3(kRedBlock), 0, s, many);
    }
    return hipGetLastError();
}

// k_multi_mx with fewer A-scans than this leaves the device's registers and LDS
// (two workgroups per CU) without tiles: four volumes of 96 x 96 x 200 in BF16
// 99 against k_struct_multi's 87 us per evaluation, 128 x 128 x 256 141 against
// 153.  Three float32 volumes stay with k_struct_multi1, which has the registers for
// them: 200 x 200 x 512 302 against 342, 300 x 300 x 640 833 against 870.
constexpr int kMxMultiMinAscans = 16384;
static_assert(kMxMinAscansF32 > kFewMaxAscans, "nor has its float32 form");
// Four float32 volumes gain from some 250 x 250 A-scans on, where a step costs 0.83
// of k_struct_multi1's, and with fewer where they exceed the 256 MB Infinity Cache,
// which k_struct_multi1 reads them from more often, and no step is added.
// k_struct_multi1 / k_multi_mx: 250 x 250 x 110 285 / 267 us, x 170 350 / 338, x 290
// (6 steps to 5) 566 / 519, x 116 (3 to 2) 283 / 329; 300 x 300 x 174 (4 to 3) 549 /
// 565; 200 x 200 x 225 282 / 305, x 340 377 / 393, x 400 (256 MB) 483 / 427, x 512
// 591 / 511; 230 x 230 x 225 367 / 376, x 340 564 / 502, x 406 (8 to 7) 645 / 655.
static bool f32_multi_mx(int na, int d)
{
    if (na >= 62500) return 5 * steps_mx(d) <= 6 * steps_one(d);
    return (int64_t)na * d >= 16000000 && steps_mx(d) <= steps_one(d);
}
template <int N>
static hipError_t launch_struct_multi_n(const void* const* vol, const float* disp, float* const* part, int w, int h,
                                        int d, int dp, uint32_t vol_bytes, float eps_h, octmc_dtype dt,
                                        hipStream_t s, const int* skip)
{
    StructMultiJob<N> J{};
    J.skip = skip;
    for (int V = 0; V < N; ++V) J.vol[V] = vol[V];
    for (int q = 0; q < N * (N - 1) / 2; ++q) J.part[q] = part[q];
    J.disp = disp;
    J.w = w;
    J.h = h;
    J.d = d;
    J.dp = dp;
    J.na = w * h;
    J.vol_bytes = vol_bytes;
    J.eps_h = eps_h;
    const int blocks = (struct_blocks(w, h) + 7) / 8 * 8;  // a multiple of the 8 XCDs
    const int mx = struct_mx_blocks(w, h);
    if constexpr (N == 4)
        if (dt == OCTMC_F32 && f32_multi_mx(J.na, d)) {
            hipLaunchKernelGGL((k_multi_mx<float, N>), dim3(mx), dim3(256), 0, s, J);
            return hipGetLastError();
        }
    if (dt == OCTMC_F32)
        hipLaunchKernelGGL((k_struct_multi1<N>), dim3(blocks), dim3(256), 0, s, J);
    else if (J.na >= kMxMultiMinAscans && dt == OCTMC_BF16)
        hipLaunchKernelGGL((k_multi_mx<bf16_t, N>), dim3(mx), dim3(256), 0, s, J);
    else if (J.na >= kMxMultiMinAscans)
        hipLaunchKernelGGL((k_multi_mx<f16_t, N>), dim3(mx), dim3(256), 0, s, J);
    else if (dt == OCTMC_BF16)
        hipLaunchKernelGGL((k_struct_multi<bf16_t, N>), dim3(blocks), dim3(256), 0, s, J);
    else
        hipLaunchKernelGGL((k_struct_multi<f16_t, N>), dim3(blocks), dim3(256), 0, s, J);
    return hipGetLastError();
}

bool struct_multi_supported(int n, int dp, octmc_dtype dt)
{
    // 16-bit storage holds two samples per lane, which needs an even pitch
    // (every level the n-volume path stores: odd depths are padded)
    return (n == 3 || n == 4) && (dt == OCTMC_F32 || ((dt == OCTMC_BF16 || dt == OCTMC_F16) && dp % 2 == 0));
}

hipError_t launch_struct_multi(const void* const* vol, int n, const float* disp, float* const* part, int w, int h,
                               int d, int dp, uint32_t vol_bytes, float eps_h, octmc_dtype dt, hipStream_t s,
                               const int* skip)
{
    if (!struct_multi_supported(n, dp, dt) || (dt == OCTMC_F32 && dp != d)) return hipErrorInvalidValue;
    if (n == 3) return launch_struct_multi_n<3>(vol, disp, part, w, h, d, dp, vol_bytes, eps_h, dt, s, skip);
    return launch_struct_multi_n<4>(vol, disp, part, w, h, d, dp, vol_bytes, eps_h, dt, s, skip);
}

}  // namespace octmc
