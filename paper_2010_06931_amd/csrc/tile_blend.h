// Device code shared by the structural and the merge kernels: the Catmull-Rom
// interpolator of Eq. 2 and the lateral resampling of tiles of A-scans on the
// matrix cores.
#pragma once

#include <hip/hip_runtime.h>

#include "octmc_internal.h"

namespace octmc {
namespace {

__device__ __forceinline__ float uni(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
}
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Cubic Hermite spline with central-difference tangents (Catmull-Rom), the
// C1 "Hermitian" interpolator of Eq. 2: weights of the samples at n-1 .. n+2
// for the fraction t in [0, 1), and their derivatives.
__device__ __forceinline__ void cr_taps(float t, float w[4], float dw[4])
{
    const float t2 = t * t, t3 = t2 * t;
    w[0] = 0.5f * (-t3 + 2.f * t2 - t);
    w[1] = 0.5f * (3.f * t3 - 5.f * t2 + 2.f);
    w[2] = 0.5f * (-3.f * t3 + 4.f * t2 + t);
    w[3] = 0.5f * (t3 - t2);
    dw[0] = 0.5f * (-3.f * t2 + 4.f * t - 1.f);
    dw[1] = 0.5f * (9.f * t2 - 10.f * t);
    dw[2] = 0.5f * (-9.f * t2 + 8.f * t + 1.f);
    dw[3] = 0.5f * (3.f * t2 - 2.f * t);
}

// Split an integer grid coordinate plus a displacement into the integer base
// and the fraction without rounding: dv = floor(dv) + frac exactly.
__device__ __forceinline__ void split(int idx, float dv, int& n, float& t)
{
    const float f = floorf(dv);
    t = dv - f;
    n = idx + (int)f;
}

__device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

struct bf16_t {};
struct f16_t {};
template <typename T> struct esize { static constexpr uint32_t v = 2; };
template <> struct esize<float> { static constexpr uint32_t v = 4; };

constexpr uint32_t kRsrcWord3 = 0x00020000u;

// Logical block of a physical one: workgroups are dispatched to the 8 XCDs
// round robin, so give every XCD a contiguous range of tiles (neighbouring
// A-scans then share that XCD's L2).  The grid is a multiple of 8.
__device__ __forceinline__ int xcd_block(int b, int nb)
{
    return (b & 7) * (nb >> 3) + (b >> 3);
}

template <int S>
__device__ __forceinline__ float row_shr_add(float v)
{
    return v + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x110 | S, 0xF,
                                                                     0xF, true));
}

// ---------------------------------------------------------------------------
// Lateral resampling of a tile of A-scans on the matrix cores.
//
// One wave serves a 2 x 2 tile of output A-scans.  Per volume the distinct
// source columns of the tile's four 4 x 4 lateral stencils (25 for a smooth
// field instead of 64) are the inner dimension of a small contraction,
//   D[4 g + o][k] = sum_slot W[4 g + o][slot] V[slot][k],
// whose rows are the lateral blends o = value (and, for NOUT = 3, x and y
// derivative) of A-scan g and whose columns are source depths.  W holds the
// Catmull-Rom products; a slot outside an A-scan's stencil has weight 0, so any
// set of displacements is served: 32 slots take one matrix product per depth
// tile, up to 48 a second one, and a tile with more (disjoint stencils) is
// served two A-scans at a time.
//   16-bit storage: v_mfma_f32_16x16x32 on the stored samples.  The float32
//     weights enter as three 16-bit parts, each the rest rounded to nearest.  Their
//     sum is the weight: exactly for BF16 (three times 8 bits) and for FP16 down to
//     2^-16 (11 + 11 + 2 bits of the weight times 2^15, undone in the depth taps);
//     binary16 ends at 2^-24, so a smaller weight is off by up to 2^-40.  The products
//     are then those of a float32 blend, and no sample is converted.  The
//     trailing parts are summed first, so that few additions round at the
//     blend's full size (error of a merged 200 x 200 x 300 volume against 64
//     bits: 6.1e-8, leading parts first 7.6e-8, vector FMAs 7.5e-8).  Splitting
//     by truncation instead would bias S_str by -2.6e-8: an addend smaller than
//     the products it is added to is truncated.
//   float32 storage: v_mfma_f32_16x16x4_f32, four slots at a time and none for
//     fours without a column.  These run on the vector units (timed: no overlap
//     with vector instructions), at twice their rate.  The last slots first: in
//     their order the error of a merged 300 x 300 x 300 volume is 7.6e-8,
//     reversed 7.3e-8, of vector FMAs 7.5e-8.
constexpr int kMxSlots = 48;
constexpr int kMxRest = 2;  // volumes of a tile that may have more than 32 slots
constexpr int kMxLimit = 1 << 28;  // positions beyond this lie outside every volume

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int i32x2 __attribute__((ext_vector_type(2)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

// Depth windows: a lane holds L consecutive source depths (one load per
// column), a row of 16 lanes a window of 16 L.  An A-scan's window starts
// sh = 0 .. kShift samples before its first depth tap, at a multiple of 4 bytes
// (loads off a 4-byte boundary take up to four times as long; those of every other
// column of a 16-bit volume with an odd pitch are); A-scans with a common start share
// their columns' loads.  Position p of the first volume's
// window holds the first tap of output kOut step + p - sh; the other volumes'
// blends are moved to the same positions.
template <int ES, int L>
struct MxGeo {
    static constexpr int es = ES;             // bytes per sample
    static constexpr int kWin = 16 * L;
    static constexpr int kShift = 3;
    static constexpr int kOut = kWin - 3 - kShift;  // outputs per step (four taps, the move), even
    static constexpr int kDw = L * ES / 4;    // dwords of a lane's load: 2 or 4
};

// A lane's samples of one column.
template <int N>
struct MxDwords;
template <>
struct MxDwords<2> {
    typedef i32x2 type;
    static __device__ __forceinline__ type load(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff)
    {
        return __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0);
    }
};
template <>
struct MxDwords<4> {
    typedef i32x4 type;
    static __device__ __forceinline__ type load(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff)
    {
        return __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0);
    }
};

// Matrix products.  A operands live in the LDS: of slot 4 q + kg (q = 0 .. 7)
// row m is element q of lane 16 kg + m; slots 32 .. 47 likewise with q = 0 .. 3.
template <typename T>
struct MxOps;

// the two samples of dword p of slots 2 t, 2 t + 1 of a lane, as the B operands of their depths
template <int NQ, typename S, typename B>
__device__ __forceinline__ void mx_pack(const S (&v)[NQ], int p, B& b0, B& b1)
{
#pragma unroll
    for (int t = 0; t < NQ / 2; ++t) {
        const unsigned lo = (unsigned)v[2 * t][p], hi = (unsigned)v[2 * t + 1][p];
        b0[t] = (int)__builtin_amdgcn_perm(hi, lo, 0x05040100u);
        b1[t] = (int)__builtin_amdgcn_perm(hi, lo, 0x07060302u);
    }
}

template <>
struct MxOps<float> {
    static constexpr float kUnscale = 1.f;
    typedef float part;
    static constexpr int kParts = 1;
    static __device__ __forceinline__ void split_weight(float w, part (&p)[1]) { p[0] = w; }
    static __device__ __forceinline__ f32x4 mfma(int a, int b, f32x4 c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(float, a), __builtin_bit_cast(float, b), c, 0, 0, 0);
    }
};

template <>
struct MxOps<bf16_t> {
    static constexpr float kUnscale = 1.f;
    typedef unsigned short part;
    static constexpr int kParts = 3;
    static __device__ __forceinline__ void split_weight(float w, unsigned short (&p)[3])
    {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const __bf16 hp = (__bf16)w;
            p[k] = __builtin_bit_cast(unsigned short, hp);
            w -= (float)hp;
        }
    }
    static __device__ __forceinline__ f32x4 mfma(i32x4 a, i32x4 b, f32x4 c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c,
                                                       0, 0, 0);
    }
    static __device__ __forceinline__ f32x4 mfma(i32x2 a, i32x2 b, f32x4 c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4, a), __builtin_bit_cast(s16x4, b), c,
                                                         0, 0, 0);
    }
};

template <>
struct MxOps<f16_t> {
    // binary16 has no room below 2^-24 for the trailing bits of a weight: the
    // weights are scaled by 2^15 (the largest, a derivative's, is 25 / 18, and 65504
    // the largest number) and the depth taps by 2^-15, both exact
    static constexpr float kScale = 32768.f, kUnscale = 1.f / kScale;
    typedef unsigned short part;
    static constexpr int kParts = 3;
    static __device__ __forceinline__ void split_weight(float w, unsigned short (&p)[3])
    {
        float r = w * kScale;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const _Float16 hp = (_Float16)r;
            p[k] = __builtin_bit_cast(unsigned short, hp);
            r -= (float)hp;
        }
    }
    static __device__ __forceinline__ f32x4 mfma(i32x4 a, i32x4 b, f32x4 c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0,
                                                      0, 0);
    }
    static __device__ __forceinline__ f32x4 mfma(i32x2 a, i32x2 b, f32x4 c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x16f16(__builtin_bit_cast(f16x4, a), __builtin_bit_cast(f16x4, b), c, 0,
                                                     0, 0);
    }
};

// The weights' arrays: of slot 4 q + kg, row m is element q (float32: q % 4 of
// array q / 4) of lane 16 kg + m.
template <int ES>
struct MxArr {  // 16-bit: one array per part
    static constexpr int kMain = 3, kRest = 3;
    typedef i32x2 rest_t;
};
template <>
struct MxArr<4> {
    static constexpr int kMain = 2, kRest = 1;
    typedef i32x4 rest_t;
};

// Per-wave LDS, for N volumes.
template <int ES, int N, int L>
struct MxLds {
    i32x4 a[N][MxArr<ES>::kMain][64];  // weights of a volume's slots 0 .. 31
    typename MxArr<ES>::rest_t rest[kMxRest][MxArr<ES>::kRest][64];  // of slots 32 .. 47, for the volumes that have them
    float edge[L][64];
    int2 key[N][64];     // per slot: byte offset of the column, first source depth of the window
    i32x4 off[N][4][2];  // [kg][q]: slot 4 q + kg, the column's byte offset at the tile's first window start, zlo
};

// The lanes of a wave exchange data through their own part of the LDS, whose
// accesses complete in order: only the compiler has to keep that order.
__device__ __forceinline__ void mx_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Lane shifts within a row of 16 lanes (DPP); the row's end reads 0.
__device__ __forceinline__ float row_next(float v)  // lane l gets lane l + 1's value
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x101, 0xF, 0xF, true));
}
__device__ __forceinline__ float row_prev(float v)  // lane l gets lane l - 1's value
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x111, 0xF, 0xF, true));
}
// sum over a row of 16 lanes, left in its last lane
__device__ __forceinline__ float row_sum_last(float x)
{
    float v = row_shr_add<1>(x);
    v = row_shr_add<2>(v);
    v = row_shr_add<4>(v);
    return row_shr_add<8>(v);
}

// Depths per lane with 16-bit storage: eight (true), since a 128-bit load brings
// twice the samples of a 64-bit one in the same time, unless windows of four
// leave enough fewer positions unused (a window of four costs 1.18 times half of
// one of eight); four where an A-scan has fewer than eight samples.
inline bool mx_eight(int d, int dp)
{
    const int n8 = (d + MxGeo<2, 8>::kOut - 1) / MxGeo<2, 8>::kOut, n4 = (d + MxGeo<2, 4>::kOut - 1) / MxGeo<2, 4>::kOut;
    return dp >= 8 && 17 * n8 <= 10 * n4;
}

// Per-scan state of one wave's tile.
struct MxScan {
    float wz[4], dwz[4]; // depth taps of this lane's A-scan and their derivatives
    int zb;              // source depth of window position 0 of this lane's A-scan at step 0
    int sh;              // position of the first depth tap
    int any;             // sh of the tile's A-scans, or-ed (wave-uniform)
    int zlo, zhi;        // smallest and largest zb of the tile (wave-uniform)
    int ns;              // slots (wave-uniform)
    int rest;            // index of the weights of slots 32 .. 47 (wave-uniform)
};

// The slots, weights and depth taps of one scan.  Lane 16 g + n stands for tap
// n of A-scan ag (at pg) of group g.  disp: the scan's field [na][3]; lead:
// position of the A-scan's output 0 (the window is laid out as if its first tap
// lay that much earlier); groups: bit mask of the groups whose stencils are
// laid out; nrest: the tile's volumes with more than 32 slots so far.  False:
// the tile needs more slots than there is room for, and fewer groups are to be
// laid out.
template <typename T, int NOUT, int N, int L>
__device__ __forceinline__ bool mx_setup(MxScan& S, MxLds<(int)esize<T>::v, N, L>& M, int V, const float* disp, int ag, int2 pg, int lead,
                                         int w, int h, int dp, int lane, int groups, int& nrest)
{
    typedef MxGeo<(int)esize<T>::v, L> Geo;
    typedef MxOps<T> Ops;
    typedef MxArr<Geo::es> Arr;
    const int g = lane >> 4, n = lane & 15;
    int nx, ny, nz;
    float tx, ty, tz;
    split(pg.x, disp[(size_t)ag * 3], nx, tx);
    split(pg.y, disp[(size_t)ag * 3 + 1], ny, ty);
    split(0, disp[(size_t)ag * 3 + 2], nz, tz);
    nx = min(max(nx, -kMxLimit), kMxLimit);
    ny = min(max(ny, -kMxLimit), kMxLimit);
    nz = min(max(nz, -kMxLimit), kMxLimit) - 1 - lead;  // source sample of the first tap of output 0, less lead
    // the tile's stencil origins, wave-uniform
    int ox[4], oy[4], oz[4], zb[4];
    int zmin = kMxLimit;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        ox[q] = __builtin_amdgcn_readlane(nx, 16 * q) - 1;
        oy[q] = __builtin_amdgcn_readlane(ny, 16 * q) - 1;
        oz[q] = __builtin_amdgcn_readlane(nz, 16 * q);
        if (groups >> q & 1) zmin = min(zmin, oz[q]);
    }
    if (Geo::es == 2) zmin &= -2;
    S.any = 0;
    S.zlo = kMxLimit;
    S.zhi = -2 * kMxLimit;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int sh = (oz[q] - zmin) & Geo::kShift;
        zb[q] = oz[q] - sh;
        S.any |= sh;
        S.zlo = min(S.zlo, zb[q]);
        S.zhi = max(S.zhi, zb[q]);
    }
    S.any = uni(S.any);
    S.zlo = uni(S.zlo);
    S.zhi = uni(S.zhi);
    S.sh = (nz - zmin) & Geo::kShift;
    S.zb = nz - S.sh;
    cr_taps(tz, S.wz, S.dwz);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        S.wz[c] *= Ops::kUnscale;
        S.dwz[c] *= Ops::kUnscale;
    }
    // Distinct columns: a lane's column is that of the first group's lane that
    // reaches the same column with the same window.
    const int cx = nx - 1 + (n & 3), cy = ny - 1 + (n >> 2);
    int owner = lane;
#pragma unroll
    for (int q = 2; q >= 0; --q) {
        const int a = cx - ox[q], b = cy - oy[q];
        const bool same = (q < g) & ((groups >> q & 1) != 0) & ((unsigned)a < 4u) & ((unsigned)b < 4u) & (S.zb == zb[q]);
        owner = same ? 16 * q + 4 * b + a : owner;
    }
    const bool active = (groups >> g & 1) != 0;
    const bool mine = active & (owner == lane);
    const unsigned long long mask = __ballot(mine);
    S.ns = uni((int)__popcll(mask));
    S.rest = nrest;
    if (S.ns > 32) ++nrest;
    if (S.ns > kMxSlots || nrest > kMxRest) return false;
    const int rank = (int)__builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
    const int slot = __builtin_amdgcn_ds_bpermute(4 * owner, rank);
    // weights: 0 but for the rows of an A-scan in the slots of its columns.
    // Unused slots: an offset beyond the volume, whose loads return 0.
#pragma unroll
    for (int k = 0; k < Arr::kMain; ++k) M.a[V][k][lane] = i32x4{};
    if (S.ns > 32) {
#pragma unroll
        for (int k = 0; k < Arr::kRest; ++k) M.rest[S.rest][k][lane] = typename Arr::rest_t{};
    }
    M.key[V][lane] = make_int2((int)0x80000000u, (int)0x80000000u);
    int* const off = reinterpret_cast<int*>(&M.off[V][0][0]);
    if (lane < 32) off[lane] = (int)0x80000000u;
    mx_lds_fence();
    if (mine) {
        const int col = min(max(cy, 0), h - 1) * w + min(max(cx, 0), w - 1);
        const int x = (int)((uint32_t)col * (uint32_t)dp * (uint32_t)Geo::es);
        M.key[V][slot] = make_int2(x, S.zb);
        if (slot < 32) off[(slot & 3) * 8 + (slot >> 2)] = x + Geo::es * (S.zb - S.zlo);
    }
    {
        float wx[4], dwx[4], wy[4], dwy[4];
        cr_taps(tx, wx, dwx);
        cr_taps(ty, wy, dwy);
        const int a = n & 3, b = n >> 2;
        float vx = wx[0], gx = dwx[0], vy = wy[0], gy = dwy[0];
#pragma unroll
        for (int c = 1; c < 4; ++c) {
            vx = a == c ? wx[c] : vx;
            gx = a == c ? dwx[c] : gx;
            vy = b == c ? wy[c] : vy;
            gy = b == c ? dwy[c] : gy;
        }
        const float wt[3] = {vx * vy, gx * vy, vx * gy};
        const int q = (slot & 31) >> 2, row = 16 * (slot & 3) + 4 * g;
        typedef typename Ops::part part;
        constexpr int kEl = 16 / (int)sizeof(part), kEl1 = (int)(sizeof(typename Arr::rest_t) / sizeof(part));
        part* a0 = reinterpret_cast<part*>(&M.a[V][0][0]) + (q / kEl * 64 + row) * kEl + q % kEl;
        part* a1 = reinterpret_cast<part*>(&M.rest[S.rest][0][0]) + row * kEl1 + q % kEl1;
        part p[NOUT][Ops::kParts];
#pragma unroll
        for (int o = 0; o < NOUT; ++o) Ops::split_weight(wt[o], p[o]);
        if (active & (slot < 32)) {
#pragma unroll
            for (int o = 0; o < NOUT; ++o)
#pragma unroll
                for (int k = 0; k < Ops::kParts; ++k) a0[(k * 64 + o) * kEl] = p[o][k];
        }
        if (active & (slot >= 32)) {
#pragma unroll
            for (int o = 0; o < NOUT; ++o)
#pragma unroll
                for (int k = 0; k < Ops::kParts; ++k) a1[(k * 64 + o) * kEl1] = p[o][k];
        }
    }
    mx_lds_fence();
    return true;
}

// wave-uniform: no window of the tile reaches over an end of the A-scans
template <typename Geo>
__device__ __forceinline__ bool mx_inside(const MxScan& S, int step, int dp)
{
    return S.zlo + Geo::kOut * step >= 0 && S.zhi + Geo::kOut * step + Geo::kWin <= dp;
}

// The samples of one depth step of one scan: kL depths of slots 4 q + kg.
template <int ES, int N, int L>
__device__ __forceinline__ void mx_load(typename MxDwords<L * ES / 4>::type (&s)[8], const MxScan& S,
                                        const MxLds<ES, N, L>& M, int V, __amdgpu_buffer_rsrc_t r, int step, int dp, int lane)
{
    typedef MxGeo<ES, L> Geo;
    const int n = lane & 15, kg = lane >> 4, z0 = Geo::kOut * step;
    uint32_t off[8];
    const i32x4 t0 = M.off[V][kg][0], t1 = M.off[V][kg][1];
    const uint32_t lo = (uint32_t)ES * (uint32_t)min(max(S.zlo + z0 + L * n, 0), dp - L);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        off[q] = (uint32_t)t0[q] + lo;
        off[4 + q] = (uint32_t)t1[q] + lo;
    }
    if (S.zlo != S.zhi && !mx_inside<Geo>(S, step, dp)) {  // windows that start apart are clamped one by one
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int2 k = M.key[V][4 * q + kg];
            off[q] = (uint32_t)k.x + (uint32_t)ES * (uint32_t)min(max(k.y + z0 + L * n, 0), dp - L);
        }
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) s[q] = MxDwords<Geo::kDw>::load(r, off[q], 0);
}

// D += the blends of NQ slots per lane group, whose samples are s: a, their weights' arrays; ns of the slots hold columns
template <typename T, int NQ, int L, typename S, typename A>
__device__ __forceinline__ void mx_mul(f32x4 (&D)[L], const S (&s)[NQ], const A* a, int lane, int ns)
{
    typedef MxOps<T> Ops;
    if constexpr (esize<T>::v == 4) {
#pragma unroll
        for (int q = NQ - 1; q >= 0; --q) {  // the outer columns of most A-scans, then the inner ones
            if (4 * q >= ns) continue;
            const int w = a[(q >> 2) * 64 + lane][q & 3];
#pragma unroll
            for (int i = 0; i < L; ++i) D[i] = Ops::mfma(w, s[q][i], D[i]);
        }
    } else {
        const A a0 = a[lane], a1 = a[64 + lane], a2 = a[128 + lane];
#pragma unroll
        for (int p = 0; p < L / 2; ++p) {
            A b0, b1;
            mx_pack(s, p, b0, b1);
            D[2 * p] = Ops::mfma(a2, b0, D[2 * p]);
            D[2 * p + 1] = Ops::mfma(a2, b1, D[2 * p + 1]);
            D[2 * p] = Ops::mfma(a1, b0, D[2 * p]);
            D[2 * p + 1] = Ops::mfma(a1, b1, D[2 * p + 1]);
            D[2 * p] = Ops::mfma(a0, b0, D[2 * p]);
            D[2 * p + 1] = Ops::mfma(a0, b1, D[2 * p + 1]);
        }
    }
}

// D += the blends of slots 0 .. 31 of volume V, whose samples are s
template <typename T, int ES, int N, int L, typename S>
__device__ __forceinline__ void mx_blend(f32x4 (&D)[L], const S (&s)[8], const MxLds<ES, N, L>& M, int V, int lane, int ns = 32)
{
    mx_mul<T, 8>(D, s, &M.a[V][0][0], lane, ns);
}

// D += the blends of slots 32 .. 47 (only where a tile has them)
template <typename T, int ES, int N, int L>
__device__ __forceinline__ void mx_rest(f32x4 (&D)[L], const MxScan& S, const MxLds<ES, N, L>& M, int V,
                                        __amdgpu_buffer_rsrc_t r, int step, int dp, int lane)
{
    typedef MxGeo<ES, L> Geo;
    const int n = lane & 15, kg = lane >> 4, z0 = Geo::kOut * step;
    typename MxDwords<Geo::kDw>::type s[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int2 k = M.key[V][32 + 4 * q + kg];
        s[q] = MxDwords<Geo::kDw>::load(r, (uint32_t)k.x + (uint32_t)ES * (uint32_t)min(max(k.y + z0 + L * n, 0), dp - L), 0);
    }
    mx_mul<T, 4>(D, s, &M.rest[S.rest][0][0], lane, S.ns - 32);
}

// L samples read at clamp(m, 0, dp - L), moved to m .. m + L - 1 with the edge
// value beyond the A-scan: every wanted sample is among the lane's own, so the
// move is an indexed read of them (through the lane's column of sh).
template <int L>
__device__ __forceinline__ void mx_edge(float (&v)[L], const int (&at)[L], float (*sh)[64], int lane)
{
#pragma unroll
    for (int i = 0; i < L; ++i) sh[i][lane] = v[i];
    mx_lds_fence();
#pragma unroll
    for (int i = 0; i < L; ++i) v[i] = sh[at[i]][lane];
    mx_lds_fence();
}

// v moved K samples down (from the next lane's first ones) where `on`
template <int K, int L>
__device__ __forceinline__ void mx_move(float (&v)[L], bool on)
{
    float nx[K];
#pragma unroll
    for (int i = 0; i < K; ++i) nx[i] = row_next(v[i]);
#pragma unroll
    for (int i = 0; i < L; ++i) v[i] = on ? (i + K < L ? v[i + K < L ? i + K : 0] : nx[i + K >= L ? i + K - L : 0]) : v[i];
}

// The first NOUT lateral blends of this lane's A-scan at its L positions: the
// edge values beyond the A-scan, then (MOVE) the window's shift.
template <bool MOVE, int NOUT, int ES, int N, int L>
__device__ __forceinline__ void mx_rows(float (&v)[NOUT][L], const f32x4 (&D)[L], const MxScan& S, MxLds<ES, N, L>& M,
                                        int step, int dp, int lane)
{
    typedef MxGeo<ES, L> Geo;
#pragma unroll
    for (int o = 0; o < NOUT; ++o)
#pragma unroll
        for (int i = 0; i < L; ++i) v[o][i] = D[i][o];
    if (!mx_inside<Geo>(S, step, dp)) {
        const int m = S.zb + Geo::kOut * step + L * (lane & 15), mc = min(max(m, 0), dp - L);
        int at[L];
#pragma unroll
        for (int i = 0; i < L; ++i) at[i] = min(max(m + i, 0), dp - 1) - mc;
#pragma unroll
        for (int o = 0; o < NOUT; ++o) mx_edge<L>(v[o], at, M.edge, lane);
    }
    if (MOVE && (S.any & 1)) {
#pragma unroll
        for (int o = 0; o < NOUT; ++o) mx_move<1>(v[o], S.sh & 1);
    }
    if (MOVE && Geo::kShift > 1 && (S.any & 2)) {
#pragma unroll
        for (int o = 0; o < NOUT; ++o) mx_move<2>(v[o], S.sh & 2);
    }
}

// sum_c w[c] x[i + c] (x: this lane's positions and three of the next lane's)
template <int N>
__device__ __forceinline__ float mx_fir(const float (&w)[4], const float (&x)[N], int i)
{
    float s = w[0] * x[i];
#pragma unroll
    for (int c = 1; c < 4; ++c) s = fmaf(w[c], x[i + c], s);
    return s;
}

// The groups to evaluate after `groups` (0: done).  bad: a sum was not finite.
__device__ __forceinline__ int mx_next(int groups, bool bad)
{
    if (groups & (groups - 1)) return bad ? 1 : (groups == 3 ? 12 : 0);  // several groups
    return groups == 8 ? 0 : groups << 1;
}

// The tile of a wave: 4 x 4 A-scans per workgroup in 8 bands of block rows (one
// per XCD when the job fills the grid), swept column by column, so that the
// rows a block reads are still in that XCD's L2 when the next column reads
// them.  False: a whole block beyond the job's, or a wave outside the scan.
__device__ __forceinline__ bool mx_tile(int w, int h, int t, int wv, int& i0, int& j0)
{
    const int bpr = (w + 3) >> 2;
    const int brows = (h + 3) >> 2;
    const int rpb = (brows + 7) >> 3;
    const int band = t / (rpb * bpr), tb = t - band * (rpb * bpr);
    const int brow = band * rpb + tb % rpb;
    i0 = 4 * (tb / rpb) + 2 * (wv & 1);
    j0 = 4 * brow + 2 * (wv >> 1);
    return t < 8 * rpb * bpr && brow < brows && i0 < w && j0 < h;
}


}  // namespace
}  // namespace octmc
