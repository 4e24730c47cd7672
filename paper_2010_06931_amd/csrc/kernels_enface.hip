// Segmentation-free en face OCTA projection (Sec. 2.3) for gfx950.
//
// Volumes are [h][w][d] float32 in the common frame (depth contiguous).  The
// fast scan axis is x for the X-fast scan (V = 0) and y for the Y-fast scan
// (V = 1); B-scans are rows j (V = 0) or columns i (V = 1).  Steps:
//   k_median_rank  3-D median of radius 1 (clamped borders) and the width-15 rank
//                  filter keeping the 3rd smallest value along the fast axis
//   k_rank15       the same rank filter along the slow axis
//   k_radix_hist   three radix passes (11, 11, 10 bits; the first counted by
//   k_radix_select the slow-axis rank filter) that select the two order
//                  statistics on each side of the 5th and 95th percentile
//                  of the filtered volume over the valid B-scans
//   k_noise_sum    sums and squared deviations of the OCT noise samples, from which
//                  the last k_radix_select forms their threshold
//   k_mask_mean    both masks and the masked depth mean per A-scan
//   k_bscan_median per-B-scan median
//   k_enface_finish median subtraction and nearest-valid substitution
// Every selection (median, rank filter, order statistic) is made with min,
// max and median-of-three instructions on the float values themselves, so
// it is exact; the thresholds are formed in FP64 with the arithmetic order
// written out and no contraction.
#include <algorithm>
#include <cmath>

#include "octmc_internal.h"
#include "row_quads.h"

namespace octmc {
namespace {

constexpr int kMedTile = 62;   // depth outputs per wave (64 lanes, one halo lane each side)
constexpr int kHistBins = 2048;
constexpr int kHistBlocks = 2048;
constexpr int kNoiseBlocks = 1024;  // at most
constexpr int kMaxBscan = 8192;  // A-scans per B-scan (LDS sort of the B-scan median)

__device__ __forceinline__ float shl1(float v)  // lane l gets lane l + 1 (lane 63 gets 0)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x130, 0xF, 0xF, true));
}
__device__ __forceinline__ float shr1(float v)  // lane l gets lane l - 1 (lane 0 gets 0)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x138, 0xF, 0xF, true));
}
__device__ __forceinline__ float min3f(float a, float b, float c) { return __builtin_fminf(__builtin_fminf(a, b), c); }
__device__ __forceinline__ float max3f(float a, float b, float c) { return __builtin_fmaxf(__builtin_fmaxf(a, b), c); }
__device__ __forceinline__ float med3f(float a, float b, float c) { return __builtin_amdgcn_fmed3f(a, b, c); }
__device__ __forceinline__ void sort3(float& a, float& b, float& c)
{
    const float lo = min3f(a, b, c), mi = med3f(a, b, c), hi = max3f(a, b, c);
    a = lo;
    b = mi;
    c = hi;
}
__device__ __forceinline__ void ce(float& a, float& b)
{
    const float lo = __builtin_fminf(a, b), hi = __builtin_fmaxf(a, b);
    a = lo;
    b = hi;
}

// ---------------------------------------------------------------------------
// 3-D median of radius 1.
//
// A wave owns one line, 64 consecutive depths (62 outputs) and consecutive
// positions x along the fast axis, which it walks in order.  For each x it sorts
// the nine samples of the (line, k) plane at that x: the three lines j-1..j+1 are
// loaded and sorted per lane, the neighbours k-1 and k+1 come from the
// adjacent lanes, the three rank rows are sorted across k, and three more
// 3-sorts complete the order of this rows-and-columns-sorted 3 x 3 grid.
// With the three sorted planes A, B, C of x-1, x, x+1, sorting each rank m
// across the planes leaves a 3 x 9 grid sorted both ways; the element at
// (a, m) has at least (a+1)(m+1) samples at or below it and (3-a)(9-m) at
// or above it, which rules out 7 samples below and 7 above the median.  The
// median of the 27 is then the 7th smallest of the 13 remaining ones: the
// minima of ranks 5..8, the medians of ranks 2..6 and the maxima of ranks
// 0..3, three sorted lists.  The first and last are merged (Batcher), and
// the 7th smallest of that list X and the medians Y is min over r + s = 7
// of max(X_r, Y_s).
struct Plane {
    float v[9];
};

__device__ __forceinline__ Plane sorted_plane(float a, float b, float c)
{
    sort3(a, b, c);
    Plane p;
    p.v[0] = shr1(a);
    p.v[1] = a;
    p.v[2] = shl1(a);
    p.v[3] = shr1(b);
    p.v[4] = b;
    p.v[5] = shl1(b);
    p.v[6] = shr1(c);
    p.v[7] = c;
    p.v[8] = shl1(c);
    sort3(p.v[0], p.v[1], p.v[2]);
    sort3(p.v[3], p.v[4], p.v[5]);
    sort3(p.v[6], p.v[7], p.v[8]);
    sort3(p.v[2], p.v[4], p.v[6]);
    sort3(p.v[1], p.v[2], p.v[3]);
    sort3(p.v[5], p.v[6], p.v[7]);
    return p;
}

__device__ __forceinline__ float median27(const Plane& A, const Plane& B, const Plane& C)
{
    float x[8], y[5];
#pragma unroll
    for (int m = 0; m < 4; ++m) x[m] = min3f(A.v[m + 5], B.v[m + 5], C.v[m + 5]);
#pragma unroll
    for (int m = 0; m < 4; ++m) x[m + 4] = max3f(A.v[m], B.v[m], C.v[m]);
#pragma unroll
    for (int m = 0; m < 5; ++m) y[m] = med3f(A.v[m + 2], B.v[m + 2], C.v[m + 2]);
    // odd-even merge of the sorted halves x[0..3], x[4..7]
    ce(x[0], x[4]);
    ce(x[2], x[6]);
    ce(x[2], x[4]);
    ce(x[1], x[5]);
    ce(x[3], x[7]);
    ce(x[3], x[5]);
    ce(x[1], x[2]);
    ce(x[3], x[4]);
    ce(x[5], x[6]);
    const float t = min3f(__builtin_fmaxf(x[1], y[4]), __builtin_fmaxf(x[2], y[3]), __builtin_fmaxf(x[3], y[2]));
    return __builtin_fminf(min3f(t, __builtin_fmaxf(x[4], y[1]), __builtin_fmaxf(x[5], y[0])), x[6]);
}

// ---------------------------------------------------------------------------
// Order statistics by radix selection on the order-preserving integer image
// of the float values.  State lives in device memory so that the passes run
// back to back on the stream.
struct SelState {
    unsigned n;            // number of samples in the valid B-scans
    unsigned any_valid;    // 0: no B-scan valid, every sample counts
    unsigned prefix[4];    // selected high bits of each target
    unsigned rank[4];      // rank of each target among the samples with that prefix
    unsigned uprefix[4];   // the distinct prefixes, one histogram each in the next pass
    unsigned slot[4];      // index of each target's prefix in uprefix
    unsigned nu;           // number of distinct prefixes
    unsigned pad;
    double value[4];       // the four order statistics
    double p5, p95, thr_r; // percentiles and the threshold on the filtered volume
    double mu, thr_s;      // OCT noise mean and threshold
};

__device__ __forceinline__ unsigned ord_key(float v)
{
    const unsigned u = __builtin_bit_cast(unsigned, v);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float from_key(unsigned k)
{
    return __builtin_bit_cast(float, (k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}

// ---------------------------------------------------------------------------
// Rank filter: the 3rd smallest of the 15 samples p-7 .. p+7 along one
// lateral axis, clamped at the ends.
//
// A wave owns 64 consecutive depths of one line and a segment of `len`
// positions, which it walks in chunks of 15 aligned so that chunk c spans
// p0-7+15c .. p0+7+15c.  The window of output p = p0+15c+t is the tail of
// chunk c from offset t joined with the head of chunk c+1 up to offset t-1:
// the three smallest of each part are kept sorted (suffix triples of chunk
// c, a running prefix triple of chunk c+1), and the 3rd smallest of the
// union of two sorted triples a, b is min(a3, b3, max(a1, b2), max(a2, b1)).
// Inserting v into a sorted triple gives (min(a1, v), med3(a1, a2, v),
// med3(a2, a3, v)).  Every sample is loaded once per segment.
//
// With kHist (the slow-axis pass, whose positions are the B-scans) the
// kernel also counts bits 31..21 of every output of a valid B-scan: the
// first radix pass of the percentile selection.  Along the walk a lane's
// outputs change bin rarely, so each lane adds runs of equal bins.
//
// Neighbouring waves take neighbouring depths, then neighbouring lines: an
// A-scan's rows are no whole cache lines, and waves that share one then run
// together (500 x 500 x 465: 325 us with the segments of a line side by side,
// 291 us so; 930 MB are read and written).
struct Tri {
    float a, b, c;
};
__device__ __forceinline__ Tri insert(Tri t, float v)
{
    return Tri{__builtin_fminf(t.a, v), med3f(t.a, t.b, v), med3f(t.b, t.c, v)};
}
__device__ __forceinline__ float third_of_union(Tri s, Tri p)
{
    return min3f(__builtin_fminf(s.c, p.c), __builtin_fmaxf(s.a, p.b), __builtin_fmaxf(s.b, p.a));
}

// The suffix triples of a chunk.
__device__ __forceinline__ void suffixes(const float (&u)[15], Tri (&s)[15])
{
    constexpr float inf = __builtin_inff();
    s[14] = Tri{u[14], inf, inf};
#pragma unroll
    for (int t = 13; t >= 0; --t) s[t] = insert(s[t + 1], u[t]);
}

// Median and fast-axis rank filter in one walk: a wave owns one line, kMedTile
// depths and `seg` positions along the fast axis (n of them, ws samples apart;
// lines are ls apart), takes the medians in order and hands each to the rank
// filter's chunks, so the median volume is never stored.  Bound by its 95 vector
// instructions a position (326 us for 500 x 500 x 465 with every cycle used; 385
// measured, 660 to 750 as two kernels); the planes are loaded three positions
// ahead (one ahead: 468 us).
__global__ __launch_bounds__(256, 4) void k_median_rank(const float* __restrict__ in, float* __restrict__ out, int n,
                                                        int lines, size_t ws, size_t ls, int d, int seg)
{
    const int lane = threadIdx.x & 63;
    const int o = blockIdx.z * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (o >= lines) return;  // uniform per wave; no barrier in this kernel
    const int kk = blockIdx.x * kMedTile - 1 + lane;
    const int k = kk < 0 ? 0 : (kk >= d ? d - 1 : kk);
    const bool store = lane >= 1 && lane <= kMedTile && kk < d;
    const int p0 = blockIdx.y * seg, p1 = min(p0 + seg, n);
    const float* __restrict__ rm = in + (size_t)max(o - 1, 0) * ls;
    const float* __restrict__ r0 = in + (size_t)o * ls;
    const float* __restrict__ rp = in + (size_t)min(o + 1, lines - 1) * ls;
    float* __restrict__ q = out + (size_t)o * ls;
    float va[3], vb[3], vc[3];  // the next three planes, in flight
    auto fetch = [&](int x, int e) {
        const size_t at = (size_t)(x < 0 ? 0 : (x >= n ? n - 1 : x)) * ws;
        va[e] = rm[at + k];
        vb[e] = r0[at + k];
        vc[e] = rp[at + k];
    };
    fetch(p0 - 8, 1);
    fetch(p0 - 7, 2);
    fetch(p0 - 6, 0);
    Plane A = sorted_plane(va[1], vb[1], vc[1]);
    fetch(p0 - 5, 1);
    Plane B = sorted_plane(va[2], vb[2], vc[2]), C;
    fetch(p0 - 4, 2);
    float last = 0.0f;
    // median at position r from the planes a, b of r - 1, r and the fetched one of r + 1
    auto step = [&](int r, int e, const Plane& a, const Plane& b, Plane& c) {
        c = sorted_plane(va[e], vb[e], vc[e]);
        fetch(r + 4, e);
        const float m = median27(a, b, c);
        last = r < n ? m : last;  // positions are clamped: r >= n repeats n - 1
        return last;
    };
    float u[15];
    Tri s[15];
#pragma unroll
    for (int t = 0; t < 15; t += 3) {
        const int r = p0 - 7 + t;
        u[t] = step(r, 0, A, B, C);
        u[t + 1] = step(r + 1, 1, B, C, A);
        u[t + 2] = step(r + 2, 2, C, A, B);
    }
    if (p0 == 0) {
#pragma unroll
        for (int t = 0; t < 7; ++t) u[t] = u[7];  // and r < 0 is position 0
    }
    suffixes(u, s);
    constexpr float inf = __builtin_inff();
    for (int c0 = p0; c0 < p1; c0 += 15) {
        Tri pre{inf, inf, inf};
        auto emit = [&](int t, float v) {
            if (c0 + t < p1) {  // uniform
                const float r = third_of_union(s[t], pre);
                if (store) q[(size_t)(c0 + t) * ws + kk] = r;
            }
            u[t] = v;
            pre = insert(pre, v);
        };
#pragma unroll
        for (int t = 0; t < 15; t += 3) {
            const int r = c0 + 8 + t;
            emit(t, step(r, 0, A, B, C));
            emit(t + 1, step(r + 1, 1, B, C, A));
            emit(t + 2, step(r + 2, 2, C, A, B));
        }
        suffixes(u, s);
    }
}

template <bool kHist>
__global__ __launch_bounds__(256) void k_rank15(const float* __restrict__ in, float* __restrict__ out, int w, int h,
                                                int d, int axis, int len, const float* __restrict__ valid,
                                                const SelState* __restrict__ st, unsigned* __restrict__ hist)
{
    __shared__ unsigned lh[kHist ? kHistBins : 1];
    if (kHist) {
        for (int t = threadIdx.x; t < kHistBins; t += blockDim.x) lh[t] = 0u;
        __syncthreads();
    }
    const int lane = threadIdx.x & 63;
    const int ktiles = (d + 63) >> 6;
    const int n = axis == 0 ? w : h;
    const int nseg = (n + len - 1) / len;
    const int nlines = axis == 0 ? h : w;
    const int wid = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (wid < nlines * ktiles * nseg) {  // uniform per wave
        const int kt = wid % ktiles, rest = wid / ktiles;
        const int o = rest % nlines, seg = rest / nlines;
        const int k = kt * 64 + lane;
        const int kc = k < d ? k : d - 1;
        const bool store = k < d;
        const int p0 = seg * len, p1 = min(p0 + len, n);
        const size_t stride = axis == 0 ? (size_t)d : (size_t)w * d;
        const size_t base = (axis == 0 ? (size_t)o * w * d : (size_t)o * d) + kc;
        const float* __restrict__ p = in + base;
        float* __restrict__ q = out + base;
        const unsigned anyv = kHist ? st->any_valid : 0u;
        int cur = -1;       // bin of the current run of this lane's outputs
        unsigned run = 0u;  // and its length
        auto ld = [&](int pos) {
            pos = pos < 0 ? 0 : (pos >= n ? n - 1 : pos);
            return p[(size_t)pos * stride];
        };
        constexpr float inf = __builtin_inff();
        float u[15];
        Tri s[15];
#pragma unroll
        for (int t = 0; t < 15; ++t) u[t] = ld(p0 - 7 + t);
        suffixes(u, s);
        for (int c0 = p0; c0 < p1; c0 += 15) {
#pragma unroll
            for (int t = 0; t < 15; ++t) u[t] = ld(c0 + 8 + t);
            Tri pre{inf, inf, inf};
#pragma unroll
            for (int t = 0; t < 15; ++t) {
                if (c0 + t < p1) {  // uniform
                    const float r = third_of_union(s[t], pre);
                    if (store) q[(size_t)(c0 + t) * stride] = r;
                    if (kHist) {
                        const bool ok = store && (!anyv || valid[c0 + t] > 0.5f);
                        const int bin = ok ? (int)(ord_key(r) >> 21) : -1;
                        if (bin != cur) {
                            if (cur >= 0) atomicAdd(&lh[cur], run);
                            cur = bin;
                            run = 0u;
                        }
                        ++run;
                    }
                }
                pre = insert(pre, u[t]);
            }
            suffixes(u, s);
        }
        if (kHist && cur >= 0) atomicAdd(&lh[cur], run);
    }
    if (kHist) {
        __syncthreads();
        for (int t = threadIdx.x; t < kHistBins; t += blockDim.x)
            if (lh[t]) atomicAdd(&hist[t], lh[t]);
    }
}

// Nearest valid B-scan of each B-scan (the lower index on a tie; itself when
// none is valid), whether any is valid, and cleared histogram counters.
__global__ __launch_bounds__(256) void k_enface_init(const float* __restrict__ valid, int nb, int* __restrict__ from,
                                                     SelState* st, unsigned* __restrict__ hist)
{
    __shared__ int any;
    if (threadIdx.x == 0) any = 0;
    __syncthreads();
    for (int b = threadIdx.x; b < nb; b += blockDim.x)
        if (valid[b] > 0.5f) any = 1;  // benign race: every writer stores 1
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
    for (int t = threadIdx.x; t < 4 * kHistBins; t += blockDim.x) hist[t] = 0u;
    if (threadIdx.x == 0) {
        st->any_valid = any;
        st->n = 0;
    }
}

// Radix passes 1 and 2 over the filtered volume: pass 1 counts bits 20..10
// of the samples whose bits 31..21 equal one of the distinct target
// prefixes, pass 2 bits 9..0 of those whose bits 31..10 do; one histogram of
// kHistBins counters per distinct prefix (kTargets of them at most).  Pass 0 is
// counted by the slow-axis rank filter.  Prefixes and digits are taken from the
// float's own bits, which the key inverts below zero: a prefix that is below
// zero is compared inverted, and so is its digit.  500 x 500 x 465, 465 MB: 110 us
// (158 with a wave to an A-scan and 4-byte loads).
template <int kTargets>
__device__ __forceinline__ void count_rows(const float* __restrict__ vol, int w, int h, int d, int V,
                                           const float* __restrict__ valid, const SelState* __restrict__ st, int pass,
                                           unsigned* lh)
{
    const unsigned any = st->any_valid, nu = st->nu;
    const int shift = pass == 1 ? 21 : 10, dshift = pass == 1 ? 10 : 0, dbits = pass == 1 ? 11 : 10;
    unsigned pre[kTargets], flip[kTargets];
#pragma unroll
    for (int t = 0; t < kTargets; ++t) {
        const unsigned p = st->uprefix[t < (int)nu ? t : 0], top = 1u << (31 - shift);
        pre[t] = p & top ? p ^ top : p ^ (2 * top - 1);
        flip[t] = (unsigned)t * kHistBins | (p & top ? 0u : (1u << dbits) - 1);
    }
    const int part = threadIdx.x & (kRowLanes - 1);
    const unsigned na = (unsigned)w * (unsigned)h, rows = gridDim.x * (blockDim.x / kRowLanes);
    for (unsigned a = blockIdx.x * (blockDim.x / kRowLanes) + threadIdx.x / kRowLanes; a < na; a += rows) {
        const unsigned j = a / (unsigned)w, i = a - j * (unsigned)w;
        const unsigned b = V == 0 ? j : i;
        if (any && !(valid[b] > 0.5f)) continue;
        const float* __restrict__ col = vol + (size_t)a * d;
        for (int k0 = 0; k0 < d; k0 += kRowLoads * kRowStep) {
            Quad q[kRowLoads];
#pragma unroll
            for (int g = 0; g < kRowLoads; ++g)
                if (k0 + g * kRowStep < d) q[g] = load_quad(col, k0 + g * kRowStep + 4 * part, d);
#pragma unroll
            for (int g = 0; g < kRowLoads; ++g) {
                if (k0 + g * kRowStep >= d) break;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const unsigned u = __builtin_bit_cast(unsigned, (float)q[g].v[e]), hi = u >> shift;
                    bool hit = hi == pre[0];
                    unsigned f = flip[0];
#pragma unroll
                    for (int t = 1; t < kTargets; ++t) {
                        const bool m = hi == pre[t];
                        f = m && !hit ? flip[t] : f;
                        hit |= m;
                    }
                    if (hit && e >= q[g].first) atomicAdd(&lh[((u >> dshift) & ((1u << dbits) - 1)) ^ f], 1u);
                }
            }
        }
    }
}

__global__ __launch_bounds__(256) void k_radix_hist(const float* __restrict__ vol, int w, int h, int d, int V,
                                                    const float* __restrict__ valid, const SelState* __restrict__ st,
                                                    int pass, unsigned* __restrict__ hist)
{
    __shared__ unsigned lh[4 * kHistBins];
    const int nu = (int)st->nu;
    for (int t = threadIdx.x; t < nu * kHistBins; t += blockDim.x) lh[t] = 0u;
    __syncthreads();
    if (nu <= 2)  // both percentiles between neighbours of one prefix: the ordinary case
        count_rows<2>(vol, w, h, d, V, valid, st, pass, lh);
    else
        count_rows<4>(vol, w, h, d, V, valid, st, pass, lh);
    __syncthreads();
    for (int t = threadIdx.x; t < nu * kHistBins; t += blockDim.x)
        if (lh[t]) atomicAdd(&hist[t], lh[t]);
}

// Sum over a block of 256 threads in a fixed order; every thread gets it.
__device__ __forceinline__ double block_sum(double v, double (&red)[4])
{
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) v += __shfl_xor(v, m);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    return (red[0] + red[1]) + (red[2] + red[3]);
}

// OCT noise mean, and threshold from the squared deviations, of the block partials
// of k_noise_sum.
__device__ __forceinline__ double partial_mean(const double* __restrict__ partial, int nblk, double cnt,
                                               double (&red)[4])
{
    double v = 0.0;
    for (int b = threadIdx.x; b < nblk; b += blockDim.x) v += partial[b];
    return block_sum(v, red) / cnt;
}

// One block of 256: for each target, the bin whose counts cross its rank; after the
// last pass the order statistics, the percentiles and the threshold, and the noise
// threshold with them (noise: k_noise_sum's partials of both passes).  Clears the
// histograms it read.  All its reading is one round: the state and the four
// histograms go to registers and LDS before anything is decided (6.3 to 8.9 us; the
// percentiles of a 64 x 64 x 128 projection and its noise threshold took 39 us in
// seven launches before, 26 in five now).
struct NoiseSums {
    const double* sum;  // [nblk] sums, then [nblk] squared deviations
    int nblk;
    double cnt;
};
__global__ __launch_bounds__(256) void k_radix_select(unsigned* __restrict__ hist, SelState* st, int pass,
                                                      const NoiseSums noise)
{
#pragma clang fp contract(off)
    __shared__ SelState S;
    __shared__ unsigned wsum[4][4];
    __shared__ unsigned target[4];
    __shared__ double red[2][4];
    const int nbins = pass == 2 ? 1024 : kHistBins;
    const int per = nbins / 256;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    for (int t = tid; t < (int)(sizeof(SelState) / 4); t += 256)
        reinterpret_cast<unsigned*>(&S)[t] = reinterpret_cast<const unsigned*>(st)[t];
    unsigned c[4][8], local[4], incl[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        local[u] = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            c[u][e] = e < per && (pass > 0 || u == 0) ? hist[(size_t)u * kHistBins + tid * per + e] : 0u;
            local[u] += c[u][e];
        }
        unsigned v = local[u];  // inclusive scan
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const unsigned x = __shfl_up(v, off);
            v += lane >= off ? x : 0u;
        }
        incl[u] = v;
        if (lane == 63) wsum[u][wv] = v;
    }
    double mu = 0.0, var = 0.0;
    if (pass == 2) {
        mu = partial_mean(noise.sum, noise.nblk, noise.cnt, red[0]);
        var = partial_mean(noise.sum + noise.nblk, noise.nblk, noise.cnt, red[1]);
    }
    __syncthreads();
    if (pass == 0 && tid == 0) {
        const unsigned n = wsum[0][0] + wsum[0][1] + wsum[0][2] + wsum[0][3];
        S.n = n;
        const double q[2] = {0.05, 0.95};
        for (int e = 0; e < 2; ++e) {
            const double pos = q[e] * (double)(n - 1);
            unsigned lo = (unsigned)floor(pos);
            if (lo >= n - 1) lo = n - 1;
            target[2 * e] = lo;
            target[2 * e + 1] = lo + 1 < n ? lo + 1 : n - 1;
        }
    } else if (pass > 0 && tid < 4) {
        target[tid] = S.rank[tid];
    }
    __syncthreads();
    const int nslot = pass == 0 ? 1 : (int)S.nu;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        if (u >= nslot) break;
        unsigned excl = incl[u] - local[u];
        for (int k = 0; k < wv; ++k) excl += wsum[u][k];
        for (int t = 0; t < 4; ++t) {
            if (pass > 0 && (int)S.slot[t] != u) continue;
            const unsigned r = target[t];
            if (r >= excl && r < excl + local[u]) {  // one thread of one slot
                unsigned cum = excl, bin = 0;
                bool found = false;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    if (!found && (e == per - 1 || r < cum + c[u][e])) {
                        bin = (unsigned)(tid * per + e);
                        found = true;
                    }
                    if (!found) cum += c[u][e];
                }
                if (pass == 0) S.prefix[t] = bin;
                else if (pass == 1) S.prefix[t] = (S.prefix[t] << 11) | bin;
                else S.value[t] = (double)from_key((S.prefix[t] << 10) | bin);
                S.rank[t] = r - cum;
            }
        }
    }
    for (int t = tid; t < nslot * kHistBins; t += 256) hist[t] = 0u;
    __syncthreads();
    if (tid == 0 && pass < 2) {
        unsigned nu = 0;
        for (int t = 0; t < 4; ++t) {
            unsigned u = 0;
            while (u < nu && S.uprefix[u] != S.prefix[t]) ++u;
            if (u == nu) S.uprefix[nu++] = S.prefix[t];
            S.slot[t] = u;
        }
        S.nu = nu;
    } else if (tid == 0) {
        const unsigned n = S.n;
        const double q[2] = {0.05, 0.95};
        double p[2];
        for (int e = 0; e < 2; ++e) {
            const double pos = q[e] * (double)(n - 1);
            unsigned lo = (unsigned)floor(pos);
            if (lo >= n - 1) lo = n - 1;
            const double frac = pos - (double)lo;
            const double x0 = S.value[2 * e], x1 = S.value[2 * e + 1];
            if (lo + 1 < n) {
                const double dx = x1 - x0;
                const double step = frac * dx;
                p[e] = x0 + step;
            } else {
                p[e] = x0;
            }
        }
        S.p5 = p[0];
        S.p95 = p[1];
        const double span = p[1] - p[0];
        const double off = 0.1 * span;
        S.thr_r = p[0] + off;
        S.mu = mu;
        S.thr_s = mu + 2.0 * sqrt(var);
    }
    __syncthreads();
    for (int t = tid; t < (int)(sizeof(SelState) / 4); t += 256)
        reinterpret_cast<unsigned*>(st)[t] = reinterpret_cast<const unsigned*>(&S)[t];
}

// A fixed normalisation mapping in place of the percentiles, and the noise threshold.
__global__ __launch_bounds__(256) void k_set_fixed(SelState* st, double p5, double p95, const NoiseSums noise)
{
#pragma clang fp contract(off)
    __shared__ double red[2][4];
    const double mu = partial_mean(noise.sum, noise.nblk, noise.cnt, red[0]);
    const double var = partial_mean(noise.sum + noise.nblk, noise.nblk, noise.cnt, red[1]);
    if (threadIdx.x != 0) return;
    st->p5 = p5;
    st->p95 = p95;
    const double span = p95 - p5;
    const double off = 0.1 * span;
    st->thr_r = p5 + off;
    st->mu = mu;
    st->thr_s = mu + 2.0 * sqrt(var);
}

// OCT noise statistics over the first nz samples of every A-scan: pass 0 sums the
// samples, pass 1 the squared deviations from their mean, which every block forms
// from the first pass's partials.  Sixteen lanes to an A-scan; partial sums per
// block, combined in a fixed order.
__global__ __launch_bounds__(256) void k_noise_sum(const float* __restrict__ oct, unsigned na, int d, int nz, int pass,
                                                   const NoiseSums noise, double* __restrict__ partial)
{
    __shared__ double red[2][4];
    const double mu = pass ? partial_mean(noise.sum, noise.nblk, noise.cnt, red[0]) : 0.0;
    const int part = threadIdx.x & (kRowLanes - 1);
    const unsigned rows = gridDim.x * (blockDim.x / kRowLanes);
    double acc = 0.0;
#pragma unroll 4
    for (unsigned a = blockIdx.x * (blockDim.x / kRowLanes) + threadIdx.x / kRowLanes; a < na; a += rows) {
        for (int k = part; k < nz; k += kRowLanes) {
            const double x = oct[(size_t)a * d + k];
            if (pass == 0) {
                acc += x;
            } else {
                const double t = x - mu;
                acc += t * t;
            }
        }
    }
    const double sum = block_sum(acc, red[1]);
    if (threadIdx.x == 0) partial[blockIdx.x] = sum;
}

// Both masks and the masked depth mean.  The FP64 thresholds are compared as the
// float32 values that part the samples alike: r < t if r < the least float not
// below t, s > t if s > the largest not above it.  500 x 500 x 465, 1.4 GB: 234 us
// (362 with a wave to an A-scan and 16-byte loads for whole multiples of 4 only).
__global__ __launch_bounds__(256) void k_mask_mean(const float* __restrict__ filt, const float* __restrict__ oct,
                                                   const float* __restrict__ octa, unsigned na, int d,
                                                   const SelState* __restrict__ st, double* __restrict__ E,
                                                   int* __restrict__ cnt)
{
    const float thr_r = __double2float_ru(st->thr_r), thr_s = __double2float_rd(st->thr_s);
    const int part = threadIdx.x & (kRowLanes - 1);
    const unsigned a = blockIdx.x * (blockDim.x / kRowLanes) + threadIdx.x / kRowLanes;
    if (a >= na) return;  // whole rows; the sums below stay within one
    const size_t o = (size_t)a * d;
    double acc = 0.0;
    int c = 0;
    constexpr int kLoads = kRowLoads / 2;  // of three volumes each
    for (int k0 = 0; k0 < d; k0 += kLoads * kRowStep) {
        Quad r[kLoads], s[kLoads], v[kLoads];
#pragma unroll
        for (int g = 0; g < kLoads; ++g) {
            const int k = k0 + g * kRowStep;
            if (k >= d) break;
            r[g] = load_quad(filt + o, k + 4 * part, d);
            s[g] = load_quad(oct + o, k + 4 * part, d);
            v[g] = load_quad(octa + o, k + 4 * part, d);
        }
#pragma unroll
        for (int g = 0; g < kLoads; ++g) {
            if (k0 + g * kRowStep >= d) break;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const bool m = e >= r[g].first && r[g].v[e] < thr_r && s[g].v[e] > thr_s;
                acc += (double)(m ? v[g].v[e] : 0.0f);
                c += m;
            }
        }
    }
    acc = row_sum(acc);
    c = row_sum(c);
    if (part == 0) {
        E[a] = c ? acc / c : 0.0;
        if (cnt) cnt[a] = c;
    }
}

// Median of each B-scan's en face values (the mean of the two middle ones
// for an even count): bitonic sort in LDS, one block per B-scan.
__global__ __launch_bounds__(512) void k_bscan_median(const double* __restrict__ E, int w, int h, int V,
                                                      double* __restrict__ med)
{
    __shared__ double s[kMaxBscan];
    const int b = blockIdx.x;
    const int na = V == 0 ? w : h;
    int P = 1;
    while (P < na) P <<= 1;
    for (int t = threadIdx.x; t < P; t += blockDim.x)
        s[t] = t < na ? (V == 0 ? E[(size_t)b * w + t] : E[(size_t)t * w + b]) : __builtin_inf();
    __syncthreads();
    for (int k = 2; k <= P; k <<= 1) {
        for (int jj = k >> 1; jj > 0; jj >>= 1) {
            for (int t = threadIdx.x; t < P; t += blockDim.x) {
                const int u = t ^ jj;
                if (u > t) {
                    const double x = s[t], y = s[u];
                    const bool up = (t & k) == 0;
                    if ((x > y) == up) {
                        s[t] = y;
                        s[u] = x;
                    }
                }
            }
            __syncthreads();
        }
    }
    if (threadIdx.x == 0) med[b] = (na & 1) ? s[na / 2] : 0.5 * (s[na / 2 - 1] + s[na / 2]);
}

__global__ void k_enface_finish(const double* __restrict__ E, const double* __restrict__ med,
                                const int* __restrict__ from, int w, int h, int V, float* __restrict__ out)
{
    const size_t a = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (a >= (size_t)w * h) return;
    const int i = (int)(a % w), j = (int)(a / w);
    const int b = V == 0 ? j : i;
    const int src = from[b];
    const size_t sa = V == 0 ? (size_t)src * w + i : (size_t)j * w + src;
    out[a] = (float)(E[sa] - med[src]);
}

__global__ void k_fill_ones(float* __restrict__ p, size_t n)
{
    const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) p[t] = 1.0f;
}

// Positions of one wave's walk along an axis of n, a multiple of 15: the axis in
// equal parts, as long as the walks reach `want` waves (the chip filled) and at
// most `longest` (the first 15 positions of a walk are work done twice, the last
// waves of long ones leave the chip idle), and at least 30.  Measured, median and
// fast rank filter / slow one in us: 250 x 250 x 300, 30 long 83 / 57, 60 80 / 48,
// 105 74 / 50 (120), 180 - / 58; 64 x 64 x 128, 30 13.6 / 13.2, 60 17.5 / 17.6, 105
// 23 / 24; the slow one at 500 x 500 x 465, 120 347, 180 324, 255 333.
int walk_length(int n, int lines, int want, int longest)
{
    const int parts = std::max((n + longest - 1) / longest, std::min((n + 29) / 30, (want + lines - 1) / lines));
    return (n + 15 * parts - 1) / (15 * parts) * 15;
}

// Blocks of a radix pass: each clears and adds its histograms, so four A-scans a
// row of lanes if that leaves a block per CU.  Measured with 1 / 2 / 4 / 8: 62 500
// A-scans of 300 35 / 34 / 25 / 28 us, 14 400 of 200 15 / 12 / 12 / 16, 4096 of
// 128 6.2 / 6.3 / 7.8 / 12.4.
unsigned hist_blocks(size_t na)
{
    constexpr size_t rows = 256 / kRowLanes;
    const size_t most = std::min<size_t>((na + rows - 1) / rows, kHistBlocks);
    return (unsigned)std::min(std::max<size_t>(na / (4 * rows), 256), most);
}

inline size_t al(size_t b) { return (b + 255) & ~(size_t)255; }

}  // namespace

size_t enface_scratch_bytes(int w, int h, int d)
{
    const size_t na = (size_t)w * h, nv = na * d, nb = (size_t)(w > h ? w : h);
    return 2 * al(nv * 4) + al(na * 8) + al(na * 4) + al(nb * 8) + al(nb * 4) + al(nb * 4) +
           al(4 * kHistBins * 4) + al(sizeof(SelState)) + al(2 * kNoiseBlocks * 8);
}

int enface_max_bscan() { return kMaxBscan; }

hipError_t launch_enface_project(const float* oct, const float* octa, int w, int h, int d, int V,
                                 const float* valid, const double* fixed, float* out, int* count, double* stats_host,
                                 void* scratch, hipStream_t s)
{
    const size_t na = (size_t)w * h, nv = na * d, nb = (size_t)(V == 0 ? h : w), nbm = (size_t)(w > h ? w : h);
    char* p = static_cast<char*>(scratch);
    auto take = [&](size_t bytes) {
        char* q = p;
        p += al(bytes);
        return q;
    };
    float* v0 = (float*)take(nv * 4);
    float* v1 = (float*)take(nv * 4);
    double* E = (double*)take(na * 8);
    int* cnt = (int*)take(na * 4);
    double* med = (double*)take(nbm * 8);
    int* from = (int*)take(nbm * 4);
    float* vd = (float*)take(nbm * 4);
    unsigned* hist = (unsigned*)take(4 * kHistBins * 4);
    SelState* st = (SelState*)take(sizeof(SelState));
    double* part = (double*)take(2 * kNoiseBlocks * 8);
    if (!valid) {
        hipLaunchKernelGGL(k_fill_ones, dim3((unsigned)((nb + 255) / 256)), dim3(256), 0, s, vd, nb);
        valid = vd;
    }
    hipLaunchKernelGGL(k_enface_init, dim3(1), dim3(256), 0, s, valid, (int)nb, from, st, hist);
    // filtering; the slow-axis pass also counts the first radix digit
    const int fast = V == 0 ? 0 : 1, slow = 1 - fast, ktiles = (d + 63) / 64;
    {
        const int n = fast == 0 ? w : h, lines = fast == 0 ? h : w, mtiles = (d + kMedTile - 1) / kMedTile;
        const size_t row = (size_t)w * d;
        const int seg = walk_length(n, lines * mtiles, 3072, 105);
        hipLaunchKernelGGL(k_median_rank, dim3(mtiles, (n + seg - 1) / seg, (lines + 3) / 4), dim3(256), 0, s, octa,
                           v1, n, lines, fast == 0 ? (size_t)d : row, fast == 0 ? row : (size_t)d, d, seg);
    }
    const int rlen = walk_length((int)nb, (int)(na / nb) * ktiles, 6144, 180);
    const dim3 gr(((unsigned)(na / nb) * ktiles * ((nb + rlen - 1) / rlen) + 3) / 4);
    // OCT noise: the partial sums that the threshold is formed from with the percentiles
    const int nz = (int)floor(0.05 * d + 0.5) < 1 ? 1 : (int)floor(0.05 * d + 0.5);
    const int nb_noise = (int)std::min<size_t>((na + 15) / 16, kNoiseBlocks);
    const NoiseSums noise{part, nb_noise, (double)na * nz};
    for (int pass = 0; pass < 2; ++pass)
        hipLaunchKernelGGL(k_noise_sum, dim3(nb_noise), dim3(256), 0, s, oct, (unsigned)na, d, nz, pass, noise,
                           part + pass * nb_noise);
    if (fixed) {
        hipLaunchKernelGGL(k_rank15<false>, gr, dim3(256), 0, s, v1, v0, w, h, d, slow, rlen,
                           valid, st, hist);
        hipLaunchKernelGGL(k_set_fixed, dim3(1), dim3(256), 0, s, st, fixed[0], fixed[1], noise);
    } else {
        hipLaunchKernelGGL(k_rank15<true>, gr, dim3(256), 0, s, v1, v0, w, h, d, slow, rlen,
                           valid, st, hist);
        hipLaunchKernelGGL(k_radix_select, dim3(1), dim3(256), 0, s, hist, st, 0, noise);
        for (int pass = 1; pass < 3; ++pass) {
            hipLaunchKernelGGL(k_radix_hist, dim3(hist_blocks(na)), dim3(256), 0, s, v0, w, h, d, V, valid, st, pass,
                               hist);
            hipLaunchKernelGGL(k_radix_select, dim3(1), dim3(256), 0, s, hist, st, pass, noise);
        }
    }
    // masks, depth mean, B-scan median, substitution
    hipLaunchKernelGGL(k_mask_mean, dim3((unsigned)((na + 15) / 16)), dim3(256), 0, s, v0, oct, octa, (unsigned)na, d,
                       st, E, count ? count : cnt);
    hipLaunchKernelGGL(k_bscan_median, dim3((unsigned)nb), dim3(512), 0, s, E, w, h, V, med);
    hipLaunchKernelGGL(k_enface_finish, dim3((unsigned)((na + 255) / 256)), dim3(256), 0, s, E, med, from, w, h, V,
                       out);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && stats_host) e = hipMemcpyAsync(stats_host, &st->p5, 3 * 8, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess && stats_host) e = hipMemcpyAsync(stats_host + 3, &st->thr_s, 8, hipMemcpyDeviceToHost, s);
    return e;
}

}  // namespace octmc
