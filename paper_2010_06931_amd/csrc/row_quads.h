// Reading A-scans by 16-byte loads at any depth and alignment (device code).
#pragma once
#include <hip/hip_runtime.h>

namespace octmc {
namespace {

// Sixteen lanes take an A-scan and a lane four consecutive samples of it at a
// time, with one 16-byte load (4-byte alignment costs nothing), so that every
// depth and alignment is read at the same rate; the loads of kRowLoads steps are
// issued together.  (Left to an unrolled loop they are not: its remainder, one
// load at a time, is where all of an A-scan falls.  A radix pass of the en face
// projection, 465 MB, took 193 us so and 110 with the loads together.)
typedef float quad_t __attribute__((ext_vector_type(4), aligned(4)));

struct Quad {
    quad_t v;
    int first;  // the samples `first`.. 3 belong to this lane
};
// samples k .. k + 3 of a column of d; beyond its end, the last four from their
// place on
__device__ __forceinline__ Quad load_quad(const float* __restrict__ col, int k, int d)
{
    Quad q;
    if (d >= 4) {  // uniform
        const int at = k < d - 4 ? k : d - 4;
        q.v = *reinterpret_cast<const quad_t*>(col + at);
        q.first = k < d ? k - at : 4;
    } else {
        // the first d places hold nothing; their samples end at place 3
#pragma unroll
        for (int e = 0; e < 4; ++e) q.v[e] = col[e - (4 - d) < 0 ? 0 : e - (4 - d)];
        q.first = k < d ? 4 - d + k : 4;
    }
    return q;
}
constexpr int kRowLanes = 16;            // lanes of an A-scan
constexpr int kRowStep = 4 * kRowLanes;  // samples they take at a time
constexpr int kRowLoads = 8;             // of these steps are in flight together

// Sum over the sixteen lanes of an A-scan; every lane gets it.
__device__ __forceinline__ double row_sum(double v)
{
#pragma unroll
    for (int m = kRowLanes / 2; m > 0; m >>= 1) v += __shfl_xor(v, m);
    return v;
}
__device__ __forceinline__ int row_sum(int v)
{
#pragma unroll
    for (int m = kRowLanes / 2; m > 0; m >>= 1) v += __shfl_xor(v, m);
    return v;
}
}  // namespace
}  // namespace octmc
