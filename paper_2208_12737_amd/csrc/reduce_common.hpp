// Device helpers shared by the reduction kernels of the direct entry points
// and of plans: the fixed-order sum of per-tile moment rows and the -ZNCC
// loss and pose gradient computed from the summed moments.
#pragma once

#include "render_kernels.hpp"

namespace drr {

constexpr int kReduceThreads = 256;

// Threads of a workgroup that sums rows of NS values: final_parts<NS> threads
// a value, each for every final_parts-th row, so that the workgroup reads
// neighbouring doubles.  (The 26 sums of 256 rows, 64 poses: 4.5 us; 7.6 us with
// a thread a row, which reads 208 bytes apart, and a tree over 256 threads.)
template <int NS>
constexpr int final_parts()
{
    return 1024 / NS < 64 ? 1024 / NS : 64;
}

template <int NS>
constexpr int final_threads()
{
    return (final_parts<NS>() * NS + 63) / 64 * 64;
}

// Sums base[0..n)[0..NS) over the first index into lds[0..NS) (of final_parts
// * NS doubles), in a fixed order.  Bound by the latency of its reads: four are
// in flight (three steps of 16 registrations at 128 x 128 pixels: 193 us, 199 us
// with eight, most of them past the last row).
template <int NS>
__device__ inline void sum_tile_partials(const double* __restrict__ base, int n, double* lds)
{
    constexpr int P = final_parts<NS>(), AHEAD = 4;
    const int i = threadIdx.x;
    double acc = 0.0;
    if (i < P * NS) {
        const int mine = i / NS;   // rows mine, mine + P, ...
        const double* column = base + i % NS;
        for (int t = mine; t < n; t += AHEAD * P) {
            // (read at a clamped index and then selected: a read under a
            // condition would be waited for before the next)
            double x[AHEAD];
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) x[u] = column[(int64_t)min(t + u * P, n - 1) * NS];
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) acc += t + u * P < n ? x[u] : 0.0;
        }
        lds[i] = acc;
    }
    __syncthreads();
    acc = 0.0;
    if (i < NS)
#pragma unroll 8
        for (int k = 0; k < P; ++k) acc += lds[k * NS + i];
    __syncthreads();
    if (i < NS) lds[i] = acc;
    __syncthreads();
}

// -ZNCC and its pose gradient from the 26 summed tile moments S (threads
// 0..6 write grad[0..6], thread 0 the loss).
__device__ inline void ncc_from_sums(const double* S, double npix, float* loss, float* grad)
{
    if ((int)threadIdx.x < 7) {
        const double mi = S[0] / npix, mt = S[2] / npix;
        const double si = sqrt(fmax(S[1] / npix - mi * mi, 0.0));
        const double st = sqrt(fmax(S[3] / npix - mt * mt, 0.0));
        const double z = (S[4] / npix - mi * mt) / (si * st);
        const int j = threadIdx.x;
        const double tj = (S[12 + j] - mt * S[5 + j]) / st;
        const double ij = (S[19 + j] - mi * S[5 + j]) / si;
        grad[j] = (float)(-(tj - z * ij) / (npix * si));
        if (j == 0) *loss = (float)(-z);
    }
}

}  // namespace drr
