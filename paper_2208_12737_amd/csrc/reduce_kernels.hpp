// Streaming reductions and elementwise kernels around the renderer:
// per-pose sums of tile partials, the stored-Jacobian pose gradient, the
// ZNCC moments / loss / image gradient, and the momentum pose update.
// Every reduction has a fixed summation order (no atomics), so results are
// bitwise reproducible and independent of what else is in the batch.
#pragma once

#include "reduce_common.hpp"

namespace drr {

constexpr int kChunkPixels = 1024;   // pixels per workgroup in streaming kernels

// Sums partials[b][0..n)[0..NS) over the middle index for pose b = blockIdx.x
// into lds row 0, in a fixed order.
template <int NS>
__device__ inline void sum_partials(const double* __restrict__ partials, int n, double* lds)
{
    sum_tile_partials<NS>(partials + (int64_t)blockIdx.x * n * NS, n, lds);
}

// grad_pose[b][j] = sum of partials (7 values per tile).
__global__ __launch_bounds__(kReduceThreads) void k_grad_finalize(const double* partials, int n,
                                                                  float* grad_pose)
{
    __shared__ double lds[kReduceThreads * 7];
    sum_partials<7>(partials, n, lds);
    if ((int)threadIdx.x < 7) grad_pose[blockIdx.x * 7 + threadIdx.x] = (float)lds[threadIdx.x];
}

// Loss and pose gradient of -ZNCC from the fused tile sums.
//   Z = cov(I, T) / (std I std T), loss = -Z
//   d loss / d pose = -1/(N std I) [ (S_TJ - mean T S_J) / std T
//                                    - Z (S_IJ - mean I S_J) / std I ]
__global__ __launch_bounds__(kReduceThreads) void k_ncc_grad_finalize(const double* partials,
                                                                      int n, double npix,
                                                                      float* loss,
                                                                      float* grad_pose)
{
    __shared__ double lds[kReduceThreads * kNccSums];
    sum_partials<kNccSums>(partials, n, lds);
    ncc_from_sums(lds, npix, loss + blockIdx.x, grad_pose + blockIdx.x * 7);
}

// Loss only, from fused tile sums (I, I^2, T, T^2, IT): loss[b] = -Z.
__global__ __launch_bounds__(kReduceThreads) void k_ncc_loss_finalize(const double* partials,
                                                                      int n, double npix,
                                                                      float* loss)
{
    __shared__ double lds[kReduceThreads * 5];
    sum_partials<5>(partials, n, lds);
    if (threadIdx.x == 0) {
        const double* S = lds;
        const double mi = S[0] / npix, mt = S[2] / npix;
        const double si = sqrt(fmax(S[1] / npix - mi * mi, 0.0));
        const double st = sqrt(fmax(S[3] / npix - mt * mt, 0.0));
        loss[blockIdx.x] = (float)(-(S[4] / npix - mi * mt) / (si * st));
    }
}

// Mean squared difference and its pose gradient from the fused tile sums
// ((I-T)^2 and, with NS = 8, (I-T) J[7]):
//   loss = S_0 / N,  d loss / d pose_j = 2 S_{1+j} / N.
template <int NS>
__global__ __launch_bounds__(kReduceThreads) void k_l2_finalize(const double* partials, int n,
                                                                double npix, float* loss,
                                                                float* grad_pose)
{
    __shared__ double lds[kReduceThreads * NS];
    sum_partials<NS>(partials, n, lds);
    const int j = threadIdx.x;
    if (j == 0) loss[blockIdx.x] = (float)(lds[0] / npix);
    if (NS == 8 && j < 7) grad_pose[blockIdx.x * 7 + j] = (float)(2.0 * lds[1 + j] / npix);
}

// Stored-Jacobian contraction: partial[b][chunk][j] = sum g * jac over the chunk.
__global__ __launch_bounds__(kReduceThreads) void k_jac_dot(const float* __restrict__ jac,
                                                            const float* __restrict__ g,
                                                            int64_t hw, int chunks,
                                                            double* partials)
{
    __shared__ double lds[7 * (kReduceThreads / 64)];
    const int b = blockIdx.y, c = blockIdx.x;
    const int64_t p0 = (int64_t)c * kChunkPixels;
    double vals[7];
#pragma unroll
    for (int j = 0; j < 7; ++j) vals[j] = 0.0;
    for (int k = 0; k < kChunkPixels / kReduceThreads; ++k) {
        const int64_t p = p0 + k * kReduceThreads + threadIdx.x;
        if (p < hw) {
            const double gv = g[(int64_t)b * hw + p];
            const float* jp = jac + ((int64_t)b * hw + p) * 7;
#pragma unroll
            for (int j = 0; j < 7; ++j) vals[j] += gv * (double)jp[j];
        }
    }
    block_sums<7, kReduceThreads / 64, 1>(vals, lds, partials + ((int64_t)b * chunks + c) * 7);
}

// ZNCC moments per chunk: sum I, I^2, T, T^2, I T.
__global__ __launch_bounds__(kReduceThreads) void k_ncc_moments(const float* __restrict__ img,
                                                                const float* __restrict__ tgt,
                                                                int64_t tstride, int64_t hw,
                                                                int chunks, double* partials)
{
    __shared__ double lds[5 * (kReduceThreads / 64)];
    const int b = blockIdx.y, c = blockIdx.x;
    const int64_t p0 = (int64_t)c * kChunkPixels;
    double vals[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    for (int k = 0; k < kChunkPixels / kReduceThreads; ++k) {
        const int64_t p = p0 + k * kReduceThreads + threadIdx.x;
        if (p < hw) {
            const double I = img[(int64_t)b * hw + p];
            const double T = tgt[(int64_t)b * tstride + p];
            vals[0] += I;
            vals[1] += I * I;
            vals[2] += T;
            vals[3] += T * T;
            vals[4] += I * T;
        }
    }
    block_sums<5, kReduceThreads / 64, 1>(vals, lds, partials + ((int64_t)b * chunks + c) * 5);
}

// stats[b] = (mean I, std I, mean T, std T, Z); loss[b] = -Z.
__global__ __launch_bounds__(kReduceThreads) void k_ncc_stats(const double* partials, int n,
                                                              double npix, double* stats,
                                                              float* loss)
{
    __shared__ double lds[kReduceThreads * 5];
    sum_partials<5>(partials, n, lds);
    if (threadIdx.x == 0) {
        const double* S = lds;
        const double mi = S[0] / npix, mt = S[2] / npix;
        const double si = sqrt(fmax(S[1] / npix - mi * mi, 0.0));
        const double st = sqrt(fmax(S[3] / npix - mt * mt, 0.0));
        const double z = (S[4] / npix - mi * mt) / (si * st);
        double* o = stats + (int64_t)blockIdx.x * 5;
        o[0] = mi;
        o[1] = si;
        o[2] = mt;
        o[3] = st;
        o[4] = z;
        loss[blockIdx.x] = (float)(-z);
    }
}

// grad_image = grad_loss * d(-Z)/dI = -grad_loss (That - Z Ihat) / (N std I).
__global__ __launch_bounds__(kReduceThreads) void k_ncc_backward(
    const float* __restrict__ img, const float* __restrict__ tgt, int64_t tstride,
    const double* __restrict__ stats, const float* __restrict__ gl, int64_t hw, double npix,
    float* __restrict__ out)
{
    const int b = blockIdx.y;
    const int64_t p = (int64_t)blockIdx.x * kReduceThreads + threadIdx.x;
    if (p >= hw) return;
    const double* st = stats + (int64_t)b * 5;
    const double ih = ((double)img[(int64_t)b * hw + p] - st[0]) / st[1];
    const double th = ((double)tgt[(int64_t)b * tstride + p] - st[2]) / st[3];
    out[(int64_t)b * hw + p] = (float)(-(double)gl[b] * (th - st[4] * ih) / (npix * st[1]));
}

// Heavy-ball step: v <- m v + g; pose <- pose - rate .* v.
__global__ void k_momentum(float* __restrict__ poses, float* __restrict__ vel,
                           const float* __restrict__ grad, const float* __restrict__ rate,
                           float m, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float v = m * vel[i] + grad[i];
    vel[i] = v;
    poses[i] = poses[i] - rate[i] * v;
}

// Copies a C-order volume into one zero-bordered copy whose memory order is
// (o0 slowest, o1, o2 fastest) over the padded dims P.
__global__ void k_pack(const float* __restrict__ src, float* __restrict__ dst, int nx, int ny,
                       int nz, int o0, int o1, int o2, uint64_t total)
{
    const uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= total) return;
    const uint64_t P[3] = {(uint64_t)nx + 2, (uint64_t)ny + 2, (uint64_t)nz + 2};
    uint64_t idx[3];
    idx[o2] = e % P[o2];
    idx[o1] = (e / P[o2]) % P[o1];
    idx[o0] = e / (P[o2] * P[o1]);
    const int i = (int)idx[0], j = (int)idx[1], k = (int)idx[2];
    float v = 0.0f;
    if (i >= 1 && i <= nx && j >= 1 && j <= ny && k >= 1 && k <= nz)
        v = src[((uint64_t)(i - 1) * ny + (j - 1)) * nz + (k - 1)];
    dst[e] = v;
}

// ------------------------------------------------------------------ crossing tables

// The largest jump must stay below 2^31 quanta after the rounding of two sums.
constexpr double kRunMost = 2147483640.0;

__global__ void k_run_clear(RunHeader* h)
{
    if (threadIdx.x < 3) {
        h->quantum[threadIdx.x] = 0.0;
        h->most[threadIdx.x] = 0ull;
    }
    if (threadIdx.x == 0) {
        h->sum_abs = 0.0;
        h->use = 0;
    }
}

// Quantum of each axis, and whether the tables may be used: an ordinary
// ray's error is a few quanta, which 2^-26 of the mean column sum keeps below
// the rounding of its FP32 pixel.  (False for sums that are not finite.)
__global__ void k_run_quanta(RunHeader* h, int nx, int ny, int nz)
{
    if (threadIdx.x != 0) return;
    const int n[3] = {nx, ny, nz};
    const double mean = h->sum_abs / ((double)nx * (double)ny * (double)nz);
    bool use = true;
    for (int q = 0; q < 3; ++q) {
        const double most = __longlong_as_double((long long)h->most[q]);
        const double quantum = most / kRunMost;
        h->quantum[q] = quantum;
        use = use && quantum > 0.0 && quantum <= 0x1p-26 * mean * (double)n[q];
    }
    h->use = use ? 1 : 0;
}

// Running sums along axis q of a strip of columns, neighbours along axis a,
// at one column c of axis b.  A workgroup takes the columns k0 - 1 .. k0 + 63
// (those outside the grid sum to 0), stages 32 voxels of each through LDS and
// lets one lane a column add them up in order; the jumps across the planes
// k0 .. k0 + 63 are differences of neighbouring lanes' sums.
//   PASS 0  ends[column] = {-total / 2, total / 2}, and the sum of |V|
//   PASS 1  the largest jump
//   PASS 2  the table; the end sums in quanta
// Sums run from -total / 2, rounded to quanta (PASS 2): entries of row (k, c)
// are the jumps before voxel i - 1 of q, i = 0 .. n + 2, held at both ends.
// Set-up once a volume: 2.0 ms for the 512 x 512 x 133 CT.
constexpr int kRunCols = 64, kRunStage = 32;

template <int PASS>
__global__ __launch_bounds__(256) void k_run_scan(const float* __restrict__ src, RunHeader* h,
                                                  int q, double2* ends, bool keep_end,
                                                  int* __restrict__ table, int na, int nb, int nq,
                                                  int64_t sa, int64_t sb, int64_t sq,
                                                  int64_t ea, int64_t eb)
{
    __shared__ float vox[kRunCols + 1][kRunStage + 1];
    __shared__ double sum[kRunCols + 1][kRunStage + 1];
    const int tid = threadIdx.x, c = blockIdx.x, k0 = (int)blockIdx.y * kRunCols;
    // column j of the strip is cell k0 - 1 + j of axis a
    auto cell = [&](int j) { return k0 - 1 + j; };
    const bool column = tid <= kRunCols && cell(tid) >= 0 && cell(tid) < na;
    // (a NaN stays)
    auto larger = [](double a, double b) { return (b > a || b != b) ? b : a; };
    double inv = 0.0, acc = 0.0, absolute = 0.0, most = 0.0;
    if (PASS == 2 && h->use == 0) return;   // the tables are not read
    if (PASS == 2) inv = 1.0 / h->quantum[q];
    const double2* end = ends + (int64_t)cell(tid) * ea + (int64_t)c * eb;
    if (PASS > 0 && column) acc = end->x;
    // (fetching along whichever of a and q is contiguous in the source)
    const bool along_q = sq == 1;
    for (int m0 = 0; m0 <= nq; m0 += kRunStage) {
        for (int e = tid; e < (kRunCols + 1) * kRunStage; e += 256) {
            const int j = along_q ? e / kRunStage : e % (kRunCols + 1);
            const int m = along_q ? e % kRunStage : e / (kRunCols + 1);
            const int a = cell(j), i = m0 + m;
            vox[j][m] = (a >= 0 && a < na && i < nq)
                            ? src[(int64_t)a * sa + (int64_t)c * sb + (int64_t)i * sq]
                            : 0.0f;
        }
        __syncthreads();
        if (tid <= kRunCols) {
            for (int m = 0; m < kRunStage; ++m) {
                sum[tid][m] = PASS == 2 ? rint(acc * inv) : acc;
                const double x = (double)vox[tid][m];
                if (column) acc += x;
                if (PASS == 0 && column && tid > 0) absolute += fabs(x);
            }
        }
        __syncthreads();
        if (PASS > 0) {
            for (int e = tid; e < kRunCols * kRunStage; e += 256) {
                const int j = e / kRunStage, m = e % kRunStage;
                const int k = k0 + j, i = m0 + m;
                if (k > na || i > nq) continue;
                const double jump = sum[j][m] - sum[j + 1][m];
                if (PASS == 1) most = larger(most, fabs(jump));
                if (PASS == 2) {
                    int* row = table + ((int64_t)k * nb + c) * (nq + kRunPad);
                    row[i + 1] = (int)jump;
                    if (i == 0) row[0] = (int)jump;
                    if (i == nq) row[nq + 2] = (int)jump;
                }
            }
            __syncthreads();
        }
    }
    double2* out = ends + (int64_t)cell(tid) * ea + (int64_t)c * eb;
    if (PASS == 0) {
        if (column && tid > 0) *out = make_double2(-0.5 * acc, 0.5 * acc);
        const double s = wave_sum(absolute);
        if ((tid & 63) == 0) atomicAdd(&h->sum_abs, s);
    }
    if (PASS == 1) {
        // the sum at the end as the tables' scans reach it (only .x is read
        // by other workgroups)
        if (keep_end && column && tid > 0) out->y = acc;
        for (int o = 32; o >= 1; o >>= 1) most = larger(most, __shfl_xor(most, o, 64));
        if ((tid & 63) == 0)
            atomicMax(&h->most[q], (unsigned long long)__double_as_longlong(fabs(most)));
    }
}

// The columns' end sums in quanta, as the tables' sums are rounded.
__global__ __launch_bounds__(256) void k_run_ends(const RunHeader* h, int q, double2* ends,
                                                  int64_t count)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= count || h->use == 0) return;
    const double inv = 1.0 / h->quantum[q];
    const double2 e = ends[i];
    ends[i] = make_double2(rint(e.x * inv), rint(e.y * inv));
}

}  // namespace drr
