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
__global__ __launch_bounds__(final_threads<7>()) void k_grad_finalize(const double* partials, int n,
                                                                  float* grad_pose)
{
    __shared__ double lds[final_parts<7>() * 7];
    sum_partials<7>(partials, n, lds);
    if ((int)threadIdx.x < 7) grad_pose[blockIdx.x * 7 + threadIdx.x] = (float)lds[threadIdx.x];
}

// Loss and pose gradient of -ZNCC from the fused tile sums.
//   Z = cov(I, T) / (std I std T), loss = -Z
//   d loss / d pose = -1/(N std I) [ (S_TJ - mean T S_J) / std T
//                                    - Z (S_IJ - mean I S_J) / std I ]
__global__ __launch_bounds__(final_threads<kNccSums>()) void k_ncc_grad_finalize(const double* partials,
                                                                      int n, double npix,
                                                                      float* loss,
                                                                      float* grad_pose)
{
    __shared__ double lds[final_parts<kNccSums>() * kNccSums];
    sum_partials<kNccSums>(partials, n, lds);
    ncc_from_sums(lds, npix, loss + blockIdx.x, grad_pose + blockIdx.x * 7);
}

// Loss only, from fused tile sums (I, I^2, T, T^2, IT): loss[b] = -Z.
__global__ __launch_bounds__(final_threads<5>()) void k_ncc_loss_finalize(const double* partials,
                                                                      int n, double npix,
                                                                      float* loss)
{
    __shared__ double lds[final_parts<5>() * 5];
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
__global__ __launch_bounds__(final_threads<NS>()) void k_l2_finalize(const double* partials, int n,
                                                                double npix, float* loss,
                                                                float* grad_pose)
{
    __shared__ double lds[final_parts<NS>() * NS];
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
__global__ __launch_bounds__(final_threads<5>()) void k_ncc_stats(const double* partials, int n,
                                                              double npix, double* stats,
                                                              float* loss)
{
    __shared__ double lds[final_parts<5>() * 5];
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

// Copies a C-order volume into one zero-bordered copy of the padded dims P
// whose memory order is o0 slowest, o1, o2 fastest: tiles of 32 x 32 over o2
// and z, read along z and written along o2 through LDS (o2 = z: as they are),
// one padded index of the third axis a workgroup.  Bound by its reads and
// writes: 101..126 us a copy of the 512 x 512 x 133 CT (279 MB), 205 us as one
// thread a voxel that reads across z.
constexpr int kPackTile = 32;

__global__ __launch_bounds__(256) void k_pack(const float* __restrict__ src,
                                              float* __restrict__ dst, int nx, int ny, int nz,
                                              int o0, int o1, int o2)
{
    __shared__ float tile[kPackTile][kPackTile + 1];
    const int n[3] = {nx, ny, nz};
    const int f = o2 == 2 ? 1 : o2;             // the axis of the tile beside z
    const int g = f == 0 ? 1 : 0;               // the third
    const int nf = f == 0 ? nx : ny;
    const uint32_t tz = (uint32_t)(nz + 1) / kPackTile + 1, tf = (uint32_t)(nf + 1) / kPackTile + 1;
    const int z0 = (int)(blockIdx.x % tz) * kPackTile, f0 = (int)(blockIdx.x / tz % tf) * kPackTile;
    const int ig = (int)(blockIdx.x / tz / tf), ng = g == 0 ? nx : ny;
    const int lane = threadIdx.x % kPackTile, line = threadIdx.x / kPackTile;
    const int64_t sf = f == 0 ? (int64_t)ny * nz : nz, sg = g == 0 ? (int64_t)ny * nz : nz;
    // pitches of the copy
    int64_t pitch_z = 0, pitch_f = 0, pitch_g = 0, at = 1;
    for (int k = 2; k >= 0; --k) {
        const int axis = k == 2 ? o2 : (k == 1 ? o1 : o0);
        if (axis == 2) pitch_z = at;
        else if (axis == f) pitch_f = at;
        else pitch_g = at;
        at *= (axis == 0 ? n[0] : (axis == 1 ? n[1] : n[2])) + 2;
    }
    // padded indices; voxel i of an axis is at i + 1
    auto voxel = [&](int pf, int pz) {
        const bool in = pf >= 1 && pf <= nf && pz >= 1 && pz <= nz && ig >= 1 && ig <= ng;
        return in ? src[(pf - 1) * sf + (ig - 1) * sg + (pz - 1)] : 0.0f;
    };
    if (o2 == 2) {
        for (int r = line; r < kPackTile; r += 8) {
            const int pf = f0 + r, pz = z0 + lane;
            if (pf < nf + 2 && pz < nz + 2) dst[pf * pitch_f + ig * pitch_g + pz] = voxel(pf, pz);
        }
        return;
    }
    for (int r = line; r < kPackTile; r += 8) tile[r][lane] = voxel(f0 + r, z0 + lane);
    __syncthreads();
    for (int r = line; r < kPackTile; r += 8) {
        const int pf = f0 + lane, pz = z0 + r;
        if (pf < nf + 2 && pz < nz + 2)
            dst[pf * pitch_f + ig * pitch_g + pz * pitch_z] = tile[lane][r];
    }
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
        use = use && quantum > 0.0 && isfinite(quantum) &&
              quantum <= 0x1p-26 * mean * (double)n[q];
    }
    h->use = use ? 1 : 0;
}

// Running sums along axis q and their jumps across the planes of axis a.
// Lanes are neighbours along whichever axis the source is contiguous in:
//   ALONG_B  along b: a lane adds up both columns of its plane
//   else     along a (or each along its own row of q): a lane adds up one
//            column, and the jumps of 63 planes are differences of
//            neighbouring lanes' sums
//   MEASURE  (!FILL) the largest jump of sums taken from the middle of the
//            columns' totals (from the extremes and the end of the jumps of
//            the plain sums); with `first`, the totals and, for q = 0, the
//            sum of |V|
//   FILL     the table, of sums from -total / 2 rounded to quanta: entries i
//            = 0 .. n + 2 of row (k, c) are the jumps before voxel i - 1 of q,
//            held at both ends; with `first`, the sums at the ends
// Columns outside the grid sum to 0.  Bound by the latency of its reads (some
// 1500 waves), so 16 voxels are read ahead of the 16 being summed; rows are
// written four entries at a time.  A table of the 512 x 512 x 133 CT measures
// in 88..119 us and fills in 149..216 us (139 MB read, as much written).
// Lanes always along a: 350 and 490 us with b the contiguous axis, all twelve
// passes 2.9 ms for 1.7.
constexpr int kRunStrip = 63, kRunAhead = 16;
typedef float run_f4 __attribute__((ext_vector_type(4), aligned(4)));
typedef int run_i4 __attribute__((ext_vector_type(4), aligned(4)));

template <bool FILL, bool ALONG_B>
__global__ __launch_bounds__(256) void k_run_scan(const float* __restrict__ src, RunHeader* h,
                                                  int q, bool first, double2* ends,
                                                  int* __restrict__ table, int na, int nb, int nq,
                                                  int64_t sa, int64_t sb, int64_t sq, int64_t ea,
                                                  int64_t eb)
{
    if (FILL && h->use == 0) return;   // the tables are not read
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // the lane's column `cell` (above its plane) at c; four neighbouring
    // waves a workgroup
    int c, cell;
    bool plane;
    if (ALONG_B) {
        c = (int)blockIdx.x * 64 + lane;
        cell = (int)blockIdx.y * 4 + wave;
        plane = c < nb && cell <= na;
    } else {
        c = (int)blockIdx.x * 4 + wave;
        if (c >= nb) return;
        cell = (int)blockIdx.y * kRunStrip - 1 + lane;
        plane = lane >= 1 && cell <= na;
    }
    const bool column = c < nb && cell >= 0 && cell < na;
    const bool under = ALONG_B && plane && cell > 0;   // the column below, added up as well
    const float* in = src + (column ? (int64_t)cell * sa + (int64_t)c * sb : 0);
    const float* in2 = src + (under ? (int64_t)(cell - 1) * sa + (int64_t)c * sb : 0);
    double2* end = ends + (column ? (int64_t)cell * ea + (int64_t)c * eb : 0);
    int* row = table + (plane ? ((int64_t)cell * nb + c) * (nq + kRunPad) : 0);
    const double inv = FILL ? 1.0 / h->quantum[q] : 0.0;
    double acc = FILL && column ? end->x : 0.0;
    double acc2 = FILL && under ? ends[(int64_t)(cell - 1) * ea + (int64_t)c * eb].x : 0.0;
    double absolute = 0.0, lo = 0.0, hi = 0.0;
    bool nan = false;
    auto below = [&](double above, double x2) { return ALONG_B ? x2 : __shfl_up(above, 1, 64); };
    float now[kRunAhead], next[kRunAhead], now2[kRunAhead], next2[kRunAhead];
    auto fetch = [&](float* v, const float* p, bool on, int i0) {
        if (!ALONG_B && sq == 1 && i0 + kRunAhead <= nq) {
#pragma unroll
            for (int u = 0; u < kRunAhead; u += 4) {
                const run_f4 x = on ? *(const run_f4*)(p + i0 + u) : run_f4{0.0f, 0.0f, 0.0f, 0.0f};
                v[u] = x.x, v[u + 1] = x.y, v[u + 2] = x.z, v[u + 3] = x.w;
            }
            return;
        }
#pragma unroll
        for (int u = 0; u < kRunAhead; ++u)
            v[u] = on && i0 + u < nq ? p[(int64_t)(i0 + u) * sq] : 0.0f;
    };
    fetch(now, in, column, 0);
    if (ALONG_B) fetch(now2, in2, under, 0);
    int held[4] = {0, 0, 0, 0};
    for (int i0 = 0; i0 <= nq; i0 += kRunAhead) {
        fetch(next, in, column, i0 + kRunAhead);
        if (ALONG_B) fetch(next2, in2, under, i0 + kRunAhead);
#pragma unroll
        for (int u = 0; u < kRunAhead; ++u) {
            const int i = i0 + u;
            const double s = FILL ? rint(acc * inv) : acc;
            const double jump = below(s, FILL ? rint(acc2 * inv) : acc2) - s;
            if (FILL) {
                const int j = (int)jump;
                if (plane && i == 0) row[0] = j;
                held[u & 3] = j;
                // entries i - 2 .. i + 1 of the row
                if ((u & 3) == 3 && plane && i <= nq)
                    *(run_i4*)(row + i - 2) = run_i4{held[0], held[1], held[2], held[3]};
                else if (plane && i <= nq && i + 3 - (u & 3) > nq)
                    row[i + 1] = j;   // the last, incomplete four
                if (plane && i == nq) row[nq + 2] = j;
            } else if (i <= nq) {
                lo = fmin(lo, jump);
                hi = fmax(hi, jump);
                nan = nan || jump != jump;
            }
            if (i < nq) {
                acc += (double)now[u];
                if (ALONG_B) acc2 += (double)now2[u];
                if (!FILL) absolute += fabs((double)now[u]);
            }
        }
#pragma unroll
        for (int u = 0; u < kRunAhead; ++u) {
            now[u] = next[u];
            if (ALONG_B) now2[u] = next2[u];
        }
    }
    const bool owned = column && (ALONG_B || lane > 0);
    if (FILL) {
        // (only .x is read by other waves)
        if (first && owned) end->y = acc;
        return;
    }
    if (first && owned) *end = make_double2(-0.5 * acc, 0.5 * acc);
    const double last = below(acc, acc2) - acc;
    double most = plane ? fmax(hi - 0.5 * last, 0.5 * last - lo) : 0.0;
    if (plane && (nan || most != most)) most = __builtin_nan("");
    for (int o = 32; o >= 1; o >>= 1) {
        const double x = __shfl_xor(most, o, 64);
        most = (x > most || x != x) ? x : most;   // a NaN stays
    }
    if (lane == 0)
        atomicMax(&h->most[q], (unsigned long long)__double_as_longlong(fabs(most)));
    if (first && q == 0) {
        const double s = wave_sum(owned ? absolute : 0.0);
        if (lane == 0) atomicAdd(&h->sum_abs, s);
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
