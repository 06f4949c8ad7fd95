// Ray traversal over the jumps of the volume's running sums ("crossing
// tables").
//
// A ray stays in one column of voxels along an axis q between two crossings
// of the planes of the other two axes, so its integral over such a run is a
// difference of the column's running sum at the run's ends.  With
//   S[i] = V[0] + ... + V[i-1] along q, and
//   P(t) = S[i] + (t - i) (S[i+1] - S[i]),  i = floor(t), t in voxels of q,
// the path sum is
//   (dalpha / dt) [ P(end, last column) - P(start, first column)
//                   + sum over the crossings of the other two axes' planes of
//                     P(t, column before) - P(t, column after) ].
// q's own planes drop out: with q the axis whose planes the ray crosses most
// often, some 190 of 690 crossings remain on a 512 x 512 x 133 CT.  Each is a
// term of its own that needs no merge with the others, only its column along
// the third axis, and it needs only the jump D = S(below) - S(above) across
// the plane, which the tables hold: two neighbouring entries D[i], D[i+1],
// one 8-byte read.  Their difference is the jump of the voxel value, which is
// what the Jacobian sums need.
//
// Entries are whole numbers of a quantum, 2^-31 of the largest |D| along q.
// S is rounded to quanta before the jumps are formed, so that the terms of a
// ray cancel exactly where it passes only zeros, and everything after that is
// FP64.  (A column's sums are taken from their middle, which halves D.)  On a
// volume whose largest jump dwarfs an ordinary column's sum the quantum would
// be felt; such a volume, and one with a voxel that is not finite, is marked
// when it is packed and traced by the plane merge of siddon.hpp instead.
//
// The terms telescope only if the order of a crossing of axis a and one of
// axis b is the same seen from both (see planes_passed); at an exact tie b's
// plane comes first.
//
// What bounds it: the bytes that miss the L2.  The rays of a wave cross a
// plane at entries a few voxels apart along q (a neighbouring ray is one
// voxel further along the crossed axis, and the ray needs 1 / slope voxels of
// q to make that up), so the entries along q are neighbours in memory, and
// 4-byte entries run 1.7 times as fast as FP64 ones.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "run_rays.hpp"
#include "siddon.hpp"

namespace drr {

// Crossings whose table entries are read together, and whether the next
// batch is read before the last is summed.
//   RunFull    launches that fill the GPU: eight at a time (an earlier build
//              with all else equal: 4 at a time, pipelined, 256 poses of
//              256 x 256 on the 512 x 512 x 133 CT level, the fused gradient
//              of 64 poses 4% slower)
//   RunWide    the same for the Jacobian modes where two waves a SIMD are
//              resident anyway: 256 registers, nothing kept in memory (the
//              fused gradient of 64 poses: 1.27 ms, 1.36 ms with 128
//              registers; pipelined or with 16 at a time 1.28..1.30 ms; the
//              modes without a Jacobian need no more than 128)
//   RunFew     launches of about a wave per SIMD, which have nothing else to
//              hide a read's latency: pairs of batches (one such DRR: 33 us
//              with eight, 38 us with four, 39-48 us without the pipeline)
//   RunRare    a wave's second direction: small, for its registers (with
//              RunFew, which has any number, as the first: a gradient of three
//              poses of 154 x 119 pixels on 421 x 105 x 125 voxels, a third of
//              its waves mixed, 31.8 us, 38.7 us with RunRare)
template <int UNROLL, bool PIPELINED>
struct RunShape {
    static constexpr int unroll = UNROLL;
    static constexpr bool pipelined = PIPELINED;
};
using RunFull = RunShape<8, false>;
struct RunWide : RunFull {};
using RunFew = RunShape<8, true>;
using RunRare = RunShape<2, true>;

// Byte offset no table reaches: a lane without a crossing reads 0 there.
constexpr uint32_t kRunNone = 0xF0000000u;

typedef uint32_t run_u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t run_u32x4 __attribute__((ext_vector_type(4)));

// D[i] and D[i + 1] - D[i], in quanta.
struct RunPair {
    double jump, step;
};

__device__ inline run_u32x2 run_load(const __amdgpu_buffer_rsrc_t& r, uint32_t off, uint32_t soff)
{
    return __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, (int)soff, 0);
}

__device__ inline RunPair run_pair(run_u32x2 v)
{
    const double a = (double)(int)v.x, b = (double)(int)v.y;
    return {a, b - a};
}

// Minimum over the wave (every lane active), wave-uniform.
__device__ inline int wave_min(int x)
{
    x = min(x, __builtin_amdgcn_update_dpp(x, x, 0x111, 0xf, 0xf, false));   // row_shr:1
    x = min(x, __builtin_amdgcn_update_dpp(x, x, 0x112, 0xf, 0xf, false));   // row_shr:2
    x = min(x, __builtin_amdgcn_update_dpp(x, x, 0x114, 0xf, 0xf, false));   // row_shr:4
    x = min(x, __builtin_amdgcn_update_dpp(x, x, 0x118, 0xf, 0xf, false));   // row_shr:8
    x = min(x, __builtin_amdgcn_update_dpp(x, x, 0x142, 0xa, 0xf, false));   // row_bcast:15
    x = min(x, __builtin_amdgcn_update_dpp(x, x, 0x143, 0xc, 0xf, false));   // row_bcast:31
    return __builtin_amdgcn_readlane(x, 63);
}

// A crossing table: planes of one axis, rows of entries along q.
struct RunTable {
    __amdgpu_buffer_rsrc_t rsrc;
    uint32_t plane;   // bytes between planes
    int row;          // bytes between rows (neighbouring columns of the third axis)
};

// One batch of crossings on its way: the entries read, and where between
// entries (f) and along the ray (alpha) each lies.
template <bool JAC, int U>
struct RunBatch {
    run_u32x2 v[U];
    double f[U];
    double alpha[JAC ? U : 1];
};

// Terms of the crossings lo..hi (ray order, lo > hi: none) of the n + 1
// planes of one axis.  Where the rays of the wave cross much the same planes,
// all take the same plane at the same time and read neighbouring entries of
// it; where the wave's pixels are so many voxels wide that the planes of all
// its rays are a quarter more than one ray's, each ray starts at its own first
// plane.  (Either way a ray's own terms are added in the same order.)
//   tr      the third axis, tr_n columns
//   q1, q0  entry of the row at alpha: fma(alpha, q1, q0)
// acc, A, B: sums of P, V and alpha V below the plane minus above it.
template <bool JAC, bool STRICT, typename S>
__device__ __forceinline__ void run_crossings(const RunTable& T, const RunAxis& dr, int lo, int hi,
                                              int n, const RunAxis& tr, int tr_n, double q1,
                                              double q0, double& acc, double& A, double& B)
{
#pragma clang fp contract(off)
    constexpr int U = S::unroll;
    const int count = lo > hi ? 0 : hi - lo + 1;
    const int most = -wave_min(-count);
    if (most == 0) return;
    const int first = wave_min(count > 0 ? lo : 0x3fffffff);
    const int span = 1 - first - wave_min(count > 0 ? -hi : 0x3fffffff);
    const uint64_t lanes = __builtin_amdgcn_ballot_w64(count > 0),
                   down = __builtin_amdgcn_ballot_w64(count > 0 && dr.neg);
    const bool together = 4 * span <= 5 * most && (down == 0 || down == lanes);
    const int steps = together ? span : most;
    if (count <= 0) return;
    const int start = together ? first : lo;
    uint32_t rel = (uint32_t)(start - lo);   // (wraps: before the lane's first plane)
    double k = (double)start;
    // third axis: with m or m + 1 planes passed the ray is in its column
    // m - 1 or m (ray order)
    const int stride = tr.neg ? -T.row : T.row;
    const int base = tr.neg ? (tr_n - 1) * T.row : 0;
    const int base0 = base - stride;
    const uint32_t step = dr.neg ? 0u - T.plane : T.plane;
    uint32_t at = (uint32_t)(dr.neg ? n - start : start) * T.plane;
    RunBatch<JAC, U> b0, b1;
    auto issue = [&](RunBatch<JAC, U>& b) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const double alpha = fma(k, dr.da, dr.a0);
            const double t = fma(alpha, q1, q0);
            const double m = rint(fma(alpha, tr.c1, tr.c0));
            const double am = fma(m, tr.da, tr.a0);
            const bool past = STRICT ? am < alpha : am <= alpha;
            const int col = __mul24((int)m, stride) + (past ? base : base0);
            const uint32_t off = at + (uint32_t)((int)t * 4 + col);
            b.f[u] = __builtin_amdgcn_fract(t);
            if (JAC) b.alpha[u] = alpha;
            b.v[u] = run_load(T.rsrc, rel < (uint32_t)count ? off : kRunNone, 0);
            k += 1.0;
            rel += 1u;
            at += step;
        }
    };
    auto consume = [&](const RunBatch<JAC, U>& b) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const RunPair e = run_pair(b.v[u]);
            acc += e.jump;
            acc = fma(b.f[u], e.step, acc);
            if (JAC) {
                A += e.step;
                B = fma(b.alpha[u], e.step, B);
            }
        }
    };
    if constexpr (S::pipelined) {
        issue(b0);
        for (int j = 0; j < steps; j += 2 * U) {
            issue(b1);
            consume(b0);
            issue(b0);
            consume(b1);
        }
    } else {
        for (int j = 0; j < steps; j += U) {
            issue(b0);
            consume(b0);
        }
    }
}

// P and V (as a RunPair read at t's entry: jump P, step V) of a column at an
// end on the lowest (plane 0) or highest face of an axis: the sum outside
// the grid is 0.
__device__ inline void run_face(const RunTable& T, bool on, bool upper, int n, uint32_t off,
                                double f, double& P, double& v)
{
    const uint32_t o = on ? off + (upper ? (uint32_t)n * T.plane : 0u) : kRunNone;
    const RunPair e = run_pair(run_load(T.rsrc, o, 0));
    const double p = fma(f, e.step, e.jump);
    P = upper ? p : -p;
    v = upper ? e.step : -e.step;
}

// Members by select: a choice between structs or array elements would be
// taken by address and put them in memory.
__device__ inline RunAxis run_pick(bool first, const RunAxis& x, const RunAxis& y)
{
    return {first ? x.a0 : y.a0, first ? x.da : y.da, first ? x.c1 : y.c1, first ? x.c0 : y.c0,
            first ? x.neg : y.neg};
}

template <typename T>
__device__ inline T run_pick3(int q, T x, T y, T z)
{
    return q == 0 ? x : (q == 1 ? y : z);
}

// Path sum (and the Jacobian sums) of the rays s + alpha d of the lanes with
// `on`, whose runs go along axis q (wave-uniform), into their r.  Every lane
// of the wave calls it.
template <bool JAC, typename S>
__device__ __forceinline__ void trace_along(const VolArgs& V, int q, bool on, const double s[3],
                                            const double d[3], RayAcc& r)
{
#pragma clang fp contract(off)
    // entry and exit (Sec. 2.3), clamped to [0, 1]
    bool miss = false;
    double exit0, exit1, exit2;
    const RunAxis X0 = run_axis(s[0], d[0], V.origin[0], V.spacing[0], V.inv_spacing[0], V.n[0],
                                &exit0, &miss);
    const RunAxis X1 = run_axis(s[1], d[1], V.origin[1], V.spacing[1], V.inv_spacing[1], V.n[1],
                                &exit1, &miss);
    const RunAxis X2 = run_axis(s[2], d[2], V.origin[2], V.spacing[2], V.inv_spacing[2], V.n[2],
                                &exit2, &miss);
    double amin = 0.0, amax = 1.0;
    int amin_ax = -1, amax_ax = -1;
    if (X0.a0 > amin) amin = X0.a0, amin_ax = 0;
    if (X1.a0 > amin) amin = X1.a0, amin_ax = 1;
    if (X2.a0 > amin) amin = X2.a0, amin_ax = 2;
    if (exit0 < amax) amax = exit0, amax_ax = 0;
    if (exit1 < amax) amax = exit1, amax_ax = 1;
    if (exit2 < amax) amax = exit2, amax_ax = 2;
    on = on && !miss && !run_too_far(X0) && !run_too_far(X1) && !run_too_far(X2) && amin < amax;
    if (__builtin_amdgcn_ballot_w64(on) == 0) return;

    // a < b: the other two axes
    const int axa = q == 0 ? 1 : 0, axb = q == 2 ? 1 : 2;
    const RunAxis a = run_pick(q == 0, X1, X0), b = run_pick(q == 2, X1, X2);
    const int na = q == 0 ? V.n[1] : V.n[0], nb = q == 2 ? V.n[1] : V.n[2];
    const int nq = run_pick3(q, V.n[0], V.n[1], V.n[2]);
    const double s0 = s[0], s1 = s[1], s2 = s[2], d0 = d[0], d1 = d[1], d2 = d[2];
    const double sq = run_pick3(q, s0, s1, s2), dq = run_pick3(q, d0, d1, d2);
    const double oq = run_pick3(q, V.origin[0], V.origin[1], V.origin[2]);
    const double iq = run_pick3(q, V.inv_spacing[0], V.inv_spacing[1], V.inv_spacing[2]);
    const double wq = run_pick3(q, V.spacing[0], V.spacing[1], V.spacing[2]);
    const uint64_t oa = run_pick3(q, V.run_off[0][0], V.run_off[1][0], V.run_off[2][0]);
    const uint64_t ob = run_pick3(q, V.run_off[0][1], V.run_off[1][1], V.run_off[2][1]);
    const uint64_t oe = run_pick3(q, V.run_off[0][2], V.run_off[1][2], V.run_off[2][2]);
    RunTable Ta, Tb;
    Ta.row = Tb.row = __builtin_amdgcn_readfirstlane((nq + kRunPad) * 4);
    Ta.plane = (uint32_t)Ta.row * (uint32_t)nb;
    Tb.plane = (uint32_t)Tb.row * (uint32_t)na;
    Ta.rsrc = make_run_rsrc(V, oa, Ta.plane * (uint32_t)(na + 1));
    Tb.rsrc = make_run_rsrc(V, ob, Tb.plane * (uint32_t)(nb + 1));
    // entry 0 of a row lies one voxel before the grid
    const double q1 = dq * iq, q0 = fma(sq - oq, iq, 1.0);

    // columns at the ray's ends, and between them the crossings strictly
    // inside (amin, amax)
    const int ia = planes_passed<false>(a, amin), ib = planes_passed<false>(b, amin);
    const int ja = planes_passed<true>(a, amax), jb = planes_passed<true>(b, amax);

    // P at the ray's ends.  On a face of a or b it is that face's crossing,
    // on a face of q the column's first or last sum; an end inside the grid
    // (alpha 0 or 1) is reached by the crossings of a path that leaves it
    // along axis a, and belongs to no axis.
    double ends = 0.0, Aa = 0.0, Ab = 0.0, Ba = 0.0, Bb = 0.0, Ac = 0.0, Bc = 0.0;
#pragma unroll 1
    for (int e = 0; e < 2; ++e) {
        const double alpha = e ? amax : amin, sign = e ? 1.0 : -1.0;
        const int face = e ? amax_ax : amin_ax;
        const int pa = e ? ja : ia, pb = e ? jb : ib;
        const int ca = a.neg ? na - pa : pa - 1, cb = b.neg ? nb - pb : pb - 1;
        const double t = fma(alpha, q1, q0), f = __builtin_amdgcn_fract(t);
        const int entry = (int)t * 4;
        double P = 0.0, p, v;
        const bool fq = on && face == q, fa = on && face == axa, fb = on && face == axb,
                   in = on && face < 0;
        if (__builtin_amdgcn_ballot_w64(fq)) {
            const __amdgpu_buffer_rsrc_t re = make_run_rsrc(V, oe, (uint32_t)(na * nb) * 16u);
            const bool last = (dq > 0.0) == (e == 1);
            const uint32_t off = (uint32_t)(ca * nb + cb) * 16u + (last ? 8u : 0u);
            const run_u32x2 c = run_load(re, fq ? off : kRunNone, 0);
            P += __hiloint2double((int)c.y, (int)c.x);
        }
        if (__builtin_amdgcn_ballot_w64(fa)) {
            run_face(Ta, fa, (e == 1) != a.neg, na, (uint32_t)(entry + cb * Ta.row), f, p, v);
            P += p;
            if (JAC) Aa = fma(sign, v, Aa), Ba = fma(sign * alpha, v, Ba);
        }
        if (__builtin_amdgcn_ballot_w64(fb)) {
            run_face(Tb, fb, (e == 1) != b.neg, nb, (uint32_t)(entry + ca * Tb.row), f, p, v);
            P += p;
            if (JAC) Ab = fma(sign, v, Ab), Bb = fma(sign * alpha, v, Bb);
        }
        if (in) {
            for (int k = ca + 1; k <= na; ++k) {
                const RunPair x = run_pair(run_load(
                    Ta.rsrc, (uint32_t)(entry + cb * Ta.row) + (uint32_t)k * Ta.plane, 0));
                P += x.jump;
                P = fma(f, x.step, P);
                if (JAC) Ac = fma(sign, x.step, Ac), Bc = fma(sign * alpha, x.step, Bc);
            }
        }
        ends = fma(sign, P, ends);
    }

    // the crossings, added to the ends' terms in the tables' sense (below
    // minus above: the ray's own where it runs upwards)
    const double scale = wq / dq;
    auto flip = [](bool neg, double x) { return neg ? -x : x; };
    double acc = flip(a.neg, ends);
    Aa = flip(a.neg, Aa), Ba = flip(a.neg, Ba);
    run_crossings<JAC, false, S>(Ta, a, on ? ia : 1, on ? ja - 1 : 0, na, b, nb, q1, q0, acc, Aa, Ba);
    Aa = flip(a.neg, Aa), Ba = flip(a.neg, Ba);
    acc = flip(a.neg != b.neg, acc);
    Ab = flip(b.neg, Ab), Bb = flip(b.neg, Bb);
    run_crossings<JAC, true, S>(Tb, b, on ? ib : 1, on ? jb - 1 : 0, nb, a, na, q1, q0, acc, Ab, Bb);
    Ab = flip(b.neg, Ab), Bb = flip(b.neg, Bb);
    acc = flip(b.neg, acc);
    if (on) {
        const RunHeader* H = (const RunHeader*)V.run;
        const double quantum = run_pick3(q, H->quantum[0], H->quantum[1], H->quantum[2]);
        r.sum = acc * (quantum * scale);
        if (JAC) {
            // the sums over all crossings are 0 and E / |d|: the q planes
            // take what the others leave
            Aa *= quantum, Ab *= quantum, Ac *= quantum;
            Ba *= quantum, Bb *= quantum, Bc *= quantum;
            const double Aq = -(Aa + Ab + Ac), Bq = r.sum - Ba - Bb - Bc;
            r.a0 = q == 0 ? Aq : Aa;
            r.b0 = q == 0 ? Bq : Ba;
            r.a1 = q == 0 ? Aa : (q == 1 ? Aq : Ab);
            r.b1 = q == 0 ? Ba : (q == 1 ? Bq : Bb);
            r.a2 = q == 2 ? Aq : Ab;
            r.b2 = q == 2 ? Bq : Bb;
        }
    }
}

// Sums of the rays of a wave, and their lengths |d|.  ray(s, d) forms the
// lane's ray; it is called again for each direction of runs in the wave (one
// but for a few waves of a launch), so that the ray's own values need not be
// kept through the crossings.  pose_axis: run_direction of the pose's central
// ray.
template <bool JAC, typename S, typename Ray>
__device__ __forceinline__ RayAcc trace_runs(const VolArgs& V, bool inside, const Ray& ray,
                                             int pose_axis, double& length)
{
    RayAcc r;
    r.sum = 0.0;
    r.a0 = r.a1 = r.a2 = r.b0 = r.b1 = r.b2 = 0.0;
    r.nseg = 0;
    r.valid = true;
    length = 0.0;
    uint64_t done = ~__builtin_amdgcn_ballot_w64(inside);
    auto pass = [&](auto shape) {
        double s[3], d[3];
        ray(s, d);
        bool finite = true;
#pragma unroll
        for (int c = 0; c < 3; ++c) finite = finite && isfinite(s[c]) && isfinite(d[c]);
        const int mine = run_direction(d, V.inv_spacing, pose_axis);
        const int q = __builtin_amdgcn_readlane(mine, __builtin_ctzll(~done));
        const bool now = inside && mine == q;
        done |= __builtin_amdgcn_ballot_w64(now);
        if (now) {
            r.valid = finite;
            length = sqrt(fma(d[0], d[0], fma(d[1], d[1], d[2] * d[2])));
        }
        trace_along<JAC, decltype(shape)>(V, q, now && finite, s, d, r);
    };
    if (~done) pass(S{});
    // (a copy of its own: in one loop the compiler would move what the pass
    // computes from the pose, detector and volume before it and hold that in
    // some 40 registers through the crossings; small batches, for
    // the same reason)
    using Rest = typename std::conditional<S::pipelined, S, RunRare>::type;
    while (~done) pass(Rest{});
    return r;
}

// Whether the volume's crossing tables are to be used (wave-uniform).
__device__ inline bool run_tables_usable(const VolArgs& V)
{
    return __builtin_amdgcn_readfirstlane(((const RunHeader*)V.run)->use) != 0;
}

}  // namespace drr
