// Host model of the crossing-table traversal: the indexes come from the
// kernels' own header (run_rays.hpp), the tables are built here and every
// read is checked against their bounds.  Compares each column index with an
// enumeration of the planes.
#include <stdint.h>
#include <string.h>

#include <vector>

#include "../../paper_2208_12737_amd/csrc/run_rays.hpp"

using namespace drr;

namespace {

struct Table {
    std::vector<double> jump;   // [planes][columns][entries]
    int planes = 0, columns = 0, entries = 0;
};

Table tab[3][2];
std::vector<double> ends[3];
int N[3];
double SP[3], INV[3], ORG[3], QUANTUM[3];
int64_t bad = 0;

double entry(const Table& t, int k, int c, int i)
{
    if (k < 0 || k >= t.planes || c < 0 || c >= t.columns || i < 0 || i >= t.entries) {
        ++bad;
        return 0.0;
    }
    return t.jump[((size_t)k * t.columns + c) * t.entries + i];
}

// The same count by trying every plane.
template <bool STRICT>
int passed(const RunAxis& x, double alpha, int n)
{
    const int got = planes_passed<STRICT>(x, alpha);
    if (x.da > 0.0) {
        int all = 0;
        for (int k = 0; k <= n; ++k) {
            const double am = fma((double)k, x.da, x.a0);
            all += (STRICT ? am < alpha : am <= alpha) ? 1 : 0;
        }
        bad += all != got;
    }
    return got;
}

}  // namespace

extern "C" int64_t crossing_bad() { return bad; }

extern "C" void crossing_volume(const float* v, const int* n, const double* sp, const double* org)
{
    for (int c = 0; c < 3; ++c) {
        N[c] = n[c];
        SP[c] = sp[c];
        INV[c] = 1.0 / sp[c];
        ORG[c] = org[c];
    }
    const int64_t st[3] = {(int64_t)n[1] * n[2], n[2], 1};
    for (int q = 0; q < 3; ++q) {
        double most = 0.0;
        for (int w = 0; w < 2; ++w) {
            const int lo = q == 0 ? 1 : 0, hi = q == 2 ? 1 : 2, a = w ? hi : lo, b = w ? lo : hi;
            Table& t = tab[q][w];
            t.planes = n[a] + 1;
            t.columns = n[b];
            t.entries = n[q] + 3;
            t.jump.assign((size_t)t.planes * t.columns * t.entries, 0.0);
            if (!w) ends[q].assign((size_t)n[lo] * n[hi] * 2, 0.0);
            // running sums of a column, from the middle of its total
            auto sums = [&](int ca, int cb, std::vector<double>& s) {
                s.assign(n[q] + 1, 0.0);
                if (ca < 0 || ca >= n[a]) return;
                double total = 0.0;
                for (int i = 0; i < n[q]; ++i) total += v[ca * st[a] + cb * st[b] + i * st[q]];
                s[0] = -0.5 * total;
                for (int i = 0; i < n[q]; ++i)
                    s[i + 1] = s[i] + v[ca * st[a] + cb * st[b] + i * st[q]];
            };
            std::vector<double> below, above;
            for (int c = 0; c < n[b]; ++c)
                for (int k = 0; k <= n[a]; ++k) {
                    sums(k - 1, c, below);
                    sums(k, c, above);
                    for (int i = 0; i <= n[q]; ++i)
                        most = fmax(most, fabs(below[i] - above[i]));
                }
        }
        const double quantum = QUANTUM[q] = most > 0.0 ? most / 2147483640.0 : 1.0;
        for (int w = 0; w < 2; ++w) {
            const int lo = q == 0 ? 1 : 0, hi = q == 2 ? 1 : 2, a = w ? hi : lo, b = w ? lo : hi;
            Table& t = tab[q][w];
            for (int c = 0; c < n[b]; ++c)
                for (int k = 0; k <= n[a]; ++k) {
                    double s[2][2] = {};
                    for (int side = 0; side < 2; ++side) {
                        const int ca = k - 1 + side;
                        if (ca < 0 || ca >= n[a]) continue;
                        double total = 0.0;
                        for (int i = 0; i < n[q]; ++i)
                            total += v[ca * st[a] + c * st[b] + i * st[q]];
                        s[side][0] = -0.5 * total;
                    }
                    for (int i = 0; i <= n[q]; ++i) {
                        double quanta[2];
                        for (int side = 0; side < 2; ++side) {
                            const int ca = k - 1 + side;
                            quanta[side] = rint(s[side][0] / quantum);
                            if (side == 1 && w == 0 && k < n[a]) {
                                if (i == 0) ends[q][((size_t)k * n[b] + c) * 2] = quanta[1];
                                ends[q][((size_t)k * n[b] + c) * 2 + 1] = quanta[1];
                            }
                            if (ca >= 0 && ca < n[a] && i < n[q])
                                s[side][0] += v[ca * st[a] + c * st[b] + i * st[q]];
                        }
                        double* row = &t.jump[((size_t)k * t.columns + c) * t.entries];
                        row[i + 1] = quanta[0] - quanta[1];
                        if (i == 0) row[0] = row[1];
                        if (i == n[q]) row[n[q] + 2] = row[n[q] + 1];
                    }
                }
        }
    }
}

// out[r] = {E / |d|, A[3], B[3], direction of the runs} of ray S + alpha D.
// `pose` is the preferred direction (-1: none).
extern "C" void crossing_trace(int rays, const double* S, const double* D, int pose, double* out)
{
    for (int r = 0; r < rays; ++r) {
        const double *s = S + 3 * r, *d = D + 3 * r;
        double* o = out + 8 * r;
        memset(o, 0, 8 * sizeof(double));
        double amin = 0.0, amax = 1.0;
        int entry_ax = -1, exit_ax = -1;
        bool miss = false, far = false;
        RunAxis ax[3];
        for (int c = 0; c < 3; ++c) {
            double exit;
            ax[c] = run_axis(s[c], d[c], ORG[c], SP[c], INV[c], N[c], &exit, &miss);
            far = far || run_too_far(ax[c]);
            if (ax[c].a0 > amin) amin = ax[c].a0, entry_ax = c;
            if (exit < amax) amax = exit, exit_ax = c;
        }
        if (miss || far || !(amin < amax)) continue;
        const int q = run_direction(d, INV, pose);
        const int axes[2] = {q == 0 ? 1 : 0, q == 2 ? 1 : 2};
        const RunAxis x[2] = {ax[axes[0]], ax[axes[1]]};
        const int n[2] = {N[axes[0]], N[axes[1]]};
        const double q1 = d[q] * INV[q], q0 = fma(s[q] - ORG[q], INV[q], 1.0);
        int p[2][2];   // [end][axis]: planes passed
        p[0][0] = passed<false>(x[0], amin, n[0]);
        p[0][1] = passed<false>(x[1], amin, n[1]);
        p[1][0] = passed<true>(x[0], amax, n[0]);
        p[1][1] = passed<true>(x[1], amax, n[1]);
        auto cell = [&](int w, int count) {
            const int c = x[w].neg ? n[w] - count : count - 1;
            bad += c < 0 || c >= n[w];
            return c;
        };
        double sum = 0.0, A[2] = {}, B[2] = {}, Ac = 0.0, Bc = 0.0;
        for (int w = 0; w < 2; ++w) {
            const double sign = x[w].neg ? -1.0 : 1.0;
            for (int k = p[0][w]; k < p[1][w]; ++k) {
                const double alpha = fma((double)k, x[w].da, x[w].a0);
                bad += !(alpha > amin && alpha < amax) || k < 1 || k > n[w] - 1;
                const int other = w ? passed<true>(x[0], alpha, n[0]) : passed<false>(x[1], alpha, n[1]);
                const double t = fma(alpha, q1, q0), f = t - floor(t);
                const int plane = x[w].neg ? n[w] - k : k, c = cell(1 - w, other);
                const double j0 = entry(tab[q][w], plane, c, (int)t),
                             j1 = entry(tab[q][w], plane, c, (int)t + 1);
                sum += sign * fma(f, j1 - j0, j0);
                A[w] += sign * (j1 - j0);
                B[w] += sign * alpha * (j1 - j0);
            }
        }
        for (int e = 0; e < 2; ++e) {
            const double alpha = e ? amax : amin, sign = e ? 1.0 : -1.0;
            const int face = e ? exit_ax : entry_ax;
            const int c[2] = {cell(0, p[e][0]), cell(1, p[e][1])};
            const double t = fma(alpha, q1, q0), f = t - floor(t);
            double P = 0.0;
            if (face == q)
                P = ends[q][((size_t)c[0] * n[1] + c[1]) * 2 + ((d[q] > 0.0) == (e == 1) ? 1 : 0)];
            for (int w = 0; w < 2; ++w) {
                if (face != axes[w]) continue;
                const bool upper = (e == 1) != x[w].neg;
                const double side = upper ? 1.0 : -1.0;
                const int plane = upper ? n[w] : 0;
                const double j0 = entry(tab[q][w], plane, c[1 - w], (int)t),
                             j1 = entry(tab[q][w], plane, c[1 - w], (int)t + 1);
                P = side * fma(f, j1 - j0, j0);
                A[w] += sign * side * (j1 - j0);
                B[w] += sign * side * alpha * (j1 - j0);
            }
            if (face < 0) {
                for (int k = c[0] + 1; k <= n[0]; ++k) {
                    const double j0 = entry(tab[q][0], k, c[1], (int)t),
                                 j1 = entry(tab[q][0], k, c[1], (int)t + 1);
                    P += fma(f, j1 - j0, j0);
                    Ac += sign * (j1 - j0);
                    Bc += sign * alpha * (j1 - j0);
                }
            }
            sum += sign * P;
        }
        const double Q = QUANTUM[q];
        o[0] = sum * Q * (SP[q] / d[q]);
        for (int w = 0; w < 2; ++w) {
            o[1 + axes[w]] = A[w] * Q;
            o[4 + axes[w]] = B[w] * Q;
        }
        o[1 + q] = -(A[0] + A[1] + Ac) * Q;
        o[4 + q] = o[0] - (B[0] + B[1] + Bc) * Q;
        o[7] = q;
    }
}
