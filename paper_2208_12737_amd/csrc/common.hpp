// Host-side helpers shared by the C-ABI entry points: argument validation,
// the thread-local error message, and conversion of public descriptors into
// kernel argument blocks.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdarg.h>
#include <stdint.h>
#include <stdio.h>

#include "../../include/drr.h"
#include "launch_budget.hpp"
#include "siddon.hpp"

namespace drr {

int32_t fail(int32_t code, const char* fmt, ...);
int32_t check_launch(const char* what);

inline bool finite_pos(double x) { return isfinite(x) && x > 0.0; }

// Largest packed volume the 32-bit buffer offsets can address.
constexpr uint64_t kMaxPackedBytes = 0xFFFFFF00ull;

// Elements of one zero-bordered copy of the grid.
inline uint64_t copy_elems(const drr_volume_desc& v)
{
    return (uint64_t)(v.nx + 2) * (uint64_t)(v.ny + 2) * (uint64_t)(v.nz + 2);
}

// Layout of the copies.
inline int base_layout(const drr_volume_desc& v) { return v.layout & ~DRR_LAYOUT_CROSSINGS; }

inline int num_copies(const drr_volume_desc& v)
{
    return base_layout(v) == DRR_LAYOUT_PER_AXIS ? 3 : 1;
}

inline uint64_t packed_elems(const drr_volume_desc& v) { return copy_elems(v) * num_copies(v); }

// Crossing tables of the runs along axis q (see runs.hpp): which = 0 the
// planes of the lower other axis, 1 of the higher, 2 the columns' end sums.
inline uint64_t run_table_bytes(const drr_volume_desc& v, int q, int which)
{
    const uint64_t n[3] = {(uint64_t)v.nx, (uint64_t)v.ny, (uint64_t)v.nz};
    const uint64_t a = n[q == 0 ? 1 : 0], b = n[q == 2 ? 1 : 2];
    if (which == 2) return a * b * 16ull;
    return (which == 0 ? (a + 1) * b : (b + 1) * a) * (n[q] + kRunPad) * 4ull;
}

// Whether the packed volume carries crossing tables: three copies always do,
// one copy if asked, where every table is within the reach of the
// traversal's offsets (32-bit bytes below kRunNone, 24-bit row lengths) --
// per axis pair, fewer than some 2^30 voxels.
inline bool has_run_tables(const drr_volume_desc& v)
{
    if (v.layout == DRR_LAYOUT_INPUT) return false;
    const int32_t most = (1 << 21) - kRunPad - 1;
    if (v.nx > most || v.ny > most || v.nz > most) return false;
    for (int q = 0; q < 3; ++q)
        for (int w = 0; w < 3; ++w)
            if (run_table_bytes(v, q, w) > 0xE0000000ull) return false;
    return true;
}

// Byte offset of a table from the header (256-byte aligned); of the end of
// the last one for q = 3.
inline uint64_t run_table_offset(const drr_volume_desc& v, int q, int which)
{
    uint64_t at = kRunHeaderBytes;
    for (int p = 0; p < 3 * q + which; ++p)
        at += (run_table_bytes(v, p / 3, p % 3) + 255) & ~255ull;
    return at;
}

// Byte offset of the header: behind the copies.
inline uint64_t run_header_offset(const drr_volume_desc& v)
{
    return (packed_elems(v) * 4ull + 255) & ~255ull;
}

// Memory order of copy q (slowest axis first).  DRR_LAYOUT_INPUT keeps the
// caller's (x, y, z).  DRR_LAYOUT_PER_AXIS: copy q serves rays running
// mostly along axis q; q is the slowest axis and, of the other two, the one
// with the finer spacing varies fastest.
struct CopyOrder {
    int axis[3];
};

inline CopyOrder copy_order(const drr_volume_desc& v, int q)
{
    CopyOrder o;
    if (base_layout(v) != DRR_LAYOUT_PER_AXIS) {
        o.axis[0] = 0;
        o.axis[1] = 1;
        o.axis[2] = 2;
        return o;
    }
    const int a = (q + 1) % 3, b = (q + 2) % 3;
    const bool a_finer = v.spacing[a] < v.spacing[b] || (v.spacing[a] == v.spacing[b] && a > b);
    o.axis[0] = q;
    o.axis[1] = a_finer ? b : a;
    o.axis[2] = a_finer ? a : b;
    return o;
}

// Element pitch of each logical axis in copy q.
inline void copy_pitch(const drr_volume_desc& v, int q, int64_t pitch[3])
{
    const int64_t P[3] = {v.nx + 2, v.ny + 2, v.nz + 2};
    const CopyOrder o = copy_order(v, q);
    pitch[o.axis[2]] = 1;
    pitch[o.axis[1]] = P[o.axis[2]];
    pitch[o.axis[0]] = P[o.axis[2]] * P[o.axis[1]];
}

// Launches on volumes with crossing tables: workgroups of two tiles per CU
// where the bytes of the tables bound the launch, 0 where single tiles, four
// a CU, are better.  The tables of one direction hold 8 bytes a voxel; up to
// 64 MB the caches keep what a pose reads of them, and more waves in flight
// are faster (16 against 8 waves a CU: 340 x 340 pixels x 196 poses on 103 x
// 173 x 42 voxels 1.56 against 2.30 ms).  Above, 16 x 32 pixels a workgroup,
// one a CU, read fewer bytes again (256 poses of 256 x 256 on the 512 x 512 x
// 133 CT: 4.26 ms against 5.14 ms with two a CU and 5.47 ms with four single
// tiles; 128 x 128 x 512 poses: 7.6 / 8.7 / 10.0 ms), unless the rays lie so
// close together that neighbours share most of what they read (512 x 512
// pixels on the 512 x 512 x 300 CT: 0.82 against 0.70 ms with two a CU).
inline int run_big_tables(const drr_volume_desc& vol, const drr_detector_desc& det)
{
    const double voxels = (double)vol.nx * vol.ny * vol.nz;
    if (voxels < 8e6) return 0;
    // rays per voxel face at the middle of the way (half the pixel pitch)
    const double face = cbrt(vol.spacing[0] * vol.spacing[1] * vol.spacing[2]);
    const double rays = face * face / (0.25 * det.delta_x * det.delta_y);
    return voxels < 1e7 || rays > 4.0 ? 2 : 1;
}

inline int32_t validate_volume(const drr_volume_desc* v)
{
    if (!v) return fail(DRR_EINVAL, "volume descriptor is NULL");
    if (v->nx < 1 || v->ny < 1 || v->nz < 1)
        return fail(DRR_EINVAL, "volume dims must be >= 1 (got %d x %d x %d)", v->nx, v->ny,
                    v->nz);
    for (int c = 0; c < 3; ++c) {
        if (!finite_pos(v->spacing[c]))
            return fail(DRR_EINVAL, "volume spacing[%d] must be finite and > 0", c);
        if (!isfinite(v->origin[c])) return fail(DRR_EINVAL, "volume origin[%d] is not finite", c);
    }
    if (base_layout(*v) != DRR_LAYOUT_INPUT && base_layout(*v) != DRR_LAYOUT_PER_AXIS)
        return fail(DRR_EINVAL, "unknown volume layout %d", v->layout);
    if (copy_elems(*v) * 4ull > kMaxPackedBytes)
        return fail(DRR_ENOTSUP, "packed volume copy of %llu bytes exceeds the 4 GiB buffer limit",
                    (unsigned long long)(copy_elems(*v) * 4ull));
    return DRR_OK;
}

inline int32_t validate_detector(const drr_detector_desc* d)
{
    if (!d) return fail(DRR_EINVAL, "detector descriptor is NULL");
    if (d->height < 1 || d->width < 1)
        return fail(DRR_EINVAL, "detector size must be >= 1 (got %d x %d)", d->height, d->width);
    if ((int64_t)d->height * d->width > (int64_t)1 << 30)
        return fail(DRR_ENOTSUP, "detector of %d x %d pixels is too large", d->height, d->width);
    if (!finite_pos(d->delta_x) || !finite_pos(d->delta_y))
        return fail(DRR_EINVAL, "detector pitch must be finite and > 0");
    if (!isfinite(d->offset_u) || !isfinite(d->offset_v))
        return fail(DRR_EINVAL, "detector offsets must be finite");
    return DRR_OK;
}

inline VolArgs vol_args(const void* packed, const drr_volume_desc& v)
{
    VolArgs a;
    a.packed = (const float*)packed;
    a.n[0] = v.nx;
    a.n[1] = v.ny;
    a.n[2] = v.nz;
    for (int c = 0; c < 3; ++c) {
        a.spacing[c] = v.spacing[c];
        a.origin[c] = v.origin[c];
    }
    a.copy_bytes = (uint32_t)(copy_elems(v) * 4ull);
    const int nc = num_copies(v);
    for (int q = 0; q < 3; ++q) {
        int64_t p[3];
        copy_pitch(v, q < nc ? q : 0, p);
        for (int c = 0; c < 3; ++c) a.pitch[q][c] = (int32_t)(p[c] * 4);
        a.copy_for[q] = q < nc ? q : 0;
    }
    const bool runs = has_run_tables(v);
    a.run = runs ? (const char*)packed + run_header_offset(v) : nullptr;
    for (int q = 0; q < 3; ++q) {
        for (int w = 0; w < 3; ++w) a.run_off[q][w] = runs ? run_table_offset(v, q, w) : 0;
        a.inv_spacing[q] = 1.0 / v.spacing[q];
    }
    return a;
}

inline DetArgs det_args(const drr_detector_desc& d)
{
    DetArgs a;
    a.H = d.height;
    a.W = d.width;
    a.dx = d.delta_x;
    a.dy = d.delta_y;
    a.ou = d.offset_u;
    a.ov = d.offset_v;
    return a;
}

inline hipStream_t as_stream(void* s) { return (hipStream_t)s; }

// Compute units of the device current at the first launch (queried once).
inline int num_cus()
{
    static const int n = [] {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) != hipSuccess) dev = 0;
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            v <= 0)
            v = 256;
        return v;
    }();
    return n;
}

// LDS per CU and per workgroup, queried once (thread-safe initialisation of
// a function-local static) on the device current at the first launch.
inline LdsLimits lds_limits()
{
    static const LdsLimits lim = [] {
        int dev = 0, v = 0, b = 0;
        if (hipGetDevice(&dev) != hipSuccess) dev = 0;
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, dev) !=
                hipSuccess || v <= 0)
            v = 160 * 1024;
        if (hipDeviceGetAttribute(&b, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) !=
                hipSuccess || b <= 0)
            b = 64 * 1024;
        return LdsLimits{(size_t)v, (size_t)(b < v ? b : v)};
    }();
    return lim;
}

// Dynamic LDS that caps residency at `wg_per_cu` workgroups per CU on this
// device (see occupancy_lds_bytes).
inline size_t occupancy_lds(int wg_per_cu, size_t static_bytes)
{
    return occupancy_lds_bytes(lds_limits(), wg_per_cu, static_bytes);
}

}  // namespace drr
