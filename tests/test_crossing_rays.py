"""The crossing-table traversal's plane and column indexes on the CPU: the
kernels' own header (csrc/run_rays.hpp) in a host model that checks every
table read against its bounds and every column index against an enumeration
of the planes, with its path sums and derivative sums compared with the
oracle's -- over rays of any direction, ties, rays on and parallel to planes,
ends inside the grid and very long rays."""

import ctypes
import math
import os
import shutil
import subprocess

import numpy as np
import pytest

import oracle

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    gxx = shutil.which("g++")
    assert gxx is not None, "g++ is needed to build the host model"
    out = tmp_path_factory.mktemp("crossing") / "libcrossing.so"
    res = subprocess.run([gxx, "-std=c++17", "-O2", "-Wall", "-Werror", "-ffp-contract=off", "-fPIC",
                          "-shared", "-o", str(out),
                          os.path.join(ROOT, "tests", "c", "crossing_rays_check.cpp")],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    lib = ctypes.CDLL(str(out))
    lib.crossing_bad.restype = ctypes.c_int64
    return lib


def _p(a):
    return a.ctypes.data_as(ctypes.c_void_p)


def _sums(lib, src, dst, pose=-1):
    d = np.ascontiguousarray(dst - src)
    out = np.zeros((len(src), 8))
    lib.crossing_trace(len(src), _p(np.ascontiguousarray(src)), _p(d), pose, _p(out))
    return out, d


def _case(rng, kind):
    """A small grid and rays through it."""
    dims = tuple(int(v) for v in rng.integers(1, 22, 3))
    sp = {"ties": np.ones(3), "half_ties": np.array([0.5, 1.0, 2.0])}.get(
        kind, rng.uniform(0.3, 3.0, 3))
    ext = np.array(dims) * sp
    tied = kind in ("ties", "half_ties", "parallel")
    org = -0.5 * ext if tied else -0.5 * ext + rng.uniform(-0.3, 0.3, 3) * ext
    v = rng.uniform(0.2, 2.0, dims).astype(np.float32)
    v[rng.uniform(size=dims) < 0.3] = 0.0
    size = float(np.linalg.norm(ext))
    n = 200
    if kind == "parallel":      # along one or two axes, many exactly on planes
        src = org + rng.integers(-2, 2 * np.array(dims) + 4, (n, 3)) * 0.5 * sp
        d = rng.integers(-1, 2, (n, 3)) * 2.0 * size
        src = src - 0.5 * d * rng.integers(0, 3, (n, 1))
        dst = src + d
    elif tied:                  # from a lattice point to a lattice point
        src = org + rng.integers(-24, 24, (n, 3)) * sp
        dst = -src + org * 0 + rng.integers(-4, 5, (n, 3)) * sp
    elif kind == "inside":      # ends inside the grid
        src = org + rng.uniform(-0.2, 1.2, (n, 3)) * ext
        dst = org + rng.uniform(-0.2, 1.2, (n, 3)) * ext
    else:
        far = {"any": 2.0, "long": 1e5}[kind]
        u = rng.normal(size=(n, 3))
        u /= np.linalg.norm(u, axis=1, keepdims=True)
        mid = org + rng.uniform(-0.1, 1.1, (n, 3)) * ext
        src, dst = mid + far * size * u, mid - far * size * u
    keep = np.linalg.norm(dst - src, axis=1) > 0
    return dims, sp, org, v, src[keep].astype(float), dst[keep].astype(float), size


@pytest.mark.parametrize("kind", ["any", "inside", "ties", "half_ties", "parallel", "long"])
def test_sums_match_the_oracle(model, kind):
    """Path sums within the tables' quantum: some 200 terms of at most one
    quantum, 2^-31 of a jump that is at most a column's sum, so 1e-7 of the
    largest pixel bounds them; rays 1e5 grids long leave their positions 1e-11
    of the grid, which the bound covers.  Every index is in range and equal to
    the enumeration."""
    rng = np.random.default_rng({"any": 1, "inside": 2, "ties": 3, "half_ties": 4, "parallel": 5,
                                 "long": 6}[kind])
    seen = 0
    for k in range(40):
        dims, sp, org, v, src, dst, size = _case(rng, kind)
        model.crossing_volume(_p(v), _p(np.array(dims, np.int32)), _p(np.ascontiguousarray(sp)),
                              _p(np.ascontiguousarray(org)))
        out, d = _sums(model, src, dst, k % 4 - 1)      # any preferred direction
        ref, _, _ = oracle.trace_rays(oracle.Grid(v, tuple(sp), tuple(org)), src, dst, nthreads=2)
        got = out[:, 0] * np.linalg.norm(d, axis=1)
        scale = max(ref.max(), float(v.max()) * sp.min())
        assert np.abs(got - ref).max() <= 1e-7 * scale, (kind, dims)
        seen += int((ref > 0).sum())
    assert seen > 500
    assert model.crossing_bad() == 0


def test_rays_through_zeros_sum_to_exactly_zero(model):
    """Past an object, columns of different totals: the terms of a ray that
    passes only zeros cancel without a remainder."""
    rng = np.random.default_rng(9)
    dims, sp = (20, 18, 22), np.array([1.0, 1.1, 0.9])
    v = np.zeros(dims, np.float32)
    v[5:9] = rng.uniform(0.1, 2.0, (4, 18, 22))
    org = -0.5 * np.array(dims) * sp
    model.crossing_volume(_p(v), _p(np.array(dims, np.int32)), _p(sp), _p(org))
    n = 300      # both ends beyond x = 9 voxels, leaving through the sides
    src = org + np.stack([rng.uniform(9.5, 19.5, n), rng.uniform(-30, -5, n),
                          rng.uniform(0, 22, n)], 1) * sp
    dst = org + np.stack([rng.uniform(9.5, 19.5, n), rng.uniform(25, 50, n),
                          rng.uniform(0, 22, n)], 1) * sp
    out, _ = _sums(model, src, dst)
    assert np.all(out[:, 0] == 0.0)


def test_derivative_sums_match_the_oracle(model):
    """dE/ds and dE/dp from the sums A, B, on rays off the ties (FP64 sums of
    quantised voxel jumps: 1e-6 of the column's scale)."""
    rng = np.random.default_rng(11)
    for _ in range(10):
        dims, sp, org, v, src, dst, size = _case(rng, "any")
        model.crossing_volume(_p(v), _p(np.array(dims, np.int32)), _p(np.ascontiguousarray(sp)),
                              _p(np.ascontiguousarray(org)))
        out, d = _sums(model, src, dst)
        E, gs, gp = oracle.trace_rays_grad(oracle.Grid(v, tuple(sp), tuple(org)), src, dst)[:3]
        L = np.linalg.norm(d, axis=1, keepdims=True)
        A, B, sums = out[:, 1:4], out[:, 4:7], out[:, :1]
        got_p = sums * d / L - L * B / d
        got_s = -(sums * d / L) + L * (B - A) / d
        scale = max(np.abs(gp).max(), np.abs(gs).max(), 1e-3)
        assert np.abs(got_p - gp).max() <= 1e-6 * scale
        assert np.abs(got_s - gs).max() <= 1e-6 * scale
    assert model.crossing_bad() == 0
