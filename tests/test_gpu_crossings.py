"""Renders from the crossing tables: against the plane merge on the same
volume and against the oracle at the edges of sizes, the volumes whose tables
are refused, and bitwise equality between the launch shapes."""

import ctypes
import math
import types

import numpy as np
import pytest
import torch

import oracle
from synth import random_poses
from _parity import assert_image_close, column_errors

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"


def _merge_volume(data, spacing, origin):
    """The single-copy layout without tables: every render takes the merge."""
    from paper_2208_12737_amd import _lib
    src = torch.from_numpy(data).to(DEV)
    desc = _lib.volume_desc(data.shape, spacing, origin, _lib.DRR_LAYOUT_INPUT)
    n = _lib.load().drr_volume_packed_bytes(ctypes.byref(desc))
    packed = torch.empty(n // 4, device=DEV)
    _lib.call("drr_volume_pack", src.data_ptr(), packed.data_ptr(), ctypes.byref(desc),
              torch.cuda.current_stream().cuda_stream)
    return types.SimpleNamespace(packed=packed, desc=desc, device=packed.device)


def _gpu(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(DEV)


@pytest.mark.parametrize("dims", [(1, 1, 1), (1, 40, 2), (31, 32, 33), (64, 65, 63), (129, 16, 70)])
def test_tables_agree_with_the_merge_and_the_oracle(dims):
    """Sizes around the packing's strips of 64 columns and stages of 32
    voxels, views along every axis, a source inside and a detector plane
    inside the grid.  Tables and merge differ by quanta (2^-31 of a column
    sum, some 100 terms) and FP32 rounding: 2e-7 of the largest pixel; their
    Jacobians by the merge's FP32 sums."""
    import paper_2208_12737_amd as P
    rng = np.random.default_rng(sum(dims))
    spacing = (1.1, 0.8, 1.7)
    ext = np.asarray(dims) * np.asarray(spacing)
    origin = tuple(float(v) for v in -0.5 * ext + rng.uniform(-0.2, 0.2, 3) * ext)
    data = rng.uniform(0.0, 2.0, dims).astype(np.float32)
    data[rng.uniform(size=dims) < 0.2] = 0.0
    size = float(np.linalg.norm(ext))
    poses = np.concatenate([rng.uniform(-math.pi, math.pi, (6, 3)), rng.uniform(-0.1, 0.1, (6, 3)) * ext,
                            np.full((6, 1), 4.0 * size)], axis=1).astype(np.float32)
    poses[1, :3] = 0.0
    poses[2, :3] = (math.pi / 2, 0.0, 0.0)
    poses[3, :3] = (0.0, math.pi / 2, 0.0)
    poses[4, 6] = 0.6 * size
    H, W = 21, 26
    pitch = 2.4 * size / W
    det = P.Detector(H, W, pitch, pitch)
    vol = P.Volume(torch.from_numpy(data), spacing, origin, device=DEV)
    plain = _merge_volume(data, spacing, origin)
    img, jac = P.render(vol, _gpu(poses), det, jacobian=True)
    old, old_jac = P.render(plain, _gpu(poses), det, jacobian=True)
    assert torch.equal(P.render(vol, _gpu(poses), det), img)
    scale = max(old.max().item(), 1e-6)
    assert (img - old).abs().max().item() <= 2e-7 * scale
    both, cnt = P.render_count(vol, _gpu(poses), det)
    assert torch.equal(both, img) and torch.equal(cnt, P.render_count(plain, _gpu(poses), det)[1])
    grid = oracle.Grid(data, spacing, origin)
    ref, rjac = oracle.render_jacobian(grid, poses.astype(np.float64), H, W, pitch, pitch)
    assert_image_close(img.cpu().numpy(), ref, what=str(dims))
    ok = np.isfinite(rjac).all(axis=-1) & (ref > 0)
    # (views 1 to 3 run along axes: their derivatives are kinks)
    ok[1:4] = False
    if ok.any():
        assert max(column_errors(jac.cpu().numpy()[ok], rjac[ok])) <= 2e-4
    assert old_jac.shape == jac.shape


@pytest.mark.parametrize("value", [1e9, float("inf"), float("nan")])
def test_volumes_beyond_the_tables_range_are_traced_by_the_merge(value):
    """One voxel that would dwarf the quantum of its axes' tables: renders are
    bitwise those of a volume without tables, for every ray."""
    import paper_2208_12737_amd as P
    rng = np.random.default_rng(4)
    data = rng.uniform(0.0, 2.0, (33, 20, 41)).astype(np.float32)
    spacing, origin = (1.0, 1.3, 0.9), (-16.0, -13.0, -18.0)
    data[16, 10, 20] = value
    poses = random_poses(5, 0.6, 6.0, 300.0, seed=3)
    poses[3, 0] += math.pi / 2
    det = P.Detector(37, 45, 2.0, 2.0)
    vol = P.Volume(torch.from_numpy(data), spacing, origin, device=DEV)
    plain = _merge_volume(data, spacing, origin)
    same = dict(rtol=0.0, atol=0.0, equal_nan=True)
    torch.testing.assert_close(P.render(vol, _gpu(poses), det), P.render(plain, _gpu(poses), det),
                               **same)
    target = P.render(plain, _gpu(poses[:1]), det)[0].nan_to_num(0.0, 0.0, 0.0)
    for a, b in zip(P.render_ncc_grad(vol, _gpu(poses), det, target),
                    P.render_ncc_grad(plain, _gpu(poses), det, target)):
        torch.testing.assert_close(a, b, **same)


@pytest.mark.parametrize("dims,n", [((60, 50, 70), 200), ((216, 216, 220), 6),
                                    ((216, 216, 220), 40)])
def test_launch_shapes_give_the_same_bits(dims, n):
    """A pose alone (about a wave per SIMD), in a batch of single tiles and, on
    the larger volume, in one of two tiles a workgroup with an odd number of
    tile rows: images, losses and gradients are bitwise equal, and so are
    those of a plan's items."""
    import paper_2208_12737_amd as P
    from paper_2208_12737_amd.plan import Item, Plan, objective_item
    g = torch.Generator(device=DEV).manual_seed(5)
    data = torch.rand(dims, device=DEV, generator=g)
    vol = P.Volume(data, (1.0, 1.1, 0.9), device=DEV)
    det = P.Detector(141, 150, 1.9, 1.8)          # 9 x 10 tiles
    poses = _gpu(random_poses(n, 0.5, 10.0, 900.0, seed=6))
    poses[1, 0] += math.pi / 4                       # rays of two directions in a wave
    img = P.render(vol, poses, det)
    target = img[3].clone()
    loss, grad = P.render_ncc_grad(vol, poses, det, target)
    l2, g2, _ = P.render_l2(vol, poses, det, target, return_image=True)
    only = P.render_ncc_loss(vol, poses, det, target)
    for k in (0, 1, n - 1):
        p = poses[k:k + 1].clone()
        assert torch.equal(P.render(vol, p, det)[0], img[k])
        one = P.render_ncc_grad(vol, p, det, target)
        assert torch.equal(one[0][0], loss[k]) and torch.equal(one[1][0], grad[k])
        two = P.render_l2(vol, p, det, target)
        assert torch.equal(two[0][0], l2[k]) and torch.equal(two[1][0], g2[k])
        assert torch.equal(P.render_ncc_loss(vol, p, det, target)[0], only[k])
    for strategy in (0, 1):
        plan = Plan([vol], max_items=2 * n, strategy=strategy)
        out = torch.empty_like(img)
        items = [Item(0, det, poses[k], out[k]) for k in range(n)]
        items += [objective_item(0, det, poses[k], target) for k in range(n)]
        plan.execute(items)
        assert torch.equal(out, img)
        assert torch.equal(torch.cat([it.loss for it in items[n:]]), loss)
        assert torch.equal(torch.stack([it.grad for it in items[n:]]), grad)
        plan.close()
