"""The matched adjoints' brick kernels at the edges of their launch rule,
against the FP64 oracle: volumes of few, some and many 16x16x8 bricks (16, 8
and 8 waves per brick; bricks of 4 or 8, 8 and 16 planes) with ragged sizes in
every axis, the interpolated adjoint at the last view count of its per-round
form and the first of its per-group form, detectors of less than one, one to
two and several pixels per voxel (the lane order's strides), and values that
form a second magnitude class.

Tolerance rel-L2 1e-4, the projectors' parity bar (FP32 positions of rays
re-anchored at the volume: 1e-5 of a path length, summed with random signs)."""
import numpy as np
import pytest

import synth
from synth import Geometry

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _geo(n, det, pix):
    return Geometry(DSD=600.0, DSO=400.0, nVoxel=n, dVoxel=(1.0, 1.0, 1.0), nDetector=det, dDetector=(pix, pix),
                    offOrigin=(0.4, -0.3, 0.6), offDetector=(0.3, -0.2))


FEW = (21, 43, 50)      # 36 bricks
SOME = (66, 120, 116)   # 576
MANY = (249, 120, 122)  # 2048
CASES = [(FEW, (40, 70), 1.1), (FEW, (70, 130), 0.6), (FEW, (14, 20), 5.0), (SOME, (60, 70), 2.4),
         (SOME, (200, 33), 0.7), (MANY, (52, 41), 6.3), (MANY, (90, 40), 4.0)]


def _rel(a, b):
    return float(np.linalg.norm(a.ravel() - b.ravel()) / np.linalg.norm(b.ravel()))


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2412_10129_amd as P
    return P


@pytest.mark.parametrize("kind,views", [("siddon", 5), ("interp", 32), ("interp", 33)])
@pytest.mark.parametrize("n,det,pix", CASES)
def test_adjoint_over_the_launch_rule(P, orc, n, det, pix, kind, views):
    geo = _geo(n, det, pix)
    ang = synth.circular_angles(views) + 0.013
    rng = np.random.Generator(np.random.PCG64(views + det[0]))
    y = rng.standard_normal((views,) + det).astype(np.float32)
    y[rng.random(y.shape) < 0.3] = 0.0
    plan = P.Plan(geo, ang)
    yd = torch.from_numpy(y).cuda()
    got = plan.backproject(yd, kind=kind)
    assert torch.equal(got, plan.backproject(yd, kind=kind))   # integer sums: the same bits
    want = orc.backward(geo, ang, y.astype(np.float64), kind)
    assert _rel(got.cpu().numpy().astype(np.float64), want) < 1e-4
    # beta accumulates onto the volume
    acc = got.clone()
    plan.backproject(yd, out=acc, kind=kind, beta=2.0)
    assert _rel(acc.cpu().numpy().astype(np.float64), 3.0 * want) < 1e-4


@pytest.mark.parametrize("kind,views", [("siddon", 6), ("interp", 40)])
def test_values_far_above_the_rest_keep_the_others_exact(P, orc, kind, views):
    """A few pixels 10^6 times the rest: the voxels their rays do not reach
    hold the same sum as without them, to the same bar."""
    geo = _geo(SOME, (60, 70), 2.4)
    ang = synth.circular_angles(views) + 0.013
    rng = np.random.Generator(np.random.PCG64(5))
    y = rng.random((views, 60, 70)).astype(np.float32) + np.float32(0.1)
    hot = np.zeros_like(y)
    hot[rng.integers(0, views, 5), rng.integers(5, 55, 5), rng.integers(5, 65, 5)] = 1e6
    plan = P.Plan(geo, ang)
    got = plan.backproject(torch.from_numpy(y + hot).cuda(), kind=kind).cpu().numpy().astype(np.float64)
    want = orc.backward(geo, ang, (y + hot).astype(np.float64), kind)
    reached = orc.backward(geo, ang, (hot > 0).astype(np.float64), kind) > 0
    assert 0 < reached.sum() < reached.size // 2
    assert _rel(got[reached], want[reached]) < 1e-4
    assert _rel(got[~reached], want[~reached]) < 1e-4


@pytest.mark.parametrize("kind", ["siddon", "interp"])
@pytest.mark.parametrize("n", [(148, 120, 122), (156, 120, 122)])    # 1216 and 1280 bricks of 8 planes
@pytest.mark.parametrize("det,pix", [((45, 61), (1.5, 0.9)), ((40, 52), (1.2, 1.2)), ((60, 50), (0.6, 1.0))])
def test_adjoint_wide_column_groups(P, orc, n, det, pix, kind):
    """Short columns (one and two row classes: groups of twice the columns per
    voxel) and three row classes (single groups), on both sides of the brick
    height's rule.  Tolerance: the parity bar above."""
    geo = Geometry(DSD=600.0, DSO=400.0, nVoxel=n, dVoxel=(1.0, 1.0, 1.0), nDetector=det, dDetector=pix,
                   offOrigin=(0.4, -0.3, 0.6), offDetector=(0.3, -0.2))
    ang = synth.circular_angles(33) + 0.013
    rng = np.random.Generator(np.random.PCG64(7 * det[0] + n[0]))
    y = rng.standard_normal((33,) + det).astype(np.float32)
    got = P.Plan(geo, ang).backproject(torch.from_numpy(y).cuda(), kind=kind)
    want = orc.backward(geo, ang, y.astype(np.float64), kind)
    assert _rel(got.cpu().numpy().astype(np.float64), want) < 1e-4


TALL = (160, 120, 122)   # 1280 bricks of 8 planes


@pytest.mark.parametrize("kind,views", [("siddon", 8), ("siddon", 9), ("siddon", 35), ("interp", 35)])
@pytest.mark.parametrize("n,det,pix", [
    (FEW, (10, 14), (7.0, 7.0)), (FEW, (3, 40), (4.0, 1.1)), (SOME, (18, 25), (6.0, 6.0)), (SOME, (1, 130), (1.2, 1.0)),
    (SOME, (66, 2), (2.4, 1.0)), (TALL, (40, 30), (7.0, 5.0)), (TALL, (70, 45), (4.0, 3.6)),      # few rays per brick
    (FEW, (210, 330), (0.17, 0.22)), (SOME, (14, 130), (8.0, 1.1)), (MANY, (38, 70), (11.0, 2.1))])   # row classes beyond 8; short columns
def test_adjoint_of_sparse_and_of_dense_footprints(P, orc, n, det, pix, kind, views):
    """Batches over the views' ends (few rays per brick and view), column groups of 4 ku,
    and more than eight pixels per voxel.  Tolerance: the parity bar above."""
    geo = Geometry(DSD=600.0, DSO=400.0, nVoxel=n, dVoxel=(1.0, 1.0, 1.0), nDetector=det, dDetector=pix,
                   offOrigin=(0.4, -0.3, 0.6), offDetector=(0.3, -0.2))
    ang = synth.circular_angles(views) + 0.013
    rng = np.random.Generator(np.random.PCG64(5 * det[0] + views))
    y = rng.standard_normal((views,) + det).astype(np.float32)
    y[rng.random(y.shape) < 0.2] = 0.0
    y[views // 2] = 0.0
    plan = P.Plan(geo, ang)
    got = plan.backproject(torch.from_numpy(y).cuda(), kind=kind)
    assert torch.equal(got, plan.backproject(torch.from_numpy(y).cuda(), kind=kind))
    want = orc.backward(geo, ang, y.astype(np.float64), kind)
    assert _rel(got.cpu().numpy().astype(np.float64), want) < 1e-4
