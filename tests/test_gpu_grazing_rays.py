"""Siddon rays that run within micrometres of a voxel plane, almost parallel to
it, and cross it inside the volume: one detector row `height` mm above or below
the source, volumes shifted so that the crossing lies within the 48 mm that a ray
spends in them (what a calibrated geometry gives).  Where such a ray enters the
volume (the adjoint: a brick), the cell of its FP32 position and the FP32
parameter at which it crosses the plane disagree by up to several voxels of
path: the walk may start in a cell that it has, by its own crossing order,
already left, and has no length there, never a negative one.  (An FP32 model of
the walk's start gives 45, 161, 771 and 843 such entries among 400 views at these
heights, of 0.3, 1.4, 5.9 and 23 voxels at most.)"""
import numpy as np
import pytest

import synth
from synth import Geometry

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

NZ, NXY, NU, PLANE, VIEWS = 256, 48, 64, 250, 400
GEO = Geometry(DSD=800.0, DSO=450.0, nVoxel=(NZ, NXY, NXY), dVoxel=(1.0, 1.0, 1.0), nDetector=(1, NU),
               dDetector=(1.0, 1.0))
HEIGHTS = [2.0 ** -6, 2.0 ** -8, 2.0 ** -10, 2.0 ** -12]


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2412_10129_amd as P
    return P


def _views(height):
    rng = np.random.Generator(np.random.PCG64(61))
    dv = height * (1.0 - rng.uniform(0.0, 0.05, VIEWS)) * rng.choice([-1.0, 1.0], VIEWS)
    # the source's height in voxels above the volume's lowest face, crossing PLANE within 3 % of the ray
    src = PLANE - dv * GEO.DSO / GEO.DSD + rng.uniform(-0.03, 0.03, VIEWS) * dv
    off = np.zeros((VIEWS, 3))
    det = np.zeros((VIEWS, 2))
    off[:, 0] = NZ / 2 - src
    det[:, 0] = dv
    return synth.views(GEO, rng.uniform(0.0, 2.0 * np.pi, VIEWS), offOrigin=off, offDetector=det)


@pytest.mark.parametrize("height", HEIGHTS)
def test_adjoint_of_ones_is_not_negative(P, height):
    """Every entry of A is a length: A_k^T 1 >= 0 view by view, exactly (a sum of
    non-negative fixed-point terms)."""
    plan = P.Plan(GEO, _views(height))
    y = torch.ones((1, 1, NU), device="cuda")
    out = torch.empty(GEO.nVoxel, device="cuda")
    low, high = torch.zeros(VIEWS, device="cuda"), torch.zeros(VIEWS, device="cuda")
    for k in range(VIEWS):
        plan.backproject(y, out=out, kind="siddon", view0=k, nviews=1)
        low[k], high[k] = out.min(), out.max()
    assert float(low.min()) == 0.0 and float(high.min()) > 0.5


@pytest.mark.parametrize("height", HEIGHTS)
def test_forward_stays_between_the_layers(P, height):
    """A volume of 1 below the plane and 0 above it: every ray's sum lies between 0
    and the ray's length, and the sums of the two halves add up to the length
    (1e-5 of it: some tens of FP32 roundings of the accumulated lengths)."""
    plan = P.Plan(GEO, _views(height))
    x = torch.zeros(GEO.nVoxel, device="cuda")
    x[:PLANE] = 1.0
    low, high, both = (plan.forward(t, kind="siddon") for t in (x, 1.0 - x, torch.ones_like(x)))
    assert float(low.min()) >= 0.0 and float(high.min()) >= 0.0
    assert bool(((low + high - both).abs() <= 1e-5 * both).all())


@pytest.mark.parametrize("height", HEIGHTS)
def test_pair_stays_matched(P, height):
    """<A x, y> = <x, A^T y> to 1e-6, the bar of rays that graze a brick face."""
    plan = P.Plan(GEO, _views(height))
    w = torch.from_numpy(synth.uniform_volume(GEO, 62)).cuda()
    y = torch.from_numpy(synth.uniform_projections(GEO, VIEWS, 63)).cuda()
    lhs = float(P.dot(plan.forward(w, kind="siddon"), y))
    rhs = float(P.dot(w, plan.backproject(y, kind="siddon")))
    assert abs(lhs - rhs) <= 1e-6 * abs(lhs)
