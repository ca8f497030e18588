"""The matched adjoints where one brick's footprint holds millions of pixels:
the lane order's quotients beyond what an FP32 reciprocal gives exactly, and a
group of views whose pixels number more than 2^31."""
import numpy as np
import pytest

from synth import Geometry

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2412_10129_amd as P
    return P


@pytest.mark.parametrize("hp", [102581, 102582])
def test_last_row_of_a_tall_footprint(P, orc, hp):
    """A footprint of 8 hp rows by 8 columns (lanes in 8 x 8 classes of hp rows):
    for hp = 102581 the FP32 quotient of the last pixel of the last class rounds
    up to 64.  Only that pixel's ray is lit.  Tolerance 1e-4, the projectors'
    parity bar."""
    nv = 8 * hp
    geo = Geometry(DSD=900.0, DSO=600.0, nVoxel=(1, 1, 1), dVoxel=(1.0, 1.0, 1.0), nDetector=(nv, 8),
                   dDetector=(1.4 / nv, 0.17))
    ang = np.array([0.2])
    y = np.zeros((1, nv, 8), dtype=np.float32)
    y[0, nv - 1, 7] = 1.0
    plan = P.Plan(geo, ang)
    got = float(plan.backproject(torch.from_numpy(y).cuda(), kind="siddon").cpu())
    want = float(orc.backward(geo, ang, y, "siddon").item())
    assert want > 0.5 and abs(got - want) <= 1e-4 * want


def test_group_of_more_pixels_than_an_int32_holds(P):
    """Nine views of 2^28 - 4096 pixels form one group on a small volume.  With one
    pixel of 10^6 among values of 10^-3 the others must keep a unit of their
    own (they fall below half of the hot pixel's), so the voxels its ray does not
    reach hold the same sum as without it.  The values lie in 512 rows through the
    volume's middle (the rest is 0 to keep the one workgroup's work short).
    Tolerance 1e-2: the unit of |y| <= 8 mean |y| = 3.3e-3 is a third of the
    rays' entries (10^7 rays per view and cell at 2^30), and the roundings of
    the 10^5 rays and more that reach a cell average out to a part in 10^3."""
    nv, nu, views = 65535, 4096, 9
    geo = Geometry(DSD=900.0, DSO=600.0, nVoxel=(4, 4, 4), dVoxel=(1.0, 1.0, 1.0), nDetector=(nv, nu),
                   dDetector=(7.0 / nv, 7.0 / nu))
    plan = P.Plan(geo, 0.1 + 0.6 * np.arange(views))
    y = torch.zeros((views, nv, nu), device="cuda")
    y[:, nv // 2 + 1000:nv // 2 + 1512] = 1e-3
    dim = plan.backproject(y, kind="siddon").cpu().numpy().astype(np.float64)
    lit = torch.zeros((1, nv, nu), device="cuda")
    lit[0, nv // 2 + 1200, nu // 2] = 1.0
    reached = plan.backproject(lit, kind="siddon", nviews=1).cpu().numpy() > 0
    y[0, nv // 2 + 1200, nu // 2] = 1e6
    both = plan.backproject(y, kind="siddon").cpu().numpy().astype(np.float64)
    look = ~reached & (dim > 0.5 * dim.max())
    assert 0 < reached.sum() < 32 and look.sum() > 4
    assert (np.abs(both - dim)[look] <= 1e-2 * dim[look]).all()
