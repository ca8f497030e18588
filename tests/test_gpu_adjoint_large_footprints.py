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
    """Views of 2^28 - 4096 pixels, a quarter turn apart, on a volume of one brick:
    values of 10^-3 in 512 rows and one pixel of 10^6 in seven views, then the same
    with two views of zeros.  Views of zeros raise the rays per cell and lower the
    mean |y| by the same factor, so the unit of the values below 8 mean |y|, and
    with it every bit, stays; nine such views hold more than 2^31 pixels."""
    nv, nu, views = 65535, 4096, 9
    geo = Geometry(DSD=900.0, DSO=600.0, nVoxel=(4, 16, 16), dVoxel=(1.0, 1.0, 1.0), nDetector=(nv, nu),
                   dDetector=(6.0 / nv, 24.0 / nu))
    plan = P.Plan(geo, 0.1 + 0.5 * np.pi * np.arange(views))
    y = torch.zeros((views, nv, nu), device="cuda")
    y[:7, nv // 2 + 1000:nv // 2 + 1512] = 1e-3
    y[0, nv // 2 + 1200, nu // 2] = 1e6
    seven = plan.backproject(y[:7], kind="siddon", nviews=7)
    assert float(seven.abs().max()) > 100.0
    assert torch.equal(plan.backproject(y, kind="siddon"), seven)
