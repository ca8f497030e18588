"""The matched adjoints where one brick's footprint holds millions of pixels:
the lane order's quotients beyond what an FP32 reciprocal gives exactly."""
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
