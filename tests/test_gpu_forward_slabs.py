"""The forward projectors' staging at its edges, against the FP64 oracle: slabs
fitted to the tile and boxes of every capacity (pixels from a third of a voxel to
several voxels), volumes narrower than one group of four voxels or thinner than
one slab, rows that do not start or end on a group, more slabs than the table
holds, and views whose rays run mostly along z.

Tolerance rel-L2 1e-4, the projectors' parity bar (FP32 positions: 1e-5 of a
path length)."""
import numpy as np
import pytest

import synth
from synth import Geometry

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _rel(a, b):
    return float(np.linalg.norm(a.ravel() - b.ravel()) / np.linalg.norm(b.ravel()))


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2412_10129_amd as P
    return P


def _check(P, orc, geo, ang, kind, seed):
    x = np.random.Generator(np.random.PCG64(seed)).random(geo.nVoxel).astype(np.float32)
    # the volume ends where its allocation does, with poison around it
    buf = torch.full((x.size + 512,), float("nan"), device="cuda")
    vol = buf[257:257 + x.size].view(x.shape)   # rows on 4 bytes only
    vol.copy_(torch.from_numpy(x))
    plan = P.Plan(geo, ang)
    got = plan.forward(vol, kind=kind)
    assert torch.equal(got, plan.forward(vol, kind=kind))
    assert _rel(got.cpu().numpy().astype(np.float64), orc.forward(geo, ang, x.astype(np.float64), kind)) < 1e-4


# volume (z, y, x), detector, pixel (mm; magnification 1.5, voxels of 1 mm)
CASES = [
    ((1, 1, 1), (3, 3), 0.4),
    ((5, 6, 3), (9, 20), 0.5),        # narrower than a group
    ((6, 3, 7), (17, 16), 0.7),
    ((2, 70, 66), (5, 130), 0.9),     # thin: one slab's boxes of few planes
    ((40, 37, 43), (61, 66), 0.5),
    ((40, 37, 43), (64, 60), 1.35),   # the second capacity
    ((40, 50, 43), (40, 48), 2.0),    # the third
    ((40, 50, 43), (20, 24), 4.0),    # the widest, clipped
    ((9, 5, 371), (20, 400), 1.4),    # more slabs than the table holds, along x
    ((9, 371, 6), (20, 400), 1.4),    # and along y
]


@pytest.mark.parametrize("kind", ["siddon", "interp"])
@pytest.mark.parametrize("n,det,pix", CASES)
def test_forward_at_the_edges_of_staging(P, orc, n, det, pix, kind):
    geo = Geometry(DSD=900.0, DSO=600.0, nVoxel=n, dVoxel=(1.0, 1.0, 1.0), nDetector=det, dDetector=(pix, pix),
                   offOrigin=(0.3, -0.4, 0.2), offDetector=(0.2, -0.3))
    ang = np.array([0.0, 0.013, 0.4, 0.78, 1.2, np.pi / 2, 2.36, 3.2, 4.4, 5.5])
    _check(P, orc, geo, ang, kind, 41 + n[2])


@pytest.mark.parametrize("kind", ["siddon", "interp"])
@pytest.mark.parametrize("n,pix", [((37, 30, 41), 0.8), ((150, 6, 9), 1.5)])
def test_rays_along_z(P, orc, n, pix, kind):
    """Orbits tilted by 1.3 rad: the tiles' dominant axis is z."""
    geo = Geometry(DSD=900.0, DSO=600.0, nVoxel=n, dVoxel=(1.0, 1.0, 1.0), nDetector=(50, 60), dDetector=(pix, pix),
                   offOrigin=(0.3, -0.4, 0.2), offDetector=(0.2, -0.3))
    k = np.arange(6)
    views = synth.views(geo, np.stack([0.3 + k, 1.3 + 0.02 * k, 0.1 * k], axis=1))
    _check(P, orc, geo, views, kind, 43)


@pytest.mark.parametrize("accuracy", [0.9, 1.0, 1.5, 2.0, 3.7])
@pytest.mark.parametrize("h", [(1.0, 1.0, 1.0), (2.5, 1.0, 1.2)])
def test_steps_of_a_voxel_and_more(P, orc, accuracy, h):
    """Interpolation steps up to several voxels: the samples one step beyond the
    volume at either end of a ray lie outside every staged box and add nothing."""
    geo = Geometry(DSD=900.0, DSO=600.0, nVoxel=(30, 37, 43), dVoxel=h, nDetector=(61, 66), dDetector=(1.1, 0.9),
                   offOrigin=(0.3, -0.4, 0.2), offDetector=(0.2, -0.3), accuracy=accuracy)
    ang = np.array([0.0, 0.013, 0.4, 0.78, 1.2, np.pi / 2, 2.36, 3.2, 4.4, 5.5])
    _check(P, orc, geo, ang, "interp", 47)
    y = np.random.Generator(np.random.PCG64(48)).random((len(ang),) + geo.nDetector).astype(np.float32)
    got = P.Plan(geo, ang).backproject(torch.from_numpy(y).cuda(), kind="interp")
    assert _rel(got.cpu().numpy().astype(np.float64), orc.backward(geo, ang, y.astype(np.float64), "interp")) < 1e-4


@pytest.mark.parametrize("nz", [2400, 3600])
@pytest.mark.parametrize("kind", ["siddon", "interp"])
def test_tall_grids_under_wide_boxes(P, orc, nz, kind):
    """Planes of 1600 words and more in the boxes: byte offsets over the whole grid
    are exact FP32 integers up to about 2600 planes, and box-relative above.  The
    rays cross the highest planes, where inexact offsets would show."""
    geo = Geometry(DSD=5000.0, DSO=2500.0, nVoxel=(nz, 60, 90), dVoxel=(1.0, 1.0, 1.0), nDetector=(40, 30),
                   dDetector=(0.6, 10.0), offDetector=(0.9 * nz, 0.3))
    _check(P, orc, geo, np.array([0.0, 0.05, 0.7, 1.2, np.pi / 2, 3.2, 4.6]), kind, 49)


@pytest.mark.parametrize("n,det,pix", [((40, 45, 50), (60, 70), 1.1), ((20, 30, 25), (120, 130), 0.4)])
def test_siddon_rays_beside_a_nan_stay_finite(P, orc, n, det, pix):
    """Voxels of NaN on the volume's faces: every ray through one is NaN, and none is that
    stays a voxel away from all of them (a ray's walk goes on for the wave's
    other rays after it has left the volume, with lengths of 0)."""
    geo = Geometry(DSD=900.0, DSO=600.0, nVoxel=n, dVoxel=(1.0, 1.0, 1.0), nDetector=det, dDetector=(pix, pix))
    ang = synth.circular_angles(9) + 0.013
    x = np.random.Generator(np.random.PCG64(81)).random(n).astype(np.float32)
    hit, near = np.zeros(n), np.zeros(n)
    for z, y, u in ((n[0] // 3, n[1] // 4, n[2] // 3), (n[0] - 1, 0, n[2] - 1), (0, n[1] // 2, 0), (n[0] // 2, n[1] - 1, n[2] // 2)):
        x[z, y, u] = np.nan
        hit[z, y, u] = 1.0
        near[max(z - 1, 0):z + 2, max(y - 1, 0):y + 2, max(u - 1, 0):u + 2] = 1.0
    got = np.isnan(P.Plan(geo, ang).forward(torch.from_numpy(x).cuda(), kind="siddon").cpu().numpy())
    assert got[orc.forward(geo, ang, hit, "siddon") > 1e-3].all()
    assert not got[orc.forward(geo, ang, near, "siddon") == 0.0].any()
