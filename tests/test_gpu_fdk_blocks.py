"""The FDK backprojector and the flattening at the edges of their work split,
against the FP64 oracle: blocks of 16 x 16 x 16 voxels cut on every axis,
footprints staged at both row pitches, cut by the detector on every side or off
it, too large to stage, and more views than the footprint table holds; the
flattening's row and view slices.

Tolerance rel-L2 1e-4, the projectors' parity bar: FP32 positions carry three
roundings of a sum that counts pixels from the detector's corner (5e-5 of a pixel at
300 pixels), and neighbouring pixels of the projections are independent; a tap
from a wrong pixel shows at 1e-2 and more."""
import numpy as np
import pytest

import synth
from synth import CurvedDetector, Geometry

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


# volume (z, y, x), detector, pixel (mm; voxels of 1 mm, magnification 1.5), offset (v, u), views
@pytest.mark.parametrize("n,det,pix,off,views", [
    ((1, 1, 1), (2, 3), 1.0, (0.0, 0.0), 1),
    ((16, 16, 16), (40, 40), 1.2, (0.2, -0.3), 33),
    ((17, 15, 33), (50, 75), 0.9, (0.2, -0.3), 70),      # narrow pitch, three tables of views
    ((31, 18, 40), (120, 160), 0.58, (0.4, 0.3), 18),    # wide pitch
    ((18, 20, 22), (200, 230), 0.25, (0.4, 0.3), 5),     # read from global memory
    ((40, 37, 43), (21, 25), 1.1, (3.0, -7.0), 20),      # the detector cuts and misses blocks on every side
    ((40, 37, 43), (5, 300), 0.7, (0.0, 0.0), 9),        # fewer rows than a block's footprint
    ((5, 40, 40), (60, 3), 1.0, (0.0, 2.0), 9),          # rows narrower than a group of four
])
def test_backprojector_blocks(P, orc, n, det, pix, off, views):
    geo = Geometry(DSD=900.0, DSO=600.0, nVoxel=n, dVoxel=(1.0, 1.0, 1.0), nDetector=det, dDetector=(pix, pix),
                   offOrigin=(0.3, -0.4, 0.2), offDetector=off)
    ang = synth.circular_angles(views) + 0.013
    y = np.random.Generator(np.random.PCG64(51)).standard_normal((views,) + det).astype(np.float32)
    buf = torch.full((y.size + 514,), float("nan"), device="cuda")   # rows on 4 bytes only, poison around
    yd = buf[257:257 + y.size].view(y.shape)
    yd.copy_(torch.from_numpy(y))
    plan = P.Plan(geo, ang)
    got = plan.backproject(yd, kind="fdk")
    assert torch.equal(got, plan.backproject(yd, kind="fdk"))
    want = orc.bfdk(geo, ang, y.astype(np.float64))
    assert np.linalg.norm(got.cpu().numpy() - want) <= 1e-4 * np.linalg.norm(want) + 1e-30
    acc = got.clone()
    plan.backproject(yd, out=acc, kind="fdk", beta=2.0)
    assert np.linalg.norm(acc.cpu().numpy() - 3.0 * want) <= 3e-4 * np.linalg.norm(want) + 1e-30


@pytest.mark.parametrize("nv,nu,views", [(1, 1, 3), (17, 65, 1), (16, 64, 40), (300, 130, 5)])
def test_flatten_slices(P, orc, nv, nu, views):
    geo = Geometry(DSD=900.0, DSO=600.0, nVoxel=(8, 8, 8), dVoxel=(1.0, 1.0, 1.0), nDetector=(nv, nu), dDetector=(1.1, 0.9))
    cd = CurvedDetector(nDetector=(nv + 3, nu + 5), dDetector=(1.05, 0.95), radius=900.0, offDetector=(0.3, -0.4))
    q = np.random.Generator(np.random.PCG64(52)).random((views,) + cd.nDetector).astype(np.float32)
    plan = P.Plan(geo, synth.circular_angles(views))
    got = plan.flatten_curved(torch.from_numpy(q).cuda(), cd).cpu().numpy().astype(np.float64)
    want = orc.flatten_curved(geo, cd, q)
    assert _rel(got, want) < 1e-5


@pytest.mark.parametrize("kind", ["fdk", "siddon", "interp"])
@pytest.mark.parametrize("beta", [0.0, 2.0])
def test_call_without_views(P, kind, beta):
    """A range of no views scales the volume by beta and reads no projection
    (none is given), also right after a call whose footprints are still in LDS."""
    geo = Geometry(DSD=900.0, DSO=600.0, nVoxel=(17, 35, 33), dVoxel=(1.0, 1.0, 1.0), nDetector=(50, 75),
                   dDetector=(0.9, 0.9))
    plan = P.Plan(geo, synth.circular_angles(20))
    y = torch.from_numpy(np.random.Generator(np.random.PCG64(53)).random((20, 50, 75)).astype(np.float32)).cuda()
    vol = plan.backproject(y, kind=kind)
    want = beta * vol
    plan.backproject(torch.empty((0, 50, 75), device="cuda"), out=vol, kind=kind, beta=beta, view0=20, nviews=0)
    assert torch.equal(vol, want)


@pytest.mark.parametrize("n,det,pix", [((17, 35, 33), (50, 75), 0.9), ((18, 20, 22), (200, 230), 0.25)])
def test_infinite_pixel_stays_an_infinity(P, orc, n, det, pix):
    """Staged and read from global memory: voxels that the pixels reach with some
    weight hold their infinity, the sum's other voxels are finite, none is NaN.
    (A FP32 position may lie 1e-4 of a pixel to the other side of the tap's edge:
    weights from 0 to 1e-3 are left open.)"""
    geo = Geometry(DSD=900.0, DSO=600.0, nVoxel=n, dVoxel=(1.0, 1.0, 1.0), nDetector=det, dDetector=(pix, pix),
                   offOrigin=(0.3, -0.4, 0.2), offDetector=(0.2, -0.3))
    ang = synth.circular_angles(7) + 0.013
    y = np.random.Generator(np.random.PCG64(54)).standard_normal((7,) + det).astype(np.float32)
    mark = np.zeros(y.shape)
    for k, v, u in ((1, det[0] // 2, det[1] // 2), (4, det[0] // 2 + 1, det[1] // 2 - 3)):
        y[k, v:v + 4, u:u + 4] = np.inf
        mark[k, v:v + 4, u:u + 4] = 1.0
    w = orc.bfdk(geo, ang, mark)
    got = P.Plan(geo, ang).backproject(torch.from_numpy(y).cuda(), kind="fdk").cpu().numpy()
    assert (w > 1e-3).sum() > 20
    assert not np.isnan(got).any()
    assert np.isposinf(got[w > 1e-3]).all()
    assert np.isfinite(got[w == 0.0]).mean() > 0.99 and np.isfinite(got).any()


# volume, voxel (z, y, x), detector, pixel (v, u), offset (v, u), views; magnification 1.5
@pytest.mark.parametrize("n,dvox,det,pix,off,views", [
    ((21, 18, 35), (1.0, 1.0, 1.0), (70, 64), (0.5, 0.9), (0.2, -0.3), 18),     # 8 planes, 48 rows
    ((8, 33, 17), (2.0, 1.0, 1.0), (50, 70), (0.9, 1.1), (1.3, 0.4), 35),       # thick slices, one layer
    ((19, 20, 31), (1.0, 1.0, 1.0), (161, 50), (0.2, 0.9), (0.2, -0.3), 17),    # 96 rows
    ((9, 16, 16), (3.0, 1.0, 1.0), (90, 31), (0.31, 1.0), (-2.0, 5.0), 33),     # 96 rows, cut on two sides
    ((25, 35, 18), (1.0, 1.0, 1.0), (90, 95), (0.45, 0.58), (0.2, -0.3), 16),   # 80 columns, 8 planes
    ((33, 31, 18), (1.0, 1.0, 1.0), (52, 170), (1.0, 0.3), (0.2, -0.3), 19),    # 128 columns, 32 rows
    ((15, 18, 33), (1.0, 1.0, 1.0), (60, 181), (0.5, 0.3), (-1.0, 6.0), 18),    # 128 columns, 8 planes
    ((15, 35, 33), (1.0, 1.0, 1.0), (60, 260), (0.5, 0.22), (0.2, -0.3), 9),    # some views wider than that
    ((40, 18, 33), (1.0, 1.0, 1.0), (500, 60), (0.12, 0.9), (0.2, -0.3), 7),    # some blocks higher than 96 rows
    ((20, 18, 33), (1.0, 1.0, 1.0), (9, 181), (0.45, 0.3), (0.0, 0.0), 9),      # fewer rows than a pass
])
def test_backprojector_shapes_of_footprints(P, orc, n, dvox, det, pix, off, views):
    geo = Geometry(DSD=900.0, DSO=600.0, nVoxel=n, dVoxel=dvox, nDetector=det, dDetector=pix,
                   offOrigin=(0.3, -0.4, 0.2), offDetector=off)
    ang = synth.circular_angles(views) + 0.013
    y = np.random.Generator(np.random.PCG64(55)).standard_normal((views,) + det).astype(np.float32)
    buf = torch.full((y.size + 514,), float("nan"), device="cuda")   # rows on 4 bytes only, poison around
    yd = buf[257:257 + y.size].view(y.shape)
    yd.copy_(torch.from_numpy(y))
    plan = P.Plan(geo, ang)
    got = plan.backproject(yd, kind="fdk")
    assert torch.equal(got, plan.backproject(yd, kind="fdk"))
    assert _rel(got.cpu().numpy().astype(np.float64), orc.bfdk(geo, ang, y.astype(np.float64))) < 1e-4
