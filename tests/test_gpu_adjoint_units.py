"""The fixed-point unit of the adjoints where a quotient shows it: A_s^T r /
A_s^T 1 of SART and EM steps, voxel by voxel, on a volume wider than its detector
(voxels at the cones' edges are reached by a few samples of small weight), for
interpolated blocks of more than 32 views and Siddon blocks of 1 to 36.

Reference: the same rays, one view, one octave of |y| and one of 16 pixel patterns at a
time, summed in FP64.  There a unit is at most 2^-30 F times 32 values within a
factor of two (F: the most one ray adds to one cell per unit y).

Tolerance: a group of at most 16 Siddon or 32 interpolated views scales N F max |y|
to more than 2^29, N the rays on a cell in all of them: (floor(2 h s) + 1)^2 a view,
h = 1/2 (Siddon) or 1 the support's half width and s < 3 the pixels that one
voxel's step along every axis moves a projection by (magnification at most
400 + 200 over 400 - 77, sqrt 2 for the two axes across the ray, 0.4 along it).  A cell takes n
terms (Siddon 16 rays a view, interpolated 16 with five samples), each rounded to
half a unit, so their sum is normal with a variance of n / 12 units; the bar is
seven of its standard deviations (1e-12 per voxel), for the numerator and for
A_s^T 1 in the quotient, and 2^-20 of the quotient for the FP32 sums over the groups."""
import numpy as np
import pytest

import synth
from synth import Geometry

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

N = (96, 112, 104)


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2412_10129_amd as P
    return P


def _fine(plan, y, kind):
    acc = torch.zeros(plan.vol_shape, dtype=torch.float64, device="cuda")
    iv = torch.arange(y.shape[1], device="cuda")[:, None]
    iu = torch.arange(y.shape[2], device="cuda")[None, :]
    pattern = iv % 4 * 4 + iu % 4
    for k in range(y.shape[0]):
        e = torch.frexp(y[k].abs())[1]
        top = int(e.max())
        e = e.clamp_min(top - 12)
        for o in torch.unique(e[y[k] != 0]).tolist():
            for q in range(16):
                part = torch.where((e == o) & (pattern == q), y[k], torch.zeros_like(y[k]))
                acc += plan.backproject(part[None].contiguous(), kind=kind, view0=k, nviews=1)
    return acc


@pytest.mark.parametrize("kind,block", [("interp", 36), ("interp", 64), ("siddon", 1), ("siddon", 2), ("siddon", 5),
                                        ("siddon", 12), ("siddon", 36)])
@pytest.mark.parametrize("det,pix", [((70, 90), 1.0), ((22, 28), 3.3)])   # batches of one view, and over the views' ends
def test_quotients_keep_weakly_reached_voxels(P, kind, block, det, pix):
    from paper_2412_10129_amd import algs, ops
    geo = Geometry(DSD=600.0, DSO=400.0, nVoxel=N, dVoxel=(1.0, 1.0, 1.0), nDetector=det, dDetector=(pix, pix),
                   offOrigin=(0.4, -0.3, 0.6), offDetector=(0.3, -0.2))
    plan = P.Plan(geo, synth.circular_angles(64) + 0.013)
    z, y, x = (torch.linspace(-1, 1, n, device="cuda") for n in N)
    ball = ((z[:, None, None] / 0.8) ** 2 + (y[None, :, None] / 0.62) ** 2 + (x[None, None, :] / 0.7) ** 2 < 1).float()
    ball += 0.6 * (((z[:, None, None] - 0.2) / 0.3) ** 2 + ((y[None, :, None] + 0.2) / 0.2) ** 2 +
                   ((x[None, None, :] - 0.1) / 0.25) ** 2 < 1).float()
    b = plan.forward(ball, kind=kind)
    rng = np.random.Generator(np.random.PCG64(71))
    cnt = torch.from_numpy(rng.poisson(1e5 * np.exp(-0.02 * b.cpu().numpy().astype(np.float64))).astype(np.float32)).cuda()
    b = -torch.log(cnt.clamp_min(1.0) / 1e5) / 0.02
    sart = algs.OSSART(plan, block, kind)
    xs = torch.zeros(N, device="cuda")
    first = (sart.W[:block] * b[:block]).contiguous()
    sart.sweep(xs, b)
    later = sart.W[:block] * (b[:block] - plan.forward(xs, kind=kind, view0=0, nviews=block))
    ratio = ops.em_ratio(b[:block].contiguous(), plan.forward(torch.ones(N, device="cuda"), kind=kind, view0=0, nviews=block),
                         torch.empty_like(later))

    half, group, samples = (1.0, 16, 1) if kind == "siddon" else (2.0, 32, 5)
    F = float(np.sqrt(3.0)) if kind == "siddon" else 0.5 * (np.floor(4 * np.sqrt(3.0)) + 2)
    rays = group * (np.floor(half * 3.0) + 1.0) ** 2
    sd = np.sqrt(16 * samples * block / 12.0)

    def bar(v):
        m = float(v.abs().max())
        return 7.0 * sd * F * m * (rays * 2.0 ** -29 + 64 * 2.0 ** -30)

    ones = torch.ones_like(first)
    s = plan.backproject(ones, kind=kind, view0=0, nviews=block).double()
    s_ref = _fine(plan, ones, kind)
    assert bool(((s - s_ref).abs() <= bar(ones) + 2.0 ** -20 * s_ref).all())
    reached = s > 0
    assert float(s[reached].min()) < 1e-2 * float(s.max())   # the cones' edges are in the volume
    for v in (first, later, ratio):
        r = plan.backproject(v.contiguous(), kind=kind, view0=0, nviews=block).double()
        r_ref = _fine(plan, v, kind)
        q, q_ref = r[reached] / s[reached], r_ref[reached] / s_ref[reached].clamp_min(1e-30)
        tol = (bar(v) + q_ref.abs() * bar(ones)) / s[reached] + 2.0 ** -20 * q_ref.abs()
        both = s_ref[reached] > 0
        assert bool(((q - q_ref).abs() <= tol)[both].all())
