"""The (adaptive-weighted) TV gradient at the edges of its work split (waves of
62 x 8 voxels marching over 4 or 8 planes, four to a workgroup) against the FP64
oracle, and a repeat that must give the same bits.  Bar 1e-5 relative: FP32 terms
take about ten roundings each and a voxel sums four of them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2412_10129_amd as P
    return P


@pytest.mark.parametrize("delta", [float("inf"), 0.25])
@pytest.mark.parametrize("shape", [(4, 8, 62), (5, 9, 63), (3, 33, 61), (8, 31, 125), (9, 65, 2), (130, 257, 310), (2, 2, 2)])
def test_awtv_grad_tiles(P, orc, delta, shape):
    from paper_2412_10129_amd import ops
    rng = np.random.Generator(np.random.PCG64(61))
    x = rng.random(shape) * 0.3
    x[shape[0] // 3: 2 * shape[0] // 3 + 1, shape[1] // 4: 3 * shape[1] // 4 + 1, 2:] += 1.0
    x = x.astype(np.float32)
    buf = torch.full((x.size + 514,), float("nan"), device="cuda")   # rows on 4 bytes only, poison around
    xd = buf[257:257 + x.size].view(shape)
    xd.copy_(torch.from_numpy(x))
    got = ops.awtv_grad(xd, delta=delta, eps=1e-8)
    for _ in range(3):
        assert torch.equal(got, ops.awtv_grad(xd, delta=delta, eps=1e-8))
    want = orc.awtv_grad(x.astype(np.float64), delta, 1e-8)
    assert np.linalg.norm(got.cpu().numpy() - want) < 1e-5 * np.linalg.norm(want)


def test_delta_with_an_infinite_square_is_plain_tv(P):
    """delta^2 overflows, so that every weight is 1, also where a difference's square does."""
    from paper_2412_10129_amd import ops
    rng = np.random.Generator(np.random.PCG64(62))
    x = torch.from_numpy((rng.random((5, 9, 70)) * 5e19).astype(np.float32)).cuda()
    assert torch.equal(ops.awtv_grad(x, delta=1e20), ops.awtv_grad(x, delta=float("inf")))
