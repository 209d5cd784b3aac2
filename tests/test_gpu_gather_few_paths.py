"""Connection of many points to few paths: each point's lanes are no more than its
paths can occupy, so the time follows the pairs (8 paths cost a small part of 200
paths, not the same), and the values at the edges of that split."""
import time

import numpy as np
import pytest

import oracle
from paper_2305_04403_amd import inputs as I
from tests import parity as PT
from tests.test_gpu_forward import _neumann
from tests.test_gpu_parity import dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def W():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2305_04403_amd import wob
    wob.lib()
    return wob


def seconds(call):
    best = 1e9
    for _ in range(10):
        torch.cuda.synchronize()
        t = time.perf_counter()
        for _ in range(5):
            call()
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t)
    return best


def test_time_follows_the_pairs(W):
    scene = W.Scene(_neumann(I.icosphere(2)), W.F32)
    pts = (torch.rand(1_000_000, 3, device="cuda") + 1.1).contiguous()
    out = (torch.empty(len(pts), device="cuda"), torch.empty(len(pts), device="cuda"))
    t = {}
    for n in (8, 200):
        vtx = torch.rand(n, 4, 4, device="cuda")
        t[n] = seconds(lambda: W.forward_gather(scene, vtx, pts, out=out))
    # 1 / 25 of the pairs
    assert t[8] < 0.4 * t[200], t
    scene.close()


# no more paths than wavefronts, at most a path for every 100 points (one lane takes
# two points: a wavefront 128), a path for 20,000, more points than 1,000 per CU;
# in between (1,500 x 300 in FP64: a path per lane of 256, below one per point)
@pytest.mark.parametrize("P,N,M", [(1, 8, 3), (200, 9, 2), (799, 8, 2), (3300, 33, 4), (3299, 33, 4), (40001, 2, 2),
                                   (257000, 40, 1), (1500, 300, 2), (250, 300, 2)])
@pytest.mark.parametrize("dim,precision", [(3, "f32"), (2, "f32"), (3, "f64"), (2, "f64")])
def test_few_paths_many_points(W, dim, precision, P, N, M):
    f32 = precision == "f32"
    pos, w = I.forward_records(N, M, dim, 9)
    pts = I.ball_points(P, 2.2, 3, r_min=1.3)[:, :dim]
    pts[::3] *= 0.3
    if f32:
        pos, w, pts = PT.f32(pos), PT.f32(w), PT.f32(pts)
    scene = W.Scene(_neumann(I.icosphere(2) if dim == 3 else I.circle_polygon(8)), W.F32 if f32 else W.F64)
    dt = torch.float32 if f32 else torch.float64
    rec = np.zeros((N, M, 4))
    rec[:, :, :dim] = pos
    rec[:, :, 3] = w
    mean, var = W.forward_gather(scene, dev(rec, dt), dev(pts, dt))
    torch.cuda.synchronize()
    om, ov, oa = oracle.forward_gather(pos, w, pts)
    # a term: distance, root and product at a few units each; a lane's sums of at
    # most 32 paths of 4 vertices: under 64 units of the absolute sum in all
    tol = 64 * (2.0 ** -24 if f32 else 2.0 ** -53)
    err = np.abs(mean.cpu().double().numpy() - om)
    assert np.all(err <= tol * oa), (err / oa).max()
    got = var.cpu().double().numpy()
    # squares carry twice the relative error of a path's own absolute sum, and the
    # sum of squares cancels against the mean's: units of (N oa)^2
    assert np.all(np.abs(got - ov) <= 4 * tol * N * N * oa ** 2)
    scene.close()
