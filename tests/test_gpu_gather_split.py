"""Connection of points to forward paths at the edges of its two splits (one
wavefront for four points below 2,048 on a 256-CU device, a quarter beyond) and
of the paths' ranges: fewer paths than lanes, one path over, whole chunks."""
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


@pytest.mark.parametrize("P,N,M", [(1, 2, 1), (3, 1025, 2), (2047, 130, 3), (2048, 129, 1), (2065, 7, 4),
                                   (2070, 4097, 2), (5, 32769, 1)])
@pytest.mark.parametrize("dim,precision", [(3, "f32"), (2, "f32"), (3, "f64"), (2, "f64")])
def test_gather_splits(W, dim, precision, P, N, M):
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
    # squares carry twice the relative error, of a path's own absolute sum: the
    # mean square bounds it where values cancel
    got = var.cpu().double().numpy()
    assert np.all(np.abs(got - ov) <= 1e-3 * np.maximum(ov, om ** 2) if f32 else
                  np.abs(got - ov) <= 1e-9 * np.maximum(ov, om ** 2))
    scene.close()
