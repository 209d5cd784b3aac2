"""Add-back of the control variate at the edges of its two splits (32,768 points
on a 256-CU device), of its tiles of 512 triangles and of the queue of near
pairs: points on the surface, at a triangle's centre and far off, in number from
one to a few past whole wavefronts and workgroups."""
import numpy as np
import pytest

import oracle
from paper_2305_04403_amd import inputs as I
from tests import parity as PT
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


# triangles: 20, 500, 1,280 (2.5 tiles), 1,620
@pytest.mark.parametrize("P", [1, 31, 33, 257, 32767, 32768, 33025])
@pytest.mark.parametrize("size", [1, 5, 8, 9])
def test_addback_splits(W, size, P):
    mesh = PT.f32_mesh(I.perturb_radial(I.icosphere(size), 0.1, 3, 4))
    tri = mesh.verts[mesh.prims]
    rng = np.random.default_rng(size)
    g = PT.f32(rng.standard_normal(mesh.n_prims))
    pts = I.ball_points(P, 1.5, 7)
    on = rng.integers(0, mesh.n_prims, P)
    pts[::2] = (tri[on].mean(1) * (1 + 0.02 * rng.standard_normal((P, 1))))[::2]
    pts[::7] = tri[on].mean(1)[::7]
    pts[::11] *= 30
    pts = PT.f32(pts)
    scene = W.Scene(mesh, W.F32)
    out = W.cv_addback(scene, dev(g, torch.float32), dev(pts, torch.float32), seed=9)
    torch.cuda.synchronize()
    got = out.cpu().double().numpy()
    assert np.isfinite(got).all()
    keep = np.unique(np.concatenate([np.arange(min(P, 40)), np.arange(max(P - 40, 0), P)]))
    om = oracle.OracleMesh(mesh)
    ref = oracle.cv_addback(om, g, pts[keep], seed=9, randomized=True)
    scale = oracle.cv_addback(om, np.abs(g), pts[keep])
    # the bar of the whole-mesh comparison: a few binary32 units per closed form
    # and per sum of the triangles
    err = np.abs(got[keep] - ref) / scale
    assert err.max() < 2e-5, err.max()
    scene.close()
