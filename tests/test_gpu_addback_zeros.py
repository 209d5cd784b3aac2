"""Add-back with tables of zeros: an all-zero table costs a small part of a full
one, and a table with few values gives each of them, wherever its tile lies
(12 tiles of 512 triangles) and on every split of the points over the lanes (from
32,768, 256,000 and 640,000 points on a 256-CU device)."""
import time

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


def test_time_of_a_zero_table(W):
    mesh = PT.f32_mesh(I.perturb_radial(I.icosphere(32), 0.1, 3, 4))
    scene = W.Scene(mesh, W.F32)
    pts = ((torch.rand(200_000, 3, device="cuda") - 0.5) * 6).contiguous()
    zero = torch.zeros(mesh.n_prims, device="cuda")
    full = torch.randn(mesh.n_prims, device="cuda")
    t0, t1 = seconds(lambda: W.cv_addback(scene, zero, pts)), seconds(lambda: W.cv_addback(scene, full, pts))
    assert t0 < 0.1 * t1, (t0, t1)
    assert torch.equal(W.cv_addback(scene, zero, pts), torch.zeros(len(pts), device="cuda"))
    scene.close()


def check(W, scene, om, g, pts, keep):
    got = W.cv_addback(scene, dev(g, torch.float32), dev(pts, torch.float32), seed=9).cpu().double().numpy()
    ref = oracle.cv_addback(om, g, pts[keep], seed=9, randomized=True)
    scale = oracle.cv_addback(om, np.abs(g), pts[keep])
    assert np.isfinite(got).all()
    # the bar of the whole-mesh comparison (a few binary32 units per term and sum)
    err = np.abs(got[keep] - ref) / scale
    assert err.max() < 2e-5, err.max()


def test_few_values(W):
    mesh = PT.f32_mesh(I.perturb_radial(I.icosphere(17), 0.1, 3, 4))  # 5,780 triangles
    T = mesh.n_prims
    scene, om = W.Scene(mesh, W.F32), oracle.OracleMesh(mesh)
    rng = np.random.default_rng(3)
    pts = PT.f32(I.ball_points(70, 1.5, 7))
    ids = [(k,) for k in np.linspace(0, T - 1, 40).astype(int)] + [rng.integers(0, T, 3) for _ in range(20)]
    for k in ids:
        g = np.zeros(T)
        g[list(k)] = PT.f32(rng.standard_normal(len(k)) + 3.0)
        check(W, scene, om, g, pts, np.arange(len(pts)))
    scene.close()


@pytest.mark.parametrize("P", [32767, 33000, 255999, 256001, 640001])
@pytest.mark.parametrize("size", [1, 9])  # 20, 1,620 triangles
def test_splits_with_zeros(W, size, P):
    mesh = PT.f32_mesh(I.perturb_radial(I.icosphere(size), 0.1, 3, 4))
    scene, om = W.Scene(mesh, W.F32), oracle.OracleMesh(mesh)
    rng = np.random.default_rng(size)
    g = PT.f32(rng.standard_normal(mesh.n_prims))
    cen = mesh.verts[mesh.prims].mean(1)
    g[cen[:, 2] < 0.5] = 0
    pts = I.ball_points(P, 1.5, 7)
    pts[::2] = (cen[rng.integers(0, mesh.n_prims, P)] * (1 + 0.02 * rng.standard_normal((P, 1))))[::2]
    pts[1::11] *= 30
    keep = np.unique(np.concatenate([np.arange(40), np.arange(P - 600, P)]))
    check(W, scene, om, g, PT.f32(pts), keep)
    scene.close()
