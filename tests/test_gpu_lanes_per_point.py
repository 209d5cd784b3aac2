"""Walks by lines at sizes around the rule for their lanes per point: the time follows
the points, whichever side of the rule they lie on, and the statistics are those of
the traced paths."""
import time

import numpy as np
import pytest

from paper_2305_04403_amd import inputs as I
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
    for _ in range(6):
        torch.cuda.synchronize()
        t = time.perf_counter()
        for _ in range(3):
            call()
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t)
    return best


def problem(W, form, precision="f64"):
    mesh = I.perturb_radial(I.icosphere(24), 0.1, 3, 4)
    mesh = I.Mesh(3, mesh.verts, mesh.prims, np.full(mesh.n_prims, I.NEUMANN, np.uint8))
    if precision == "f32":
        mesh = mesh.as_float32_geometry()
    return W.Scene(mesh, W.F64 if precision == "f64" else W.F32), W.BC(-1, 2 if form == "direct" else 3, W.PROG_INVDIST, (0.2, -0.1, 0.05))


@pytest.mark.parametrize("form", ["direct", "single"])
def test_time_follows_the_points(W, form):
    scene, bc = problem(W, form)
    pts = dev(I.ball_points(120_000, 2.0, 5, r_min=1.2), torch.float64)
    t = {n: seconds(lambda: W.solve(scene, pts[:n], bc, 64, 4, 1)) for n in (30_000, 120_000)}
    # a quarter of the points: no more than 0.32 of the time
    assert t[30_000] < 0.32 * t[120_000], t
    scene.close()


@pytest.mark.parametrize("form", ["direct", "single"])
def test_time_follows_the_points_f32(W, form):
    scene, bc = problem(W, form, "f32")
    pts = dev(I.ball_points(120_000, 2.0, 5, r_min=1.2), torch.float32)
    t = {n: seconds(lambda: W.solve(scene, pts[:n], bc, 64, 4, 1)) for n in (30_000, 120_000)}
    # a quarter of the points: no more than 0.36 of the time (the last wavefronts'
    # end weighs more than in FP64)
    assert t[30_000] < 0.36 * t[120_000], t
    scene.close()


# 8 wavefronts per CU of 32 lanes a point: 4,096 points on a 256-CU device
@pytest.mark.parametrize("P", [4095, 4097, 8193])
@pytest.mark.parametrize("form", ["direct", "single"])
def test_statistics(W, form, P):
    scene, bc = problem(W, form)
    tp = dev(I.ball_points(P, 2.0, 5, r_min=1.2), torch.float64)
    val, _, _ = W.trace(scene, tp, bc, 64, 3, 4, want_vertices=False)
    mean, var = W.solve(scene, tp, bc, 64, 3, 4)
    torch.cuda.synchronize()
    v = val.cpu().numpy()
    top = np.abs(v).max(axis=1)
    assert np.all(np.abs(mean.cpu().numpy() - v.mean(axis=1)) <= 64 * 2.0 ** -52 * top)
    assert np.all(np.abs(var.cpu().numpy() - v.var(axis=1, ddof=1)) <= 4 * 64 * 2.0 ** -52 * top ** 2)
    scene.close()
