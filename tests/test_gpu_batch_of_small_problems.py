"""Many small problems in one batch: together they fill the chip, so the batch
takes little longer than one problem of the same points, and the values follow
the single solves."""
import dataclasses
import time

import numpy as np
import pytest

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
    for _ in range(5):
        torch.cuda.synchronize()
        t = time.perf_counter()
        call()
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t)
    return best


def scene_and_bc(W, form, precision):
    mesh = I.perturb_radial(I.icosphere(16), 0.1, 3, 4)
    mesh = I.Mesh(3, mesh.verts, mesh.prims, np.full(mesh.n_prims, I.NEUMANN, np.uint8))
    if precision == "f32":
        mesh = PT.f32_mesh(mesh)
    return (W.Scene(mesh, W.F32 if precision == "f32" else W.F64),
            W.BC(-1, 2 if form == "direct" else 3, W.PROG_INVDIST, (0.2, -0.1, 0.05)))


@pytest.mark.parametrize("data", ["program", "vertex"])
@pytest.mark.parametrize("form", ["direct", "single"])
def test_time_of_many_small_problems(W, form, data):
    scene, bc = scene_and_bc(W, form, "f32")
    if data == "vertex":
        bc = dataclasses.replace(bc, vertex_data=torch.ones(scene.n_verts, device="cuda"))
    pts = dev(I.ball_points(64_000, 2.0, 5, r_min=1.2), torch.float32)
    one = W.Batch([dict(scene=scene, points=pts, bc=bc, samples=256, walk_len=4, seed=3)])
    many = W.Batch([dict(scene=scene, points=pts[1000 * k:1000 * (k + 1)].contiguous(), bc=bc, samples=256, walk_len=4,
                         seed=3) for k in range(64)])
    t1, t64 = seconds(one.launch), seconds(many.launch)
    assert t64 < 1.4 * t1, (t1, t64)
    one.close()
    many.close()
    scene.close()


@pytest.mark.parametrize("precision", ["f32", "f64"])
@pytest.mark.parametrize("problems,P,N", [(64, 1000, 64), (100, 200, 300), (3, 4000, 256)])
@pytest.mark.parametrize("form", ["direct", "single"])
def test_values_follow_the_single_solves(W, form, problems, P, N, precision):
    scene, bc = scene_and_bc(W, form, precision)
    dt = torch.float32 if precision == "f32" else torch.float64
    probs = [dict(scene=scene, points=dev(I.ball_points(P, 2.0, k, r_min=1.2), dt), bc=bc, samples=N, walk_len=3, seed=k)
             for k in range(problems)]
    b = W.Batch(probs)
    outs = b.launch()
    torch.cuda.synchronize()
    u = 2.0 ** -24 if precision == "f32" else 0.0
    for k in (0, problems // 2, problems - 1):
        p = probs[k]
        val, _, _ = W.trace(scene, p["points"], bc, N, 3, k, want_vertices=False)
        v = val.cpu().double().numpy()
        top, m, s = np.abs(v).max(axis=1), v.mean(axis=1), v.var(axis=1, ddof=1)
        mean, var = (o.cpu().double().numpy() for o in outs[k])
        # binary64 statistics in any order, rounded once to the output's type
        assert np.all(np.abs(mean - m) <= u * np.abs(m) * 1.01 + N * 2.0 ** -52 * top)
        assert np.all(np.abs(var - s) <= u * s * 1.01 + 4 * N * 2.0 ** -52 * top ** 2)
    b.close()
    scene.close()
