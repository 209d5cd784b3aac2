"""Scenes on both sides of the record layouts (48-byte triangle records, or
64-byte ones that hold the normal), a double-layer solve on a scene large enough
for the reduced number of wavefronts, and lines that cross more leaves at once
than the wavefront's leaf queue holds; per path against the FP64 oracle."""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2305_04403_amd import inputs as I
from tests import parity as PT
from tests.test_gpu_parity import dev, obc, run_trace_parity, wbc

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def W():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2305_04403_amd import wob
    wob.lib()
    return wob


@pytest.mark.parametrize("freq,stride", [(44, 48), (45, 64)])  # 38,720 and 40,500 triangles
@pytest.mark.parametrize("form", ["dirichlet", "mixed", "neumann"])
def test_triangle_record_layouts(W, freq, stride, form):
    mesh = PT.f32_mesh(I.perturb_radial(I.icosphere(freq), 0.1, 3, 4))
    if form == "dirichlet":
        pts = PT.f32(I.ball_points(6, 0.8, 1))
        bc = dict(domain=1, formulation=1, program=3, params=(2.0, 0.5, 0.0))
    else:
        kinds = (I.NEUMANN, I.ROBIN) if form == "mixed" else (I.NEUMANN,)
        kind = I.assign_kinds(mesh.n_prims, kinds, 3)
        mesh = dataclasses.replace(mesh, kind=kind, alpha=np.where(kind == I.ROBIN, 1.0, 0.0))
        pts = PT.f32(I.ball_points(6, 2.0, 2, r_min=1.2))
        bc = dict(domain=-1, formulation=3 if form == "mixed" else 2, program=3, params=(0.2, -0.1, 0.05))
    scene = W.Scene(mesh, W.F32)
    assert scene.info()["prim_bytes"] == stride
    scene.close()
    run_trace_parity(W, mesh, pts, None, bc, 8, 3, 5, "f32")


def test_double_layer_on_a_large_scene(W):
    # 100,820 triangles: fewer wavefronts per CU for the double layer's solves
    mesh = PT.f32_mesh(I.perturb_radial(I.icosphere(71), 0.1, 3, 4))
    pts = PT.f32(I.ball_points(130, 0.8, 1))
    bc = wbc(W, dict(domain=1, formulation=1, program=3, params=(2.0, 0.5, 0.0)))
    scene = W.Scene(mesh, W.F32)
    tp = dev(pts, torch.float32)
    val, _, _ = W.trace(scene, tp, bc, 100, 4, 9, want_vertices=False)
    mean, var = W.solve(scene, tp, bc, 100, 4, 9)
    torch.cuda.synchronize()
    v = val.cpu().double().numpy()
    # one binary32 rounding of each statistic
    np.testing.assert_allclose(mean.cpu().numpy(), v.mean(axis=1), rtol=2.0 ** -23, atol=2.0 ** -24 * np.abs(v).max())
    np.testing.assert_allclose(var.cpu().numpy(), v.var(axis=1, ddof=1), rtol=2.0 ** -23)
    scene.close()


@pytest.mark.parametrize("precision", ["f32", "f64"])
def test_lines_that_cross_more_leaves_than_the_queue_holds(W, precision):
    # 240 stacked plates: a steep line crosses most of them, so that the lanes
    # of a wavefront together hold more leaves than the queue's 256 entries
    n = 240
    z = np.linspace(-1.0, 1.0, n)
    verts = np.concatenate([np.stack([[-9.0, -9.0, h], [15.0, -3.0, h], [-3.0, 15.0, h]]) for h in z])
    mesh = I.Mesh(3, verts, np.arange(3 * n, dtype=np.int32).reshape(n, 3))
    if precision == "f32":
        mesh = PT.f32_mesh(mesh)
    pts = I.ball_points(4, 0.8, 7)
    if precision == "f32":
        pts = PT.f32(pts)
    bc = dict(domain=1, formulation=1, program=1, params=(0.3, -0.2, 0.5, 1.0))
    res = run_trace_parity(W, mesh, pts, None, bc, 64, 3, 11, precision)
    assert res.n_checked > 0.9 * res.n
