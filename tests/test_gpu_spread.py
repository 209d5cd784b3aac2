"""Solves of few paths, whose points take up to a whole workgroup of lanes: mean
and variance against the traced paths of the same points, for every number of
lanes per point that the launch rule reaches (one wavefront, several
wavefronts of one workgroup, one path per lane and less) and every form."""
import dataclasses

import numpy as np
import pytest

from paper_2305_04403_amd import inputs as I
from tests import parity as PT
from tests.test_gpu_parity import dev, wbc

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def W():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2305_04403_amd import wob
    wob.lib()
    return wob


def problem(form, f32):
    mesh = I.perturb_radial(I.icosphere(6), 0.1, 3, 4)
    if f32:
        mesh = PT.f32_mesh(mesh)
    if form == "double":
        return mesh, dict(domain=1, formulation=1, program=3, params=(2.0, 0.5, 0.0)), 0.0, 0.8
    kind = I.assign_kinds(mesh.n_prims, (I.NEUMANN,) if form == "direct" else (I.NEUMANN, I.ROBIN), 3)
    mesh = dataclasses.replace(mesh, kind=kind, alpha=np.where(kind == I.ROBIN, 0.5, 0.0))
    bc = dict(domain=-1, formulation=2 if form == "direct" else 3, program=3, params=(0.2, -0.1, 0.05))
    if form == "ris":
        bc.update(sampling=1, candidates=8)
    return mesh, bc, 1.2, 2.0


# points x paths: 1 x 1500 (a workgroup's 1,024 or 512 lanes), 3 x 700, 9 x 200 (256 lanes),
# 70 x 65 (128), 2,100 x 63 (64 lanes, one path each, the last group short), 900 x 2, 5 x 1
@pytest.mark.parametrize("P,N", [(1, 1500), (3, 700), (9, 200), (70, 65), (2100, 63), (900, 2), (5, 1)])
@pytest.mark.parametrize("form", ["double", "direct", "single", "ris"])
@pytest.mark.parametrize("precision", ["f32", "f64"])
def test_few_paths_equal_their_traces(W, form, P, N, precision):
    f32 = precision == "f32"
    mesh, bc, r0, r1 = problem(form, f32)
    dt = torch.float32 if f32 else torch.float64
    scene = W.Scene(mesh, W.F32 if f32 else W.F64)
    tp = dev(I.ball_points(P, r1, 5, r_min=r0), dt)
    b = wbc(W, bc)
    val, _, _ = W.trace(scene, tp, b, N, 3, 4, want_vertices=False)
    mean, var = W.solve(scene, tp, b, N, 3, 4, want_var=N > 1)
    torch.cuda.synchronize()
    v = val.cpu().double().numpy()
    assert np.isfinite(v).all()
    # binary64 statistics, rounded once to the output's type; the sums' own
    # rounding (N binary64 units of the largest path) beside it
    u = 2.0 ** -24 if f32 else 0.0
    top = np.abs(v).max(axis=1)
    m = v.mean(axis=1)
    assert np.all(np.abs(mean.cpu().double().numpy() - m) <= u * np.abs(m) * 1.01 + N * 2.0 ** -52 * top)
    if N > 1:
        s = v.var(axis=1, ddof=1)
        assert np.all(np.abs(var.cpu().double().numpy() - s) <= u * s * 1.01 + 4 * N * 2.0 ** -52 * top ** 2)
    scene.close()


@pytest.mark.parametrize("tune", [(64, 8), (128, 4), (256, 2), (512, 1)])
def test_few_paths_in_a_batch_equal_their_solves(W, tune):
    """Points of more lanes than a workgroup of the batch has, walked in parts."""
    probs, ref = [], []
    for form in ("double", "direct", "single", "ris"):
        mesh, bc, r0, r1 = problem(form, True)
        scene = W.Scene(mesh, W.F32)
        for P, N in ((1, 1500), (3, 700), (70, 65), (900, 2), (2100, 63)):
            tp = dev(I.ball_points(P, r1, 5, r_min=r0), torch.float32)
            probs.append(dict(scene=scene, points=tp, bc=wbc(W, bc), samples=N, walk_len=3, seed=4))
            ref.append(W.solve(scene, tp, wbc(W, bc), N, 3, 4))
    b = W.Batch(probs, tune=tune)
    for rep in range(2):
        outs = b.launch()
        torch.cuda.synchronize()
        for i, ((m, v), (mr, vr)) in enumerate(zip(outs, ref)):
            assert torch.equal(m, mr) and torch.equal(v, vr), (tune, rep, i)
    b.close()
