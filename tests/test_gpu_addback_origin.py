"""Add-back at points that coincide with no triangle's sample but with what fills
up its last tile: the origin, points nearer to it than the square root of the
least binary32 number, and points as far off as that sum can hold; triangle
counts that are no multiple of a wavefront's lanes, points on both sides of the
split's rule (32,768 on a 256-CU device)."""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2305_04403_amd import inputs as I
from tests import parity as PT
from tests.test_gpu_parity import dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SPECIAL = np.array([[0, 0, 0], [-0.0, 0, 0], [1e-20, 0, 0], [0, -3e-22, 1e-25], [1e-30, 1e-30, -1e-30],
                    [1e18, 1e18, 1e18], [-1e18, 0, 0]])


@pytest.fixture(scope="module")
def W():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2305_04403_amd import wob
    wob.lib()
    return wob


@pytest.mark.parametrize("P", [7, 33025])
@pytest.mark.parametrize("size", [1, 5, 9])  # 20, 500, 1,620 triangles
def test_addback_at_the_origin(W, size, P):
    mesh = PT.f32_mesh(I.perturb_radial(I.icosphere(size), 0.1, 3, 4))
    g = PT.f32(np.random.default_rng(size).standard_normal(mesh.n_prims))
    pts = PT.f32(np.resize(SPECIAL, (P, 3)))
    scene = W.Scene(mesh, W.F32)
    got = W.cv_addback(scene, dev(g, torch.float32), dev(pts, torch.float32), seed=9).cpu().double().numpy()
    om = oracle.OracleMesh(mesh)
    ref = np.resize(oracle.cv_addback(om, g, pts[:7], seed=9, randomized=True), P)
    # (the closed form of a triangle cancels to nothing in binary64 at 1e18)
    scale = np.resize(oracle.cv_addback(om, np.abs(g), pts[:7], seed=9, randomized=True), P)
    assert np.isfinite(got).all()
    # the bar of the whole-mesh comparison (a few binary32 units per term and sum)
    err = np.abs(got - ref) / scale
    assert err.max() < 2e-5, err.max()
    scene.close()


def test_corrected_solve_at_the_origin(W):
    """Exterior problem around three tori whose common centre lies in the domain."""
    mesh = I.torus_union(grid_n=16)[0]
    mesh = PT.f32_mesh(dataclasses.replace(mesh, kind=np.full(mesh.n_prims, I.NEUMANN, np.uint8)))
    assert mesh.n_prims % 32 != 0
    rng = np.random.default_rng(2)
    g = PT.f32(rng.standard_normal(mesh.n_prims))
    pts = PT.f32(np.array([[0, 0, 0], [0, 0, 1.9], [1e-22, 0, 0]]))
    scene = W.Scene(mesh, W.F32)
    bc = W.BC(-1, W.SINGLE_LAYER, W.PROG_INVDIST, (1.0, 0.1, 0.0))
    tp, tg = dev(pts, torch.float32), dev(g, torch.float32)
    mean, var = W.solve_cv(scene, tp, bc, 64, 3, tg, seed=5)
    val = W.trace_cv(scene, tp, bc, 64, 3, tg, seed=5)
    torch.cuda.synchronize()
    paths = val.cpu().double().numpy().reshape(3, 64).mean(axis=1)
    om = oracle.OracleMesh(mesh)
    add = oracle.cv_addback(om, g, pts, seed=5, randomized=True)
    scale = oracle.cv_addback(om, np.abs(g), pts)
    # the paths' mean and the sum's value each rounded to binary32, the add-back's bar
    tol = 2.0 ** -23 * (np.abs(paths) + np.abs(add)) + 2e-5 * scale
    assert np.isfinite(var.cpu().numpy()).all()
    assert np.all(np.abs(mean.cpu().double().numpy() - (paths + add)) <= tol)
    scene.close()
