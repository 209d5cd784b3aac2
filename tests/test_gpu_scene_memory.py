"""Device memory of a scene: beside the table of RIS candidates (64 bytes a
primitive in FP32, 128 in FP64) it is no more than records, normals of four values,
a 4-byte guide entry per bucket and the tree's records came to; and the area-uniform
picks of RIS on meshes whose areas crowd many primitives into one bucket or leave
buckets empty."""
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


LIMITS = {  # primitives: bytes in FP32, in FP64, without the table
    3: {500: (63404, 111228), 5120: (666276, 1169660), 32000: (4096996, 7259740), 62720: (8123364, 14542428)},
    2: {500: (44012, 78892), 5120: (488780, 911980), 32000: (2818124, 5055724), 62720: (6176076, 12180076)},
}


@pytest.mark.parametrize("precision", ["f32", "f64"])
@pytest.mark.parametrize("dim", [3, 2])
def test_scene_bytes(W, dim, precision):
    for size in (5, 16, 40, 56):
        mesh = I.perturb_radial(I.icosphere(size), 0.1, 3, 4) if dim == 3 else I.circle_polygon(20 * size * size)
        scene = W.Scene(mesh.as_float32_geometry(), W.F32 if precision == "f32" else W.F64)
        limit = LIMITS[dim][mesh.n_prims][precision == "f64"]
        table = mesh.n_prims * (64 if precision == "f32" else 128)
        assert scene.info()["device_bytes"] <= limit + table, mesh.n_prims
        scene.close()


def crowded(dim):
    """A mesh of which a few large primitives hold nearly the whole area: their buckets
    hold nothing else, and one bucket holds hundreds of small ones."""
    if dim == 3:
        mesh = I.icosphere(8)
        r = np.linalg.norm(mesh.verts, axis=1)
        v = mesh.verts / r[:, None]
        v = np.where((v[:, 2] > -0.9)[:, None], v * np.array([0.04, 0.04, 0.04]) + np.array([0, 0, -0.8]), v)
        return I.Mesh(3, v, mesh.prims, np.full(mesh.n_prims, I.NEUMANN, np.uint8))
    t = np.concatenate([np.linspace(0, 0.05, 400), np.linspace(0.05, 2 * np.pi, 9)[1:-1]])
    v = np.stack([np.cos(t), np.sin(t)], 1)
    p = np.stack([np.arange(len(t)), np.roll(np.arange(len(t)), -1)], 1).astype(np.int32)
    return I.Mesh(2, v, p, np.full(len(p), I.NEUMANN, np.uint8))


@pytest.mark.parametrize("precision", ["f32", "f64"])
@pytest.mark.parametrize("dim", [3, 2])
def test_picks_on_crowded_areas(W, dim, precision):
    mesh = crowded(dim)
    if precision == "f32":
        mesh = mesh.as_float32_geometry()
    dt = torch.float32 if precision == "f32" else torch.float64
    scene = W.Scene(mesh, W.F32 if precision == "f32" else W.F64)
    n, seed = 20000, 3
    pts = I.ball_points(40, 3.0, 5, r_min=2.0)[:, :dim]
    pts = pts / np.linalg.norm(pts, axis=1, keepdims=True) * 2.5
    if precision == "f32":
        pts = PT.f32(pts)
    bc = W.BC(-1, W.SINGLE_LAYER, W.PROG_CONST, (1.0,), sampling=W.SAMPLE_RIS, candidates=32)
    val, vprim, _ = W.trace(scene, dev(pts, dt), bc, n // 40, 1, seed)
    torch.cuda.synchronize()
    ob = oracle.make_bc(-1, 3, oracle.PROG_CONST, (1.0,), sampling=1, candidates=32)
    orc = oracle.trace(oracle.OracleMesh(mesh), pts, None, ob, 1, seed, np.repeat(np.arange(40), n // 40),
                       np.tile(np.arange(n // 40), 40), want_pos=False)
    same = vprim.cpu().numpy().reshape(-1) == orc["vtx_prim"].reshape(-1)
    # a reservoir decision on the rounding of the kernel may fall either way; picks of
    # another primitive of the bucket would be wrong throughout
    assert same.mean() > 0.999, same.mean()
    assert len(np.unique(orc["vtx_prim"])) > 50
    scene.close()
