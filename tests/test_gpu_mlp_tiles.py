"""Gradient of the network at the edges of its row tiles (64) and of the sum of
their partial gradients (16 tiles at a time), and the training step, whose sum
takes the Adam step with it, against the gradient followed by the step alone."""
import numpy as np
import pytest

import oracle
from tests.test_gpu_mlp import MLP_ACC, f32, rand_net

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def W():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2305_04403_amd import wob
    wob.lib()
    return wob


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 1024, 1025, 2111])
def test_gradient_and_step_over_tiles(W, n, dim):
    params, B = rand_net(12)
    params, B = f32(params), f32(B)[:, :dim]
    rng = np.random.default_rng(n)
    y = f32(rng.uniform(-1.5, 1.5, (n, dim)))
    t = f32(rng.standard_normal(n))
    ty = torch.as_tensor(y, dtype=torch.float32, device="cuda")
    tt = torch.as_tensor(t, dtype=torch.float32, device="cuda")
    one, two = W.MLP(dim, B, params, max_batch=n), W.MLP(dim, B, params, max_batch=n)
    loss, grad = one.backward(ty, tt)
    lo, go = oracle.mlp_loss_grad(params, B, y, t, bf16=True)
    # the outputs' own error bound through the squares, and the sum's rounding;
    # the gradient at the whole-network bar, ten times that where a single
    # activation that rounds to the other neighbour is not averaged away
    res = oracle.mlp_forward_bound(params, B, y, MLP_ACC)
    e, b = np.abs(res["out"] - t), res["bound"]
    assert abs(loss.item() - lo) <= np.mean(2 * e * b + b * b) + 1e-5 * lo
    bar = 1e-3 if n >= 1024 else 1e-2
    assert np.linalg.norm(grad.cpu().double().numpy() - go) <= bar * np.linalg.norm(go)
    for step in (1, 2):
        loss, grad = one.backward(ty, tt)
        one.adam_step(grad, step, 1e-3, 0.9, 0.999, 1e-8)
        loss2 = torch.empty(1, dtype=torch.float32, device="cuda")
        two.train_step(ty, tt, step, 1e-3, loss=loss2)
        torch.cuda.synchronize()
        assert torch.equal(loss, loss2)
        np.testing.assert_array_equal(one.params(), two.params())
    one.close()
    two.close()
