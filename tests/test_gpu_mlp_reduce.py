"""The sum of the training step's wave partials (one per 16 rows, up to 1,024) by sixteenths:
fewer partials than waves, as many, one more, and the most, against the oracle at the bounds of
the gradient test of other sizes (loss 1e-4, gradients 2e-3: bfloat16 operands, float32 sums)."""
import numpy as np
import pytest

from oracle import budget as B
from test_gpu_budget import DEV, flat, np_, oracle_inputs, random_inputs, random_net, srw, torch, unflat  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [225, 256, 257, 16384 + 16])
def test_gradient_sums_match_oracle(srw, n):  # noqa: F811
    p = random_net(5)
    X, mu, sd, t = random_inputs(n, 6)
    P = torch.as_tensor(flat(p).astype(np.float32), device=DEV)
    musd = torch.as_tensor(np.concatenate([mu, sd]), device=DEV)
    grad = torch.full((4801,), float("nan"), dtype=torch.float32, device=DEV)
    loss = torch.empty(1, dtype=torch.float32, device=DEV)
    srw.mlp_train_step(P, musd, torch.as_tensor(X, device=DEV), torch.as_tensor(t, device=DEV),
                       grad=grad, loss=loss)
    torch.cuda.synchronize()
    ref_loss, ref_g = B.loss_and_grads(p, oracle_inputs(X, mu, sd), t.astype(np.float64),
                                       round_bf16=True)
    assert abs(float(np_(loss)[0]) - ref_loss) <= 1e-4 * ref_loss
    g = unflat(np_(grad))
    for k in ref_g:
        assert np.linalg.norm(g[k] - ref_g[k]) <= 2e-3 * np.linalg.norm(ref_g[k]) + 1e-12, k
