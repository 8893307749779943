"""The degree model's loss and gradient kernels at the edges of their work groups, against the FP64 oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle import mlp  # noqa: E402


# 8 samples a round, at most 208 work groups: one round less one sample, one and two
# rounds, every group one round, and a second round for one group
@pytest.mark.parametrize("n", [1, 7, 8, 9, 16, 1663, 1664, 1665, 5000])
def test_loss_gradient_at_the_work_groups_edges(n):
    from paper_2012_06925_amd import api
    rng = np.random.default_rng(80 + n)
    model = rng.normal(0, 0.3, api.mlp_model_size()).astype(np.float32)
    model[mlp.N_PARAMS + 4:mlp.N_PARAMS + 8] = rng.uniform(0.5, 2, 4)
    f = rng.normal(0, 1.5, (n, 4)).astype(np.float32)
    t = rng.normal(-6, 2, (n, 11)).astype(np.float32)
    t[rng.random(t.shape) < 0.05] = np.nan
    t[0, 0] = -6.0
    dev = lambda a: torch.from_numpy(a).cuda()                               # noqa: E731
    loss, g = api.mlp_loss_grad(dev(model), dev(f), dev(t))
    g = g.cpu().numpy()
    m64 = model.astype(np.float64)
    ref = mlp.grad(m64, f.astype(np.float64), t.astype(np.float64))
    assert loss == pytest.approx(mlp.loss(m64, f.astype(np.float64), t.astype(np.float64)), rel=1e-5)
    assert np.linalg.norm(g - ref) <= 1e-4 * np.linalg.norm(ref)
    again = api.mlp_loss_grad(dev(model), dev(f), dev(t))
    assert again[0] == loss and np.array_equal(again[1].cpu().numpy(), g)


def test_no_valid_target_gives_zero():
    from paper_2012_06925_amd import api
    rng = np.random.default_rng(90)
    model = torch.from_numpy(rng.normal(0, 0.3, api.mlp_model_size()).astype(np.float32)).cuda()
    f = torch.from_numpy(rng.normal(0, 1, (33, 4)).astype(np.float32)).cuda()
    loss, g = api.mlp_loss_grad(model, f, torch.full((33, 11), float("nan"), device="cuda"))
    assert loss == 0.0 and not np.any(g.cpu().numpy())


def test_samples_past_the_end_do_not_meet_the_model():
    # a feature far from 0 on a fine scale: (0 - mean) * scale is infinite, and the
    # rows that fill up the last group of 8 must not bring it into the gradient
    from paper_2012_06925_amd import api
    rng = np.random.default_rng(91)
    n = 13
    model = rng.normal(0, 0.3, api.mlp_model_size()).astype(np.float32)
    model[mlp.N_PARAMS + 4:mlp.N_PARAMS + 8] = 1.0
    model[mlp.N_PARAMS], model[mlp.N_PARAMS + 4] = 1e25, 1e20
    f = rng.normal(0, 1.5, (n, 4)).astype(np.float32)
    f[:, 0] = np.float32(1e25)
    t = rng.normal(-6, 2, (n, 11)).astype(np.float32)
    loss, g = api.mlp_loss_grad(*(torch.from_numpy(a).cuda() for a in (model, f, t)))
    m64 = model.astype(np.float64)
    ref = mlp.grad(m64, f.astype(np.float64), t.astype(np.float64))
    assert loss == pytest.approx(mlp.loss(m64, f.astype(np.float64), t.astype(np.float64)), rel=1e-5)
    assert np.linalg.norm(g.cpu().numpy() - ref) <= 1e-4 * np.linalg.norm(ref)
