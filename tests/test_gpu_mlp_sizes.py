"""GPU: the network's gradient where the reduction over wavefronts can go wrong: one partial sum, fewer partial
sums than ranges, counts that do not divide into them, a single sample."""
import numpy as np
import pytest

pytestmark = [pytest.mark.gpu]


@pytest.mark.parametrize("n", [1, 64, 65, 64 * 15 + 1, 64 * 16, 64 * 17 + 3, 64 * 37])
def test_gradient_reduction_sizes(n):
    """Against the reference network with the kernels' bfloat16 roundings, within 2e-2 of each layer's largest
    gradient component (a cotangent or activation rounded the other way, as in the tests of the network); a partial
    sum lost or taken twice is one part in their number (37 at most, 2.7e-2)."""
    import torch
    from oracle import mlp_ref as M
    from paper_2406_11669_amd import asterx as ax
    rng = np.random.default_rng(n)
    feat = rng.normal(size=(8, n)).astype(np.float32)
    tgt = rng.normal(size=(2, n)).astype(np.float32)
    params = (0.2 * rng.normal(size=ax.MLP_NPARAMS)).astype(np.float32)
    one = dict(in_shift=[0.0] * 8, in_scale=[1.0] * 8, out_shift=[0.0] * 2, out_scale=[1.0] * 2)
    dev = lambda a: torch.from_numpy(a).cuda()
    p = dev(params)
    grad = torch.full((ax.MLP_NPARAMS + 1,), float("nan"), device="cuda")
    ws = torch.full((ax.mlp_grad_workspace_size(n) // 4 + 1,), float("nan"), device="cuda")
    print("case mlp gradient reduction", n, flush=True)
    ax.mlp_grad(ax.make_mlp(p, one), dev(feat), dev(tgt), grad, ws)
    torch.cuda.synchronize()
    g = grad.cpu().numpy()
    loss, ref = M.loss_grad(params, feat, tgt, {k: np.asarray(v, np.float32) for k, v in one.items()})
    assert abs(g[-1] - loss) <= 1e-4 * loss
    for a, b in ((0, 512), (512, 576), (576, 4672), (4672, 4736), (4736, 4864), (4864, 4866)):
        e, s = np.abs(g[a:b] - ref[a:b]), np.max(np.abs(ref[a:b]))
        assert np.max(e) <= 2e-2 * s, (a, np.max(e) / s)
