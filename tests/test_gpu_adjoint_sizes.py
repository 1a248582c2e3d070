"""The right-hand side's adjoint at sizes where the transposed reconstruction's launches have edges: rows around the
60 points an x wavefront completes, marches of eight points with remainders, columns around 64, the smallest
periodic block.  <ybar, J v> (oracle dual numbers) = <J^T ybar, v>, to 1e-10 of the sum of the terms' magnitudes:
rounding of a few hundred operations per term (1e-14), times the conditioning of the recovery (below 1e3)."""
import numpy as np
import pytest

from paper_2406_11669_amd import workloads as W

pytestmark = pytest.mark.gpu


def _at_kink(f):
    """Whether tau = |beta_0 - beta_2| of WENO-Z is zero to rounding in some cell (the seeded modes on periods of four
    cells): the kink of the absolute value, where kernel and oracle may take different slopes."""
    for ax in (1, 2, 3):
        m2, m1, c0, p1, p2 = (np.roll(f, -k, axis=ax) for k in (-2, -1, 0, 1, 2))
        b0 = 13 / 12 * (m2 - 2 * m1 + c0) ** 2 + 0.25 * (m2 - 4 * m1 + 3 * c0) ** 2
        b2 = 13 / 12 * (c0 - 2 * p1 + p2) ** 2 + 0.25 * (3 * c0 - 4 * p1 + p2) ** 2
        if np.any(np.abs(b0 - b2) <= 1e-12 * (b0 + b2)):
            return True
    return False


@pytest.mark.parametrize("recon", ["minmod", "ppm", "wenoz", "mp5"])
@pytest.mark.parametrize("n", [(4, 4, 4), (53, 5, 4), (54, 4, 10), (6, 11, 9), (7, 7, 18)])
def test_rhs_adjoint_sizes(orc, n, recon):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2406_11669_amd import asterx as ax
    print("case rhs_adjoint sizes", n, recon, flush=True)
    w = W.curved_block(seed=52, n=n, recon=recon, nsteps=1, vmax=0.3)
    L = w.layout
    if recon == "wenoz" and _at_kink(L.owned(w.prim)):
        pytest.skip("WENO-Z has no derivative at this state")
    rng = np.random.default_rng(sum(n))
    cons = orc.prim2con(L, w.params, w.metric, w.A, w.prim)
    orc.fill_ghosts(L, cons, w.bc_cell)
    psi = L.zeros(1)

    def rand(nf):
        t = L.zeros(nf)
        L.owned(t)[...] = rng.normal(size=L.owned(t).shape)
        return t

    dcons, dA, ybar = rand(5), rand(3), rand(9)
    L.periodic_wrap(dcons)
    L.periodic_wrap(dA)
    _, dL = orc.stage_jvp(L, w.params, w.metric, w.curv, cons, w.A, psi, w.prim, w.dt, dcons=dcons, dA=dA, dpsi=None,
                          dgamma=0.0)
    t = {k: torch.from_numpy(np.ascontiguousarray(a)).cuda() for k, a in
         dict(metric=w.metric, curv=w.curv, cons=cons, prim=w.prim, A=w.A, psi=psi, ybar=ybar, cb=L.zeros(5),
              ab=L.zeros(3), pb=L.zeros(1)).items()}
    gb = torch.zeros(1, dtype=torch.float64, device="cuda")
    ws = torch.empty(-(-ax.adjoint_workspace_size(L) // 8), dtype=torch.float64, device="cuda")
    ax.rhs_adjoint(L, w.params, t["metric"], t["curv"], t["cons"], t["prim"], t["A"], t["psi"], w.dt,
                   t["ybar"], t["cb"], t["ab"], t["pb"], gb, ws)
    torch.cuda.synchronize()
    cb, ab = t["cb"].cpu().numpy(), t["ab"].cpu().numpy()
    lhs = L.owned(ybar) * L.owned(dL)
    rhs = np.concatenate([(L.owned(cb) * L.owned(dcons)).ravel(), (L.owned(ab) * L.owned(dA)).ravel()])
    scale = np.abs(lhs).sum() + np.abs(rhs).sum()
    assert abs(lhs.sum() - rhs.sum()) <= 1e-10 * scale, (lhs.sum(), rhs.sum(), scale)
