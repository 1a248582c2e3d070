"""GPU: the recovery's counters (one push per workgroup) where tiles are ragged, workgroups hold no or few failing
cells, and every cell fails: equal to the flags' own counts, and accumulated over calls."""
import numpy as np
import pytest

from paper_2406_11669_amd import workloads as W

pytestmark = [pytest.mark.gpu, pytest.mark.filterwarnings("ignore::RuntimeWarning")]


@pytest.mark.parametrize("src", [False, True])
@pytest.mark.parametrize("shape,share", [((1, 1, 1), 1.0), ((17, 5, 3), 0.3), ((33, 9, 5), 1.0), ((32, 8, 8), 0.0),
                                         ((40, 13, 6), 0.02)])
def test_counters_equal_the_flags(orc, shape, share, src):
    import torch
    from paper_2406_11669_amd import asterx as ax
    w = W.curved_block(seed=21, n=shape, recon="ppm", rho_atm=1e-6)
    L, P = w.layout, w.params
    cons = orc.prim2con(L, P, w.metric, w.A, w.prim)
    rng = np.random.default_rng(21)
    bad = rng.uniform(size=L.shape3) < share
    kind = rng.integers(0, 3, size=L.shape3)
    cons[0][bad & (kind == 0)] = 1e-9        # below the floor
    cons[4][bad & (kind == 1)] = -5.0        # no physical state
    cons[1][bad & (kind == 2)] = np.nan
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    stats = torch.zeros(6, dtype=torch.int64, device="cuda")
    flags = torch.zeros(L.shape3, dtype=torch.uint8, device="cuda")
    expect = np.zeros(5, dtype=np.int64)
    iters = 0
    print("case counters", shape, share, src, flush=True)
    for rep in range(2):
        c, p = dev(cons), dev(w.prim * (1.0 + 0.01 * rep))
        if src:
            out = torch.zeros((ax.SRC_FIELDS,) + L.shape3, dtype=torch.float64, device="cuda")
            ax.c2p_src(L, P, dev(w.metric), dev(w.curv), dev(w.A), c, p, out, flags, stats)
        else:
            ax.c2p(L, P, dev(w.metric), dev(w.A), c, p, flags, stats)
        torch.cuda.synchronize()
        fl = L.owned(flags.cpu().numpy())
        fl_ref, st_ref = orc.c2p(L, P, w.metric, w.A, cons.copy(), w.prim * (1.0 + 0.01 * rep))
        assert np.array_equal(fl, L.owned(fl_ref))
        expect += np.array([np.count_nonzero(fl & b) for b in (1, 2, 4, 8, 16)])
        iters = max(iters, int(st_ref[5]))
        st = stats.cpu().numpy()
        assert np.array_equal(st[:5], expect), (st, expect)
        assert abs(int(st[5]) - iters) <= 1, (st[5], iters)
