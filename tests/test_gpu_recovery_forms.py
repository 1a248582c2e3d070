"""GPU: the recovery kernels that a block's stages choose between, each at what only it can get wrong: the learned
guess inside the recovery with sources (asterx_c2p_src, whose network shares LDS with the interpolation passes) and
with stored geometry, in steps against the oracle; the counters of the recovery with stored geometry (linear tiles,
ragged last workgroups) where no, few or all cells fail."""
import numpy as np
import pytest

from paper_2406_11669_amd import workloads as W
from tests.parity import assert_fields_close

pytestmark = [pytest.mark.gpu, pytest.mark.filterwarnings("ignore::RuntimeWarning")]


@pytest.fixture(scope="module")
def ax():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2406_11669_amd import asterx
    asterx.lib()
    return asterx


@pytest.fixture(scope="module")
def network(ax):
    """A network trained on a few batches: better than none, and its misses exercise the plain start behind it."""
    from paper_2406_11669_amd import learned
    feat, tgt = learned.training_set(200_000, seed=21)
    st = learned.standardization(feat, tgt)
    params, _ = learned.train(feat, tgt, st, epochs=4, batch=8192, seed=3)
    return params, st


@pytest.mark.parametrize("stored", [False, True])
@pytest.mark.parametrize("cold_planes", [0, 3])
def test_learned_block_steps(ax, network, orc, cold_planes, stored):
    """Two RK4 steps with the learned guess in every recovery within 1e-10 of the oracle's (the bound of the other
    parity tests of whole steps), the previous primitives of some z planes zeroed before the first stage (those
    wavefronts evaluate the network, the oracle starts cold).  Without stored geometry the stages take asterx_c2p_src."""
    import torch
    params, st = network
    w = W.curved_block(seed=31, n=(35, 13, 11), recon="ppm", nsteps=2)
    L = w.layout
    print("case learned block", cold_planes, stored, flush=True)
    blk = ax.Block(w, stored_geometry=stored)
    assert (blk.geo is not None) == stored
    blk.mlp = ax.make_mlp(params, st)
    prim0 = w.prim.copy()
    for k in range(cold_planes):
        prim0[:, L.ng + 1 + 3 * k] = 0.0
        blk.prim[:, L.ng + 1 + 3 * k] = 0.0
    blk.run(2)
    torch.cuda.synchronize()
    cons = orc.prim2con(L, w.params, w.metric, w.A, w.prim)
    orc.fill_ghosts(L, cons, w.bc_cell)
    state = w.state(cons)
    orc.run(L, w.params, w.metric, w.curv, state, prim0, w.dt, 2, w.rk, w.bc_cell, w.bc_A)
    names = ["D", "Sx", "Sy", "Sz", "tau", "Ax", "Ay", "Az", "Psi"]
    assert_fields_close(blk.state.cpu().numpy(), state, 1e-10, L.owned, names)
    assert_fields_close(blk.prim.cpu().numpy(), prim0, 1e-10, L.owned, ["rho", "p", "vx", "vy", "vz"])


@pytest.mark.parametrize("learned", [False, True])
@pytest.mark.parametrize("shape,share", [((1, 1, 1), 1.0), ((17, 5, 3), 0.3), ((33, 9, 5), 1.0), ((32, 8, 8), 0.0),
                                         ((40, 13, 6), 0.02)])
def test_stored_geometry_counters_equal_the_flags(ax, network, orc, shape, share, learned):
    """asterx_c2p_geo's counters equal the flags' own counts and accumulate over calls; the flags are the oracle's
    (with a network, but for its own bit: a guess that did not converge)."""
    import torch
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
    z = lambda nf: torch.zeros((nf,) + L.shape3, dtype=torch.float64, device="cuda")
    stats = torch.zeros(6, dtype=torch.int64, device="cuda")
    flags = torch.zeros(L.shape3, dtype=torch.uint8, device="cuda")
    geo, src = z(ax.GEO_FIELDS), z(4)
    mlp = ax.make_mlp(*network) if learned else None
    expect = np.zeros(5, dtype=np.int64)
    print("case geometry counters", shape, share, learned, flush=True)
    ax.geometry(L, P, dev(w.metric), dev(w.curv), geo)
    for rep in range(2):
        p0 = w.prim * (1.0 + 0.01 * rep)
        c, p = dev(cons), dev(p0)
        ax.c2p_geo(L, P, geo, dev(w.A), c, p, src, flags, stats, mlp=mlp)
        torch.cuda.synchronize()
        fl = L.owned(flags.cpu().numpy())
        fl_ref, _ = orc.c2p(L, P, w.metric, w.A, cons.copy(), p0.copy())
        assert np.array_equal(fl & ~np.uint8(32), L.owned(fl_ref))
        expect += np.array([np.count_nonzero(fl & b) for b in (1, 2, 4, 8, 16)])
        st = stats.cpu().numpy()
        assert np.array_equal(st[:5], expect), (st, expect)
