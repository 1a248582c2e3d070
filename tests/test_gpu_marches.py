"""GPU: the lengths of the kernels' marches that small blocks never take.  Faces along y and z march over up to three
faces where their wavefronts fill the chip several times; the interpolation of the stored geometry marches over eight
and sixteen planes on larger blocks.  Thin blocks with many columns reach all of them, with clipped last marches.  The
rules are mirrored here, so that a change of them shows."""
import numpy as np
import pytest

from paper_2406_11669_amd import workloads as W
from tests import test_gpu_geometry as G
from tests.parity import assert_fields_close

pytestmark = pytest.mark.gpu
SLOTS = 256 * 4 * 3


@pytest.fixture(scope="module")
def ax():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2406_11669_amd import asterx
    asterx.lib()
    return asterx


def _face_rows(n, d, recon, ct):
    lo = 3 if ct == "uct" else 1
    cols = -(-(n[0] + 2 * lo - 1) * (n[2 if d == 1 else 1] + 2 * lo - 1) // 64)
    best, least = 1, None
    for r in range(1, (2 if recon == "minmod" else 3) + 1):
        cost = -(-cols * ((n[d] + r) // r) // SLOTS) * (2 * r + 1)
        if least is None or cost <= least:
            best, least = r, cost
    return best


@pytest.mark.parametrize("recon,ct,n,rows", [("ppm", "fct", (300, 291, 4), 3), ("wenoz", "fct", (300, 291, 4), 3),
                                             ("mp5", "uct", (300, 291, 4), 3), ("minmod", "fct", (350, 340, 4), 2),
                                             ("mp5", "fct", (300, 4, 291), 3)])
def test_step_with_long_face_marches(ax, orc, recon, ct, n, rows):
    """One Heun step within 1e-10 of the oracle (the bound of the other parity tests of whole steps), the last marches
    along y and z clipped."""
    import torch
    w = W.curved_block(seed=81, n=n, recon=recon, ng=4 if ct == "uct" else 3, nsteps=1, rk=2)
    w.params["ct"] = ct
    print("case long marches", recon, ct, n, flush=True)
    for d in (1, 2):
        assert _face_rows(n, d, recon, ct) == rows and (n[d] + 1) % rows != 0
    L = w.layout
    blk = ax.Block(w)
    blk.run(1)
    torch.cuda.synchronize()
    cons = orc.prim2con(L, w.params, w.metric, w.A, w.prim)
    orc.fill_ghosts(L, cons, w.bc_cell)
    state, prim = w.state(cons), w.prim.copy()
    orc.run(L, w.params, w.metric, w.curv, state, prim, w.dt, 1, w.rk, w.bc_cell, w.bc_A, A_shift=w.A_shift,
            lib_=orc.lib_omp()[0])
    assert_fields_close(blk.state.cpu().numpy(), state, 1e-10, L.owned, G.STATE_NAMES)
    assert_fields_close(blk.prim.cpu().numpy(), prim, 1e-10, L.owned, G.PRIM_NAMES)


@pytest.mark.parametrize("ct,n,planes", [("fct", (130, 120, 20), 8), ("uct", (130, 120, 20), 8),
                                         ("fct", (200, 180, 41), 16)])
def test_geometry_with_long_marches(ax, ct, n, planes):
    """The stored geometry against the Lagrange interpolation at sizes whose marches take 8 and 16 planes, the last one
    clipped (bound and comparison of the sizes with marches of four)."""
    lo = 3 if ct == "uct" else 1
    e = [m + 2 * lo - 1 + (1 if lo < 2 else 0) for m in n]
    waves = (e[0] * e[1] + 63) // 64 * e[2]
    assert (16 if waves >= 16384 else 8 if waves >= 2048 else 4) == planes and e[2] % planes != 0 and e[2] > planes
    G.test_geometry_against_lagrange(ax, n, ct)
