"""Stored spacetime data (asterx_geometry and the stage entry points that read it): the data against the four-point
Lagrange interpolation in numpy, steps against the oracle at sizes around the launches' edges (63 faces per x
wavefront, 64 columns, marches of one to three faces, two rows per lane in the interpolation), and the older entry
points with sources (face metric from the recovery) against the ones without."""
import numpy as np
import pytest

from paper_2406_11669_amd import workloads as W
from tests.parity import assert_fields_close

pytestmark = pytest.mark.gpu

STATE_NAMES = ["D", "Sx", "Sy", "Sz", "tau", "Ax", "Ay", "Az", "Psi"]
PRIM_NAMES = ["rho", "p", "vx", "vy", "vz"]
V = np.array([-1.0, 9.0, 9.0, -1.0]) / 16.0
D = np.array([1.0, -27.0, 27.0, -1.0]) / 24.0


@pytest.fixture(scope="module")
def ax():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2406_11669_amd import asterx
    asterx.lib()
    return asterx


def _pass(f, axis, w):
    """Four-point stencil from vertices i-1..i+2 along the numpy axis (the ends wrap: not compared)."""
    return sum(c * np.roll(f, 1 - k, axis=axis) for k, c in enumerate(w))


@pytest.mark.parametrize("ct", ["fct", "uct"])
@pytest.mark.parametrize("n", [(1, 1, 1), (5, 3, 2), (61, 2, 3), (64, 5, 9), (65, 4, 17), (3, 33, 34)])
def test_geometry_against_lagrange(ax, n, ct):
    """Tolerance: the weights' magnitudes sum to 1.25 per value pass and 2.34 per derivative pass, so every rounding
    error is below 1.25^3 (2.34 / dx times 1.25^2) eps max|f|; 20 operations per pass, three passes: 60 of them."""
    import torch
    w = W.curved_block(seed=61, n=n, ng=4, nsteps=1)
    w.params["ct"] = ct
    L = w.layout
    print("case geometry", n, ct, flush=True)
    rng = np.random.default_rng(1)
    met, curv = rng.normal(size=(10,) + L.shape3), rng.normal(size=(6,) + L.shape3)
    geo = torch.full((ax.GEO_FIELDS,) + L.shape3, float("nan"), dtype=torch.float64, device="cuda")
    ax.geometry(L, w.params, torch.from_numpy(met).cuda(), torch.from_numpy(curv).cuda(), geo)
    geo = geo.cpu().numpy()
    ng, lo = L.ng, 3 if ct == "uct" else 1
    eps = np.finfo(np.float64).eps

    def box(d):  # faces along d (numpy slices over z, y, x), or the owned cells
        r = [slice(ng, ng + m) if d < 0 else (slice(ng, ng + m + 1) if a == d else slice(ng - lo, ng + m + lo - 1))
             for a, m in enumerate(n)]
        return (slice(None), r[2], r[1], r[0])

    def check(got, want, b, tol):
        assert np.all(np.isfinite(got[b])) and np.max(np.abs(got[b] - want[b])) <= tol, (n, ct)

    for d in range(3):
        want = met
        for a in range(3):
            if a != d:
                want = _pass(want, 3 - a, V)
        check(geo[10 * d:10 * d + 10], want, box(d), 60 * 1.25 ** 2 * eps * np.abs(met).max())
    for d in range(-1, 3):  # centre values, then their derivatives
        want = met
        for a in range(3):
            want = _pass(want, 3 - a, D if a == d else V)
        scale = 1.25 ** 3
        if d >= 0:
            want, scale = want / L.dx[d], 2.34 * 1.25 ** 2 / L.dx[d]
        check(geo[40 + 10 * d:50 + 10 * d], want, box(-1), 60 * scale * eps * np.abs(met).max())
    want = curv
    for a in range(3):
        want = _pass(want, 3 - a, V)
    check(geo[70:76], want, box(-1), 60 * 1.25 ** 3 * eps * np.abs(curv).max())


@pytest.mark.parametrize("recon,ct", [("minmod", "fct"), ("ppm", "fct"), ("wenoz", "fct"), ("mp5", "fct"),
                                      ("ppm", "uct"), ("mp5", "uct")])
@pytest.mark.parametrize("n", [(61, 4, 3), (62, 3, 6), (5, 63, 4), (6, 13, 65), (130, 2, 3)])
def test_step_at_launch_edges(ax, orc, n, recon, ct):
    """One Heun step within 1e-10 of the oracle (the bound of the other parity tests of whole steps)."""
    import torch
    w = W.curved_block(seed=62, n=n, recon=recon, ng=4 if ct == "uct" else 3, nsteps=1, rk=2)
    w.params["ct"] = ct
    print("case step", n, recon, ct, flush=True)
    L = w.layout
    blk = ax.Block(w)
    blk.run(1)
    torch.cuda.synchronize()
    cons = orc.prim2con(L, w.params, w.metric, w.A, w.prim)
    orc.fill_ghosts(L, cons, w.bc_cell)
    state, prim = w.state(cons), w.prim.copy()
    orc.run(L, w.params, w.metric, w.curv, state, prim, w.dt, 1, w.rk, w.bc_cell, w.bc_A, A_shift=w.A_shift)
    assert_fields_close(blk.state.cpu().numpy(), state, 1e-10, L.owned, STATE_NAMES)
    assert_fields_close(blk.prim.cpu().numpy(), prim, 1e-10, L.owned, PRIM_NAMES)


@pytest.mark.parametrize("recon,ct,n", [("ppm", "fct", (33, 12, 10)), ("wenoz", "fct", (62, 5, 7)),
                                        ("mp5", "uct", (20, 13, 11))])
def test_stage_variants_agree(ax, n, recon, ct):
    """The same stage through the recovery with sources (asterx_c2p_src, asterx_rhs_rk_src), with stored geometry and
    without either: within 1e-13 of the fields' scales (they differ in the order of the interpolation's passes)."""
    import torch
    w = W.curved_block(seed=63, n=n, recon=recon, ng=4 if ct == "uct" else 3, nsteps=1)
    w.params["ct"] = ct
    L = w.layout
    print("case stage variants", n, recon, ct, flush=True)
    outs = {}
    for kind in ("plain", "src", "geo"):
        blk = ax.Block(w, src_in_c2p=False)
        U, out = blk.state, torch.zeros_like(blk.state)
        rk = [([1.0], [U], w.dt, out)]
        z = lambda nf: torch.zeros((nf,) + L.shape3, dtype=torch.float64, device="cuda")
        if kind == "plain":
            blk.stage(U, rk)
        elif kind == "src":
            src = z(ax.SRC_FIELDS)
            ax.c2p_src(L, w.params, blk.metric, blk.curv, U[5:8], U[0:5], blk.prim, src, blk.flags, blk.stats)
            ax.fill_ghosts(L, blk.prim, w.bc_cell)
            ax.rhs_rk_src(L, w.params, blk.metric, blk.prim, U[5:8], U[8:9], src, w.dt, rk, blk.red, blk.ws)
        else:
            src, geo = z(4), z(ax.GEO_FIELDS)
            ax.geometry(L, w.params, blk.metric, blk.curv, geo)
            ax.c2p_geo(L, w.params, geo, U[5:8], U[0:5], blk.prim, src, blk.flags, blk.stats)
            ax.fill_ghosts(L, blk.prim, w.bc_cell)
            ax.rhs_rk_geo(L, w.params, blk.metric, geo, blk.prim, U[5:8], U[8:9], src, w.dt, rk, blk.red, blk.ws)
        torch.cuda.synchronize()
        outs[kind] = (out.cpu().numpy(), blk.prim.cpu().numpy())
    for kind in ("src", "geo"):
        assert_fields_close(outs[kind][0], outs["plain"][0], 1e-13, L.owned, STATE_NAMES)
        assert_fields_close(outs[kind][1], outs["plain"][1], 1e-13, L.owned, PRIM_NAMES)


def test_block_without_room_for_the_geometry(ax, monkeypatch):
    """A block whose stored geometry cannot be allocated takes the recovery with sources: the same steps within 1e-13."""
    import torch
    w = W.curved_block(seed=64, n=(18, 9, 7), recon="ppm", nsteps=2, rk=4)
    print("case block without stored geometry", flush=True)
    ref = ax.Block(w)
    real = torch.empty

    def empty(*a, **k):
        if a and isinstance(a[0], tuple) and a[0][0] == ax.GEO_FIELDS:
            raise torch.OutOfMemoryError("no room")
        return real(*a, **k)

    monkeypatch.setattr(torch, "empty", empty)
    blk = ax.Block(w)
    monkeypatch.undo()
    assert blk.geo is None and ref.geo is not None
    for b in (ref, blk):
        b.run(2)
    torch.cuda.synchronize()
    assert torch.equal(blk.stats, ref.stats)
    assert_fields_close(blk.state.cpu().numpy(), ref.state.cpu().numpy(), 1e-13, w.layout.owned, STATE_NAMES)
    assert_fields_close(blk.prim.cpu().numpy(), ref.prim.cpu().numpy(), 1e-13, w.layout.owned, PRIM_NAMES)
