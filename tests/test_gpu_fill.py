"""The one-pass ghost fill against axis passes (x, then y, then z, each over the full extents of the others), bit for
bit: every mix of boundary kinds, blocks thinner than their ghosts, the smallest extrapolated block, whole states with
kinds of their own for the potential, and a batch."""
import itertools

import numpy as np
import pytest

from paper_2406_11669_amd import workloads as W

pytestmark = pytest.mark.gpu
KINDS = ("periodic", "copy", "linear")


def _passes(L, f, kinds, shift=None):
    """Axis passes on fields f (nf, z, y, x) in place."""
    for d in range(3):
        n, ng, ax = L.n[d], L.ng, 2 - d
        line = lambda s: tuple([slice(None)] * ax + [s + ng])
        for q in range(f.shape[0]):
            F = f[q]
            for s in list(range(-ng, 0)) + list(range(n, n + ng + 1)):
                if kinds[d] == "periodic":
                    v = F[line(s % n)].copy()
                    if shift is not None and shift[q][d] != 0.0:
                        v = v + float((s - s % n) // n) * shift[q][d]
                elif kinds[d] == "copy":
                    v = F[line(0 if s < 0 else n - 1)].copy()
                elif s < 0:
                    v = F[line(0)] + float(s) * (F[line(1)] - F[line(0)])
                else:
                    v = F[line(n - 1)] + float(s - n + 1) * (F[line(n - 1)] - F[line(n - 2)])
                F[line(s)] = v


def _field(L, nf, seed):
    f = np.full((nf,) + L.shape3, np.nan)
    L.owned(f)[...] = np.random.default_rng(seed).normal(size=L.owned(f).shape)
    return f


def _ext(L, f):
    e = [m + 2 * L.ng + 1 for m in L.n]
    return f[..., :e[2], :e[1], :e[0]]


@pytest.fixture(scope="module")
def ax():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2406_11669_amd import asterx
    asterx.lib()
    return asterx


@pytest.mark.parametrize("n", [(2, 2, 2), (2, 7, 3), (33, 5, 6)])
def test_fill_every_mix_of_kinds(ax, n):
    import torch
    L = W.Layout(n, 3)
    for i, kinds in enumerate(itertools.product(KINDS, repeat=3)):
        print("case fill", n, kinds, flush=True)
        f = _field(L, 4, i)
        t = torch.from_numpy(f.copy()).cuda()
        ax.fill_ghosts(L, t, kinds)
        _passes(L, f, kinds)
        assert np.array_equal(_ext(L, t.cpu().numpy()), _ext(L, f)), kinds


@pytest.mark.parametrize("n,ng", [((2, 3, 4), 3), ((19, 6, 5), 4)])
@pytest.mark.parametrize("cell,A", [("copy", "linear"), ("periodic", "periodic"), ("linear", "copy"), ("copy", "shift")])
def test_fill_state(ax, n, ng, cell, A):
    import torch
    L = W.Layout(n, ng)
    print("case fill_state", n, ng, cell, A, flush=True)
    shift = np.array([[0.0, 0.5, -1.25], [2.0, 0.0, 0.1], [0.3, 0.7, 0.0]]) if A == "shift" else None
    kA = ("periodic" if A == "shift" else A,) * 3
    u = _field(L, 9, 5)
    t = torch.from_numpy(u.copy()).cuda()
    ax.fill_state(L, t, (cell,) * 3, kA, shift)
    for part, kinds, sh in ((u[0:5], (cell,) * 3, None), (u[5:8], kA, shift), (u[8:9], (cell,) * 3, None)):
        _passes(L, part, kinds, sh)
    assert np.array_equal(_ext(L, t.cpu().numpy()), _ext(L, u))


def test_fill_state_batch(ax):
    import torch
    wls = [W.riemann_block(seed=s, n=n) for s, n in ((3, (16, 8, 8)), (4, (9, 12, 7)))]
    b = ax.Batch(wls)
    rng = np.random.default_rng(9)
    b.state.copy_(torch.from_numpy(rng.normal(size=tuple(b.state.shape))))
    before = b.state.cpu().clone()
    b.fill_state(b.state)
    torch.cuda.synchronize()
    for p, w in enumerate(wls):
        L = w.layout
        u = b.unpack(before, p).numpy().copy()
        for part, kinds in ((u[0:5], w.bc_cell), (u[5:8], w.bc_A), (u[8:9], w.bc_cell)):
            _passes(L, part, kinds)
        assert np.array_equal(_ext(L, b.unpack(b.state, p).cpu().numpy()), _ext(L, u)), p
