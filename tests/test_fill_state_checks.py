"""Argument checks of the whole-state ghost fills, which the library cannot make (it sees an address)."""
import pytest
import torch

from paper_2406_11669_amd import asterx as ax


@pytest.mark.parametrize("nf", [0, 5, 8])
def test_batch_fill_state_refuses_partial_states(nf):
    """Fewer than nine fields: refused before the pointer is taken (a launch would write past the tensor's end)."""
    b = ax.Batch.__new__(ax.Batch)
    b.h, b.bc_cell, b.bc_A = None, ("copy",) * 3, ("linear",) * 3
    with pytest.raises(ValueError, match="nine fields"):
        b.fill_state(torch.zeros((nf, 64), dtype=torch.float64))


@pytest.mark.parametrize("kinds_A", [None, ("unused",) * 3])
def test_fill_state_with_shift_ignores_the_potentials_kinds(monkeypatch, kinds_A):
    """A potential filled with a shift per period has no boundary kinds: whatever stands there is not looked at."""
    from paper_2406_11669_amd import workloads as W
    calls = []

    class Lib:
        def asterx_fill_state(self, g, u, kinds_cell, kA, shift, stream):
            calls.append((list(kinds_cell), kA, list(shift)))
            return 0

    monkeypatch.setattr(ax, "lib", Lib)
    monkeypatch.setattr(ax, "_ptr", lambda t: None)
    monkeypatch.setattr(ax, "_stream", lambda s: None)
    L = W.Layout((4, 4, 4), 3)
    ax.fill_state(L, torch.zeros((9,) + L.shape3, dtype=torch.float64), ("periodic",) * 3, kinds_A,
                  [[0.0, 1.0, 2.0]] * 3)
    assert calls == [([ax.BC["periodic"]] * 3, None, [0.0, 1.0, 2.0] * 3)]
