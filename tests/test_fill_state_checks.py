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
