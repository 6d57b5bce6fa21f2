"""The three row addresses of a [3, N] array taken from its base and stride, against those of
its rows, over the layouts a caller can pass."""
import numpy as np
import pytest
import torch

from paper_2204_12573_amd import binding as B

BASE = torch.arange(240, dtype=torch.float64)
LAYOUTS = {
    "contiguous": BASE.view(3, 80),
    "wide rows": BASE.view(4, 60)[:3, :7],
    "more rows": BASE.view(6, 40),
    "transposed": BASE.view(80, 3).t(),
    "offset": BASE.view(3, 80)[:, 5:],
    "broadcast": BASE[:80].expand(3, 80),
    "one atom": BASE[:3].view(3, 1),
    "empty": torch.empty((3, 0)),
    "float32": BASE.float().view(3, 80),
    "parameter": torch.nn.Parameter(BASE.clone().view(3, 80)),
    "rows apart": [BASE[100:180], BASE[:80], BASE[40:120]],
    "numpy": np.zeros((3, 5)),
}


@pytest.mark.parametrize("name", list(LAYOUTS))
def test_row_addresses(name):
    t = LAYOUTS[name]
    assert tuple(B.row_ptrs(t)) == (B.ptr(t[0]), B.ptr(t[1]), B.ptr(t[2]))


def test_too_few_rows_refused():
    with pytest.raises(IndexError):
        B.row_ptrs(BASE[:160].view(2, 80))
