"""The list build's routes: 16 lanes an atom up to 81,920 atoms, one thread an atom beyond;
lists of more than the 32 cached pairs an atom (searched again, reverse pairs found in a
later pass); boxes with one, two and many bins a side. Every route must give the oracle's
pairs exactly, and the evaluation built on the list (its slots and reverse pairs) the same
forces when one structure's list is built alone or beside others that move the build to the
other route."""
import numpy as np
import pytest
import torch

from oracle import neighbors as onb
from paper_2204_12573_amd import engine, structures as S

pytestmark = pytest.mark.gpu


def _exact(ev, st, r_list, lo=0):
    off, j, sh = ev.export_list()
    n = st.n
    oi, oj, os_ = onb.neighbor_list(st.pos, st.box, r_list)
    o = np.lexsort((os_[:, 2], os_[:, 1], os_[:, 0], oj, oi))
    want = np.column_stack([oi, oj, os_])[o]
    a, b = off[lo], off[lo + n]
    i = np.repeat(np.arange(n), np.diff(off[lo:lo + n + 1]))
    got = np.column_stack([i, j[a:b] - lo, sh[a:b]])
    assert np.array_equal(got, want)


@pytest.mark.parametrize("nx,ny,nl,gap,skin", [(2, 2, 2, 3.0, 0.2), (1, 2, 1, 2.0, 0.5), (3, 4, 3, 9.0, 1.6),
                                               (6, 6, 12, 40.0, 0.2), (7, 8, 4, 2.0, 2.0)])
def test_list_of_small_and_dense_cells(nx, ny, nl, gap, skin):
    # narrow boxes list many images of each atom; a wide skin lists more than 32 pairs
    st = S.h2_over_pt111(nx, ny, nl, gas_height=gap, n_mol=2 if gap > 6 else 0, seed=3, density=0.0)
    print(f"case: {st.n} atoms, box {st.box}, skin {skin}", flush=True)
    model = engine.Model(*S.random_model(544))
    ev = engine.Evaluator(model, max_atoms=st.n, max_pairs=2000 * st.n)
    p, s = engine.to_device(st.pos, st.species)
    ev.neighbors(p, s, [0, st.n], st.box, skin)
    _exact(ev, st, 4.5 + skin)


def test_both_routes_give_the_same_evaluation():
    small = S.adsorbed_slab(700, 0.6, 5)
    dense = S.h2_over_pt111(4, 4, 3, gas_height=2.5, n_mol=0, seed=2)
    filler = S.adsorbed_slab(82_000, 0.5, 9)
    model = engine.Model(*S.random_model(544))
    runs = []
    for cells in ([small, dense], [small, dense, filler]):
        b = S.concat(cells)
        print(f"case: {b.n} atoms in {len(cells)} cells", flush=True)
        ev = engine.Evaluator(model, max_atoms=b.n, max_pairs=80 * b.n)
        p, s = engine.to_device(b.pos, b.species)
        ev.neighbors(p, s, b.offsets, b.boxes, 1.0)
        out = ev.compute(p, want_var=True)
        torch.cuda.synchronize()
        assert ev.status() == 0
        _exact(ev, small, 5.5)
        _exact(ev, dense, 5.5, lo=small.n)
        m = small.n + dense.n
        runs.append((out["e"][:m].clone(), out["f"][:, :m].clone(), out["sigma"][:m].clone(), out["E"][:2].clone()))
    for a, b in zip(*runs):
        assert torch.equal(a, b)
