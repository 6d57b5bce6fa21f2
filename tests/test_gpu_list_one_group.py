"""Builds of up to 2,048 atoms and 8,192 bins run their first and last passes in one work-group:
at the edges of both limits and of the group's 1,024 threads, with empty cells and with several
cells, the list must be the oracle's and the evaluation on it the same as when the same cells are
built beside a larger one (by the general passes)."""
import numpy as np
import pytest
import torch

from oracle import neighbors as onb
from paper_2204_12573_amd import engine, structures as S

pytestmark = pytest.mark.gpu


def _part(n, seed, gap=6.0):
    """The first n atoms of a slab with gas, in a box of the slab's sides."""
    k = max(2, int(np.ceil(np.sqrt(n / 6.0))))
    st = S.h2_over_pt111(k + k % 2, k + k % 2, 6, gas_height=gap, jitter=0.05, seed=seed)
    order = np.random.default_rng(seed).permutation(st.n)[:n]
    return S.Structure(st.pos[order], st.species[order], st.box)


def _run(cells, m):
    off = np.concatenate([[0], np.cumsum([len(c.species) for c in cells])]).astype(np.int32)
    pos = np.concatenate([c.pos for c in cells])
    species = np.concatenate([c.species for c in cells])
    boxes = np.stack([np.asarray(c.box, float) for c in cells])
    model = engine.Model(*S.random_model(544))
    ev = engine.Evaluator(model, max_atoms=len(species), max_pairs=80 * len(species) + 4096)
    p, s = engine.to_device(pos, species)
    ev.neighbors(p, s, off, boxes, 0.2)
    lists = ev.export_list()
    out = ev.compute(p, want_var=True)
    torch.cuda.synchronize()
    assert ev.status() == 0
    return lists, {k: out[k][..., :m].clone() for k in ("e", "f", "var")}


@pytest.mark.parametrize("sizes,gap", [((1,), 6.0), ((63, 2), 6.0), ((1024,), 6.0), ((1025, 0, 700), 6.0),
                                       ((2048,), 6.0), ((2049,), 6.0), ((300,), 900.0),
                                       ((300,), 4000.0), ((50,) * 40, 6.0)])
def test_one_group_build(sizes, gap):
    cells = [_part(n, 7 + k, gap) for k, n in enumerate(sizes)]
    m = sum(sizes)
    print(f"case: cells of {sizes[:4]} atoms, gas {gap} A", flush=True)
    (off, j, sh), res = _run(cells, m)
    lo = 0
    for c in cells[:4]:
        n = len(c.species)
        oi, oj, os_ = onb.neighbor_list(c.pos, c.box, 4.7) if n else (np.zeros(0, int),) * 2 + (np.zeros((0, 3), int),)
        o = np.lexsort((os_[:, 2], os_[:, 1], os_[:, 0], oj, oi))
        a, b = off[lo], off[lo + n]
        got = np.column_stack([np.repeat(np.arange(n), np.diff(off[lo:lo + n + 1])), j[a:b] - lo, sh[a:b]])
        assert np.array_equal(got, np.column_stack([oi, oj, os_])[o])
        lo += n
    _, big = _run(cells + [S.adsorbed_slab(6000, 0.5, 9)], m)
    for k in res:
        assert torch.equal(res[k], big[k]), k
