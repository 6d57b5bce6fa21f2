"""Calls between the energies and the separate backward at the same positions: variances and the
monitor form the mixed rows' descriptors again in the same workspace, without the densities and
the geometry that the backward reads. Its forces and the virial must be the fused call's, bit for
bit, with few rows, with many, and with more mixed rows than one chunk of the workspace."""
import numpy as np
import pytest
import torch

from paper_2204_12573_amd import engine, structures as S

pytestmark = pytest.mark.gpu


def _alloy(n_cells):
    rng = np.random.default_rng(6)
    at = np.stack(np.meshgrid(*[np.arange(4)] * 3, indexing="ij"), -1).reshape(-1, 3) * 2.6
    return [S.Structure(at + rng.uniform(0, 0.5, (64, 3)), rng.integers(0, 2, 64).astype(np.int32), np.full(3, 10.4))
            for _ in range(n_cells)]


CASES = {"few": lambda: [S.adsorbed_slab(700, 0.6, 5)], "many": lambda: [S.adsorbed_slab(30_000, 0.6, 5)],
         "all mixed": lambda: _alloy(20), "chunks": lambda: _alloy(300)}


@pytest.mark.parametrize("name", sorted(CASES))
def test_variance_and_monitor_before_the_backward(name):
    b = S.concat(CASES[name]())
    print(f"case: {name}, {b.n} atoms", flush=True)
    ev = engine.Evaluator(engine.Model(*S.random_model(544)), max_atoms=b.n, max_pairs=100 * b.n)
    p, s = engine.to_device(b.pos, b.species)
    ev.neighbors(p, s, b.offsets, b.boxes, 0.2)
    ref = {k: v.clone() for k, v in ev.compute(p).items()}
    w = ev.virial().clone()
    q = p + 0.01
    ev.descriptors(q)          # other positions in between: nothing of the first pass may be left
    ev.energies()
    ev.descriptors(p)
    e = ev.energies()["e"]
    var = ev.variance()["var"]
    cells = len(b.boxes)
    ev.uncertainty_monitor(1.0, torch.zeros(cells, device="cuda"), torch.zeros(cells, dtype=torch.int32, device="cuda"))
    f = ev.forces()
    assert torch.equal(e, ref["e"]) and torch.equal(var, ref["var"]) and torch.equal(f, ref["f"])
    assert torch.equal(ev.virial(), w)


def test_export_over_chunks():
    """Descriptors and norms written out: the same bits from one chunk of mixed rows and from two,
    norms alone the same as beside the descriptors, and an evaluation after them undisturbed."""
    cells = _alloy(300)
    model = engine.Model(*S.random_model(544))
    got = []
    for n in (20, 300):
        b = S.concat(cells[:n])
        print(f"case: {b.n} atoms", flush=True)
        ev = engine.Evaluator(model, max_atoms=b.n, max_pairs=100 * b.n)
        p, s = engine.to_device(b.pos, b.species)
        ev.neighbors(p, s, b.offsets, b.boxes, 0.2)
        d, norm = ev.descriptors(p, want_d=True, want_norm=True)
        alone = ev.descriptors(p, want_norm=True)[1]
        f = ev.energy_forces()["f"]
        m = 20 * 64
        assert torch.equal(norm, alone)
        assert float((d.double().square().sum(1) - 1).abs().max()) < 1e-6
        got.append((d[:m].clone(), norm[:m].clone(), f[:, :m].clone()))
    for a, b in zip(*got):
        assert torch.equal(a, b)
