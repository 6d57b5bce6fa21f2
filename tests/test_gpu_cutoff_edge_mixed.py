"""Rows that list both species but have one neighbour inside the cutoff, just inside it: |d~| goes
down to 1e-27 and its square below the FP32 range, while the normalised descriptor, the energy
and the uncertainty are ordinary. Cells of a centre, one atom of species t at r_c - delta and
one of the other species between r_c and the list radius, both centre species, against the FP64
oracle; alone (the kernels for few rows) and beside a slab of 20 k atoms (those for many).

The distances are FP32 numbers along an axis, so that the pair vector is exact and the norm,
which goes with delta^4, can be compared too.

Tolerance. e, sigma and |d~| of the mixed rows: the FP32 bar in every form. A force is the sum of
an ordinary term and of one of size (2 / delta) e that cancels exactly (d does not change with the
size of d~); rounding leaves up to about 2^-22 of it per product chain, and the neighbour's own
row, 144 wide, has its form's error: 40 x 2^-22 (2 / delta) e beside the form's bar, both in
proportion to it."""
import numpy as np
import pytest
import torch

from oracle import evaluate as oev
from paper_2204_12573_amd import binding as Bd, engine, structures as S

pytestmark = pytest.mark.gpu
BAR = {Bd.FP32: 1e-5, Bd.BF16X6_SPLIT: 1e-5, Bd.BF16X6_SPLIT | Bd.VAR_FP32: 1e-5, Bd.BF16_SPLIT: 1e-4,
       Bd.FP8_SPLIT: 1e-2}


def _cells():
    cells = []
    for ulps in (1 << 20, 1 << 14, 1 << 8, 21, 6, 1):       # of 2^-21, the spacing of FP32 numbers at r_c
        for centre in (0, 1):
            for t in (0, 1):
                axis = len(cells) % 3
                pos = np.full((3, 3), 10.0)
                pos[1, axis] += 4.5 - ulps * 2.0 ** -21
                pos[2, axis] -= 4.625
                sp = np.array([centre, t, 1 - t], np.int32)
                cells.append((ulps * 2.0 ** -21, S.Structure(pos, sp, np.full(3, 30.0))))
    return cells


@pytest.mark.parametrize("many", [False, True])
@pytest.mark.parametrize("prec", sorted(BAR))
def test_one_neighbour_at_the_cutoff_of_a_mixed_row(prec, many):
    beta, sigma = S.random_model(544)
    cells = _cells()
    b = S.concat([c for _, c in cells] + ([S.adsorbed_slab(20_000, 0.5, 9)] if many else []))
    ev = engine.Evaluator(engine.Model(beta, sigma, precision=prec), max_atoms=b.n, max_pairs=64 * b.n + 4096)
    print(f"case: precision {prec}, {b.n} atoms", flush=True)
    p, s = engine.to_device(b.pos, b.species)
    ev.neighbors(p, s, b.offsets, b.boxes, 0.2)
    d, norm = ev.descriptors(p, want_d=True, want_norm=True)
    out = ev.compute(p, want_var=True)
    m = 3 * len(cells)
    got = {k: out[k][..., :m].cpu().numpy() for k in ("e", "f", "sigma")}
    # a separate backward (energies first, then forces) and the variance alone
    ev.descriptors(p)
    ev.energies()
    f2 = ev.forces()[:, :m].cpu().numpy()
    ev.descriptors(p)
    sg2 = ev.variance()["sigma"][:m].cpu().numpy()
    d, norm = d[:m].cpu().numpy().astype(np.float64), norm[:m].cpu().numpy()
    assert all(np.isfinite(x).all() for x in (*got.values(), f2, sg2, d, norm))
    refs = [oev.evaluate(c.pos, c.species, c.box, beta, sigma) for _, c in cells]
    e_max = max(np.abs(r.e).max() for r in refs)
    f_max = max(np.abs(r.f).max() for r in refs)
    for k, ((dl, _), r) in enumerate(zip(cells, refs)):
        i, q = 3 * k, slice(3 * k, 3 * k + 3)
        assert abs(norm[i] - r.norm[0]) <= 1e-5 * r.norm[0], (k, dl)
        assert abs((d[i] ** 2).sum() - 1.0) <= 1e-6, (k, dl)
        assert abs(got["e"][i] - r.e[0]) <= 1e-5 * e_max, (k, dl)
        for sg in (got["sigma"], sg2):
            assert abs(sg[i] - r.sigma[0]) <= 1e-5 * r.sigma[0], (k, dl)
        noise = BAR[prec] / 1e-5 * 40 * 2.0 ** -22 * 2.0 / dl * e_max
        for f in (got["f"], f2):
            assert np.abs(f.T[q] - r.f).max() <= BAR[prec] * f_max + noise, (k, dl)
