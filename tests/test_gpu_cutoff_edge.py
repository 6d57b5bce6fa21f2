"""Atoms whose only neighbour is just inside the cutoff: the densities are of the size
(r_c - r)^2 and |d~|^2 of its fourth power, far below the FP32 range, while the normalised
descriptor, the energy and the uncertainty are ordinary. Two equal atoms a distance
r_c - delta apart (and one pair at an ordinary distance in the same call) against the FP64
oracle.

Tolerance. e and sigma depend on r smoothly once d~ is normalised: the form's own bar. A
force is the sum of an ordinary term and of one of size (2 / delta) e that cancels exactly
(d does not change with the size of d~), so rounding leaves up to about 2^-22 of it per
product chain: 40 x 2^-22 (2 / delta) e beside the form's bar."""
import numpy as np
import pytest
import torch

from oracle import evaluate as oev
from paper_2204_12573_amd import binding as Bd, engine, structures as S

pytestmark = pytest.mark.gpu
BAR = {Bd.FP32: 1e-5, Bd.BF16X6_SPLIT: 1e-5, Bd.BF16_SPLIT: 1e-4, Bd.FP8_SPLIT: 1e-2}


@pytest.mark.parametrize("prec", sorted(BAR))
def test_single_neighbour_at_the_cutoff(prec):
    beta, sigma = S.random_model(544)
    model = engine.Model(beta, sigma, precision=prec)
    ev = engine.Evaluator(model, max_atoms=64, max_pairs=4096)
    deltas = [1e-2, 1e-4, 1e-5, 3e-6]
    cells = []
    for sp in (0, 1):
        for dl in [1.5] + deltas:
            u = np.array([0.6, 0.48, 0.64])
            pos = np.stack([np.full(3, 10.0), 10.0 + (4.5 - dl) * u])
            cells.append((dl, S.Structure(pos, np.full(2, sp, np.int32), np.full(3, 30.0))))
    b = S.concat([c for _, c in cells])
    print(f"case: precision {prec}, {b.n} atoms", flush=True)
    p, s = engine.to_device(b.pos, b.species)
    ev.neighbors(p, s, b.offsets, b.boxes, 0.2)
    out = ev.compute(p, want_var=True)
    torch.cuda.synchronize()
    e, f, sg = out["e"].cpu().numpy(), out["f"].cpu().numpy().T, out["sigma"].cpu().numpy()
    # the gradients of a separate backward (energies first, then forces) as well
    ev.descriptors(p)
    ev.energies()
    f2 = ev.forces().cpu().numpy().T
    assert np.isfinite(e).all() and np.isfinite(f).all() and np.isfinite(sg).all() and np.isfinite(f2).all()
    refs = [oev.evaluate(c.pos, c.species, c.box, beta, sigma) for _, c in cells]
    e_max = max(np.abs(r.e).max() for r in refs)
    f_max = max(np.abs(r.f).max() for r in refs)
    for k, ((dl, _), r) in enumerate(zip(cells, refs)):
        q = slice(2 * k, 2 * k + 2)
        assert np.abs(e[q] - r.e).max() <= BAR[prec] * e_max, dl
        assert np.abs(sg[q] - r.sigma).max() <= 1e-5 * np.abs(r.sigma).max(), dl
        noise = BAR[prec] / 1e-5 * 40 * 2.0 ** -22 * 2.0 / dl * e_max
        assert np.abs(f[q] - r.f).max() <= BAR[prec] * f_max + noise, dl
        assert np.abs(f2[q] - r.f).max() <= BAR[prec] * f_max + noise, dl
