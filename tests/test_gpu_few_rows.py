"""Few rows: the kernel that shares a 32-row sub-tile out over four waves, with the mixed rows'
descriptors in the same launch, against the kernels for many rows. A structure's atoms are the
same rows alone and beside a large second cell, and every product and sum has the same order on
both routes: descriptors, norms, energies, forces and variances must agree bit for bit, in each
arithmetic, from one fused call and from the calls one by one, also where a row lists more than
the 48 slots whose pair terms are kept on chip."""
import pytest
import torch

from paper_2204_12573_amd import binding as B, engine, structures as S

pytestmark = pytest.mark.gpu

CELLS = {
    "slab": lambda: [S.adsorbed_slab(700, 0.6, 5)],
    "gas_only_and_bare_metal": lambda: [S.h2_over_pt111(4, 4, 3, gas_height=60.0, seed=2),
                                        S.h2_over_pt111(5, 6, 6, gas_height=20.0, n_mol=0, seed=3)],
    "one_cell": lambda: [S.config_tiny(seed=4)],
    "near_the_limit": lambda: [S.adsorbed_slab(11500, 0.15, 7)],
}


def _run(model, b, m, skin):
    ev = engine.Evaluator(model, max_atoms=b.n, max_pairs=110 * b.n)
    p, s = engine.to_device(b.pos, b.species)
    ev.neighbors(p, s, b.offsets, b.boxes, skin)
    d, nrm = ev.descriptors(p, want_d=True, want_norm=True)
    out = ev.compute(p, want_var=True)
    res = {"d": d[:m].clone(), "norm": nrm[:m].clone(), "e": out["e"][:m].clone(),
           "f": out["f"][:, :m].clone(), "var": out["var"][:m].clone()}
    ev.descriptors(p)
    res["e alone"] = ev.energies()["e"][:m].clone()
    res["f alone"] = ev.forces()[:, :m].clone()
    ev.descriptors(p)
    res["var alone"] = ev.variance()["var"][:m].clone()
    torch.cuda.synchronize()
    assert ev.status() == 0
    return res


@pytest.mark.parametrize("prec", [B.FP32, B.BF16_SPLIT, B.FP8_SPLIT, B.BF16X6_SPLIT, B.BF16X6_SPLIT | B.VAR_FP32])
@pytest.mark.parametrize("name,skin", [("slab", 0.2), ("gas_only_and_bare_metal", 1.9), ("one_cell", 0.2),
                                       ("near_the_limit", 0.2)])
def test_same_bits_as_the_kernels_for_many_rows(name, skin, prec):
    model = engine.Model(*S.random_model(544), precision=prec)
    cells = CELLS[name]()
    b = S.concat(cells)
    print(f"case: {name}, {b.n} atoms, skin {skin}, precision {prec}", flush=True)
    few = _run(model, b, b.n, skin)
    many = _run(model, S.concat(cells + [S.adsorbed_slab(20_000, 0.5, 9)]), b.n, skin)
    for k, a in few.items():
        assert torch.equal(a, many[k]), k
    assert torch.equal(few["f"], few["f alone"]) and torch.equal(few["var"], few["var alone"])
