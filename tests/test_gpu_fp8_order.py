"""The FP8 form's descriptors and energies follow the order of sums that the form documents: slots
in list order, the products of a pair's harmonics in turn, with the last channel the two first
exchanged. Its energy pass is a step function of d~ (two e4m3 parts of the scaled row), so
another order moves a row's energy and forces by far more than rounding.

d~ is emulated on the CPU in FP32 with that order and compared bit for bit: with the exported
descriptors, and through the energy pass itself, by giving the emulated rows to the quadratic
forms (no normalisation there: e of the row is their value times 1 / |d~|^2).

Cells of four equal atoms in a box of one bin, so that the list order is the plain one: images
z, y, x, then atoms. 12,000 rows take the kernels for few rows, 32,000 those for many."""
import numpy as np
import pytest
import torch

from paper_2204_12573_amd import binding as B, engine, structures as S

F, RC, SKIN, BOX = np.float32, 4.5, 0.2, 9.0


def _fma(a, b, c):
    return (a.astype(np.float64) * b + c).astype(F)        # the product of two FP32 values is exact


def _harmonics(x, y, z):
    k0, k1, k2a, k20, k22 = map(F, (0.28209479177387814, 0.48860251190291992, 1.0925484305920792,
                                    0.31539156525252005, 0.54627421529603959))
    k33, k32a, k31, k30, k32b = map(F, (0.59004358992664352, 2.8906114426405538, 0.45704579946446572,
                                        0.37317633259011540, 1.4453057213202769))
    xx, yy, zz = x * x, y * y, z * z
    dxy = _fma(-y, y, xx)
    z4 = _fma(-y, y, _fma(F(4), zz, -xx))
    return [k0 + 0 * x, k1 * y, k1 * z, k1 * x, k2a * x * y, k2a * y * z, k20 * _fma(-y, y, _fma(F(2), zz, -xx)),
            k2a * x * z, k22 * dxy, k33 * y * _fma(F(3), xx, -yy), k32a * x * y * z, k31 * y * z4,
            k30 * z * _fma(F(-3), yy, _fma(F(2), zz, F(-3) * xx)), k31 * x * z4, k32b * z * dxy,
            k33 * x * _fma(F(-3), yy, xx)]


def _densities(pos):
    """c [rows, 8, 16] in FP32 for cells pos [cells, 4, 3]."""
    n = pos.shape[0] * 4
    c = np.zeros((n, 8, 16), F)
    for sz in (-1, 0, 1):
        for sy in (-1, 0, 1):
            for sx in (-1, 0, 1):
                for j in range(4):
                    d = (pos[:, j][:, None] - pos) + np.array([sx, sy, sz]) * BOX
                    f = d.reshape(n, 3).astype(F)
                    r2 = _fma(f[:, 2], f[:, 2], _fma(f[:, 1], f[:, 1], f[:, 0] * f[:, 0]))
                    k = np.nonzero((r2 > 0) & (r2 < F(RC * RC)))[0]
                    r = np.sqrt(r2[k])
                    inv = F(1) / r
                    y = np.stack(_harmonics(*(f[k, a] * inv for a in range(3))), 1)
                    x = _fma(r, F(2) / F(RC), F(-1))
                    t = [np.ones_like(x), x]
                    while len(t) < 8:
                        t.append(_fma(F(2) * x, t[-1], -t[-2]))
                    rad = np.stack(t, 1) * ((F(RC) - r) * (F(RC) - r))[:, None]
                    c[k] = _fma(rad[:, :, None], y[:, None, :], c[k])
    return c


def _b2(c):
    """d~ [rows, 144]."""
    def chain(a, b, q):
        s = a[:, q[0]] * b[:, q[0]]
        for m in q[1:]:
            s = _fma(a[:, m], b[:, m], s)
        return s
    out = []
    for p in range(8):
        for q in range(p, 8):
            a, b = c[:, p], c[:, q]
            first = [(2, 1, 3), (5, 4, 6, 7), (10, 9, 11), (13, 12, 14, 15)] if q == 7 else \
                [(1, 2, 3), (4, 5, 6, 7), (9, 10, 11), (12, 13, 14, 15)]
            v = [chain(a, b, o) for o in first]
            out += [a[:, 0] * b[:, 0], v[0], _fma(a[:, 8], b[:, 8], v[1]), v[2] + v[3]]
    return np.stack(out, 1)


def _norms(dt):
    """|d~|: FP32 squares in pairs, FP64 sums of each half of the components, rounded once."""
    x = dt.reshape(len(dt), 36, 2, 2)
    sq = _fma(x[..., 0], x[..., 0], x[..., 1] * x[..., 1]).astype(np.float64)
    half = np.zeros((len(dt), 2))
    for k in range(36):
        half += sq[:, k]
    return np.sqrt(half.sum(1)).astype(F)


def _cells(n, seed):
    rng = np.random.default_rng(seed)
    pos = np.empty((n, 4, 3))
    for k in range(n):
        while True:
            p = rng.uniform(0, BOX, (4, 3))
            d = p[:, None] - p
            d = np.sqrt(((d - BOX * np.round(d / BOX)) ** 2).sum(-1))[np.triu_indices(4, 1)]
            if d.min() > 0.7:
                break
        pos[k] = p
    return pos


@pytest.mark.gpu
@pytest.mark.parametrize("cells", [3000, 8000])
def test_fp8_order_of_sums(cells):
    beta, sigma = S.random_model(544)
    model = engine.Model(beta, sigma, precision=B.FP8_SPLIT)
    ev = engine.Evaluator(model, max_atoms=4 * cells, max_pairs=200 * cells)
    pos = _cells(cells, 3)
    species = np.repeat(np.arange(cells) % 2, 4).astype(np.int32)
    print(f"case: {cells} cells of four atoms", flush=True)
    p, s = engine.to_device(pos.reshape(-1, 3), species)
    ev.neighbors(p, s, np.arange(cells + 1) * 4, np.full((cells, 3), BOX), SKIN)
    d, norm = (t.cpu().numpy() for t in ev.descriptors(p, want_d=True, want_norm=True))
    fused = ev.energy_forces()["e"].cpu().numpy()
    alone = ev.energies()["e"].cpu().numpy()
    c = _densities(pos)
    for sp, bucket, block in ((0, 0, slice(0, 144)), (1, 3, slice(400, 544))):
        k = (species == sp) & (norm > 0)
        dt = _b2(c[k])
        nrm = _norms(dt)
        assert np.array_equal(nrm, norm[k])
        assert np.array_equal(d[k][:, block], dt / nrm[:, None])
        e = ev.quadratic_forms(bucket, torch.from_numpy(dt).cuda())[0].cpu().numpy() * (F(1) / (nrm * nrm))
        assert np.array_equal(fused[k], e) and np.array_equal(alone[k], e)
