"""Virial of batches whose longest reduction task picks each size of work-group (64, 256, 1,024
threads) at the edges of its range: every cell gives the same bits as alone, whatever the batch
it is in (against the oracle: test_gpu_virial.py). A batch of many small cells also in time: with 1,024
threads a cell of four atoms the virial took four fifths of the whole evaluation."""
import numpy as np
import pytest
import torch

from paper_2204_12573_amd import engine, structures as S

pytestmark = pytest.mark.gpu


def _cell(n, seed):
    """n atoms of both species, jittered around a cubic grid of 2.6 A."""
    rng = np.random.default_rng(seed)
    g = max(2, int(np.ceil(n ** (1 / 3))))
    at = np.stack(np.meshgrid(*[np.arange(g)] * 3, indexing="ij"), -1).reshape(-1, 3)[:n]
    return S.Structure(2.6 * at + rng.uniform(0, 0.5, (n, 3)), rng.integers(0, 2, n).astype(np.int32), np.full(3, 2.6 * g))


def _evaluator(model, cells):
    b = S.concat(cells)
    ev = engine.Evaluator(model, max_atoms=b.n, max_pairs=200 * b.n)
    p, s = engine.to_device(b.pos, b.species)
    ev.neighbors(p, s, b.offsets, b.boxes, 0.2)
    return ev, p


def _virial(model, cells):
    ev, p = _evaluator(model, cells)
    ev.compute(p)
    return ev.virial().cpu().numpy()


@pytest.mark.parametrize("sizes", [(1, 15, 16, 17, 63, 64), (3, 64, 65, 128, 255, 256), (5, 64, 256, 257, 1025),
                                   (40, 256, 2048, 2049, 5000)])
def test_same_bits_alone_and_in_a_batch(sizes):
    model = engine.Model(*S.random_model(544))
    cells = [_cell(n, n) for n in sizes]
    print(f"case: cells of {sizes} atoms", flush=True)
    w = _virial(model, cells)
    for k, c in enumerate(cells):
        assert np.array_equal(w[k], _virial(model, [c])[0]), c.n


def test_time_of_many_small_cells():
    model = engine.Model(*S.random_model(544))
    ev, p = _evaluator(model, [_cell(4, k) for k in range(8000)])
    print("case: 8,000 cells of 4 atoms", flush=True)
    out, w = ev.compute(p), ev.virial()

    def time_of(fn):
        best = 1e9
        for _ in range(5):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(20):
                fn()
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        return best

    assert time_of(lambda: ev.virial(w)) < 0.4 * time_of(lambda: ev.compute(p, out=out))
