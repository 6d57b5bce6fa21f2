"""The 544-wide quadratic forms over row counts around their edges: the padding tile (128
rows), the 16-row blocks, the switch between the few-row and the many-row kernel (2,560
padded rows) and the workspace chunk (16,384 rows). The reference is the FP64 matrices at the
FP32 vectors in numpy.

Tolerance. Operands carry 24 bits, the six part products drop less than 2^-23 of a term and
the sums are FP32 over at most 17 x 6 accumulations per product column and 40 additions of
the row sum, so an error is at most about 2^-24 (102 + 40) of sum_kl |d_k||M_kl||d_l|; rounding
errors of either sign add up like the square root of their number, 2^-24 * 12 = 7e-7 of that
sum. The random PSD forms are about 1/20 of the sum of absolute terms: 1.5e-5 of a form
pointwise; 1e-5 of the largest form is the FP32 bar used throughout. Rows must not depend
on how many others are evaluated with them: prefixes agree bit for bit."""
import numpy as np
import pytest
import torch

from paper_2204_12573_amd import binding as Bd, engine, structures as S

pytestmark = pytest.mark.gpu
ND = 544
NMAX = 16385


@pytest.fixture(scope="module")
def rows():
    d = np.random.default_rng(11).standard_normal((NMAX, ND))
    return (d / np.linalg.norm(d, axis=1, keepdims=True)).astype(np.float32)


@pytest.mark.parametrize("prec", [pytest.param(Bd.FP32, id="fp32"),
                                  pytest.param(Bd.BF16X6_SPLIT | Bd.VAR_FP32, id="bf16x6-var32"),
                                  pytest.param(Bd.BF16_SPLIT, id="bf16"), pytest.param(-1, id="fp32-full-sigma")])
@pytest.mark.parametrize("bucket", [4, 5])
def test_forms_at_row_counts(rows, bucket, prec):
    beta, sigma = S.random_model(ND)
    if prec < 0:                 # not positive definite: V from the full matrix
        sigma = sigma - 1e-4 * np.eye(ND)
        prec = Bd.FP32
        assert np.linalg.eigvalsh(sigma[0]).min() < 0
    model = engine.Model(beta, sigma, precision=prec)
    ev = engine.Evaluator(model, max_atoms=NMAX, max_pairs=1024)
    d64 = rows.astype(np.float64)
    e_ref = ((d64 @ beta[bucket - 4]) * d64).sum(1)
    v_ref = ((d64 @ sigma[bucket - 4]) * d64).sum(1)
    dev = torch.from_numpy(rows).cuda()
    last = None
    for n in (NMAX, 2561, 2560, 2433, 2432, 129, 128, 17, 16, 1):
        print(f"case: bucket {bucket}, precision {prec}, {n} rows", flush=True)
        e, v = ev.quadratic_forms(bucket, dev[:n].contiguous())
        torch.cuda.synchronize()
        assert np.abs(e.cpu().numpy() - e_ref[:n]).max() <= 1e-5 * np.abs(e_ref).max()
        assert np.abs(v.cpu().numpy() - v_ref[:n]).max() <= 1e-5 * np.abs(v_ref).max()
        if last is not None:
            assert torch.equal(e, last[0][:n]) and torch.equal(v, last[1][:n])
        last = (e, v)
