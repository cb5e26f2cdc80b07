"""Working sets around the sizes where a column solve changes its path.

One response is the sum of m others, so its working set holds about m
coordinates: 32 (register rows), one lane per coordinate up to 64, two up to
128, the dense tier beyond; against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from tests.parity import rel_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_15031_amd import spmesl
    c = spmesl.Context(0)
    yield c
    c.close()


# 1e-6 in double and mixed: both stop at 1e-10 in double
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("m", [31, 32, 33, 63, 64, 65, 100, 126, 127, 128, 129])
def test_working_set_sizes(ctx, prec, m):
    rng = np.random.default_rng(m)
    X = rng.standard_normal((700, 160))
    X[:, 7] = X[:, 20:20 + m].sum(1) + 2.0 * rng.standard_normal(700)
    ref = oracle.spmesl(X, 0.06, tol=1e-12, original_scale=True)
    r = ctx.solve(torch.from_numpy(X).to("cuda:0"), 0.06, tol=1e-10, precision=prec)
    for got, want in ((r.B, ref["B"]), (r.sigma, ref["sigma"]), (r.Omega, ref["Omega"])):
        assert rel_err(got.cpu().numpy(), want) <= 1e-6
    assert r.stats["columns_noconv"] == 0


# the double Gram matrix of the mixed form's polish: rows around its blocks of
# 16 (m + 1 of them), samples around its steps of 32 and 16, odd and even
@pytest.mark.parametrize("n", [41, 64, 250, 701])
@pytest.mark.parametrize("m", [3, 7, 8, 14, 15, 16, 17, 30])
def test_polish_gram_sizes(ctx, m, n):
    rng = np.random.default_rng(100 * m + n)
    X = rng.standard_normal((n, 50))
    X[:, 7] = X[:, 20:20 + m].sum(1) + 0.5 * rng.standard_normal(n)
    lam0 = 0.4 if n < 100 else 0.15
    ref = oracle.spmesl(X, lam0, tol=1e-12, original_scale=True)
    r = ctx.solve(torch.from_numpy(X).to("cuda:0"), lam0, tol=1e-10, precision="mixed")
    for got, want in ((r.B, ref["B"]), (r.sigma, ref["sigma"]), (r.Omega, ref["Omega"])):
        assert rel_err(got.cpu().numpy(), want) <= 1e-6
