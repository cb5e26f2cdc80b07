"""The dense tier at the edges of its paths.

Working-set unions of one block or less (each column iterated by its own
wave), of up to 384 rows (gradients and coefficients in LDS) and beyond, with
sample counts around the 16 samples of a round and the 768 whose residuals
fit LDS, for every block size, against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from tests.parity import rel_err, standardized_cov

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_15031_amd import spmesl
    c = spmesl.Context(0)
    yield c
    c.close()


def _data(n, p, seed=0):
    rng = np.random.default_rng(1000 * n + p + seed)
    return rng.standard_normal((n, p)) + 0.4 * rng.standard_normal((n, 1))


def _solve(ctx, X, lam0, **kw):
    r = ctx.solve(torch.from_numpy(X).to("cuda:0"), lam0, tol=1e-10, max_outer=200, max_sweeps=20000, **kw)
    assert r.stats["columns_noconv"] == 0
    return r


# V of the 16-column groups: up to 64 rows, 65 and a few more, a few hundred;
# n on either side of a round of 16 samples and of 768
@pytest.mark.parametrize("n,p,lam0", [(5, 3, 0.6), (15, 9, 0.5), (33, 64, 0.45), (113, 65, 0.1), (112, 82, 0.1),
                                      (768, 70, 0.02), (769, 150, 0.03), (801, 64, 0.02)])
def test_data_form_paths(ctx, n, p, lam0):
    # 1e-6: the double forms' bar; both sides stop at 1e-10 or below
    X = _data(n, p)
    ref = oracle.spmesl(X, lam0, tol=1e-12, original_scale=True)
    r = _solve(ctx, X, lam0, precision="fp64", data_form=True)
    for got, want in ((r.B, ref["B"]), (r.sigma, ref["sigma"]), (r.Omega, ref["Omega"])):
        assert rel_err(got.cpu().numpy(), want) <= 1e-6


@pytest.mark.parametrize("b", [16, 32, 64])
@pytest.mark.parametrize("p", [210, 384, 385, 421])
def test_dense_tier_rows_around_the_lds_limit(ctx, b, p):
    # small penalties (the supports beyond 128 total fewer than 32 p + 65536
    # entries): (nearly) every variable is in some column's working
    # set, so a group's V has about p rows, on either side of the 384.  The
    # result has to be stationary: a sweep's changes below 1e-10 on p
    # coordinates, |S| <= 1, leave a gradient within p 1e-10 < 1e-7 of its bound
    X, lam0 = _data(2 * p + 3, p), 0.004 if p < 256 else 0.025
    try:
        ctx.set_tuning(dict(dense_block=b))
        r = _solve(ctx, X, lam0, precision="fp64", output_scale="standardized")
    finally:
        ctx.set_tuning(None)
    assert r.stats["max_working_set"] > 128
    S, B, sig = standardized_cov(X), r.B.cpu().numpy(), r.sigma.cpu().numpy()
    np.fill_diagonal(S, 1.0)
    R = S - S @ B
    assert np.abs(1.0 - (B * (S + R)).sum(0) - sig ** 2).max() <= 1e-7
    lam = lam0 * sig
    off = ~np.eye(p, dtype=bool)
    assert (np.abs(R) - lam)[off].max() <= 1e-7
    nz = off & (B != 0)
    assert np.abs(R - lam * np.sign(B))[nz].max() <= 1e-7
