"""Scaled lassos whose working sets pass 128 coordinates and together cover
(nearly) the whole design, so that they end in the dense tier with every
predictor in its rows: the responses of one call stay out of each other's
regressions."""
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


# the most responses for which 15/16 of p + m rows can be predictors is p / 15
@pytest.mark.parametrize("n,p,m", [(1000, 200, 1), (1000, 200, 2), (1000, 200, 8), (1000, 200, 13), (1000, 200, 14),
                                   (900, 160, 5), (1300, 260, 3)])
def test_responses_stay_apart_in_the_dense_tier(ctx, n, p, m):
    rng = np.random.default_rng(n + p + m)
    X = rng.standard_normal((n, p)) + 0.3 * rng.standard_normal((n, 1))
    # a common part, so that a response would explain the others
    Y = X @ rng.standard_normal((p, 1)) + 0.5 * rng.standard_normal((n, 1)) + 0.5 * rng.standard_normal((n, m))
    lam0 = 0.004
    Xg, Yg = torch.from_numpy(X).to("cuda:0"), torch.from_numpy(Y).to("cuda:0")
    beta, sig, _, st, stats = ctx.scaled_lasso(Xg, Yg, lam0, tol=1e-10, max_outer=200, max_sweeps=20000)
    assert st == 0 and stats["max_working_set"] > 128
    beta, sig = beta.cpu().numpy(), sig.cpu().numpy()
    Xs, _, c = oracle.standardize(X)
    for r in range(m):
        ys, _, cy = oracle.standardize(Y[:, r:r + 1])
        b, s, _, _, so = oracle.scaled_lasso(Xs, ys[:, 0], lam0, tol=1e-12)
        assert so == 0
        # 1e-6: the double form's bar; both sides stop at 1e-10 or below
        assert rel_err(beta[:, r], b * c / cy[0]) <= 1e-6
        assert abs(sig[r] - s / cy[0]) <= 1e-6 * s / cy[0]
        if r in (0, m - 1):  # the response on its own
            b1, s1, _, st1, _ = ctx.scaled_lasso(Xg, Yg[:, r].contiguous(), lam0, tol=1e-10, max_outer=200,
                                                 max_sweeps=20000)
            assert st1 == 0 and rel_err(b1.cpu().numpy(), beta[:, r]) <= 1e-6
            assert abs(float(s1) - sig[r]) <= 1e-6 * sig[r]
