"""The mixed form's double dense stage with more samples than its LDS holds
residuals of: they then lie in the memory of the covariance's operands.  By
itself, after a smaller solve in the same workspace, in a batch and in the
no-allocation entry point's array."""
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


def _data(n, p):
    rng = np.random.default_rng(n + p)
    return rng.standard_normal((n, p)) + 0.4 * rng.standard_normal((n, 1))


# n around the 768 samples of LDS, a multiple of 16 and not, and beyond the
# 1638 of the fused standardisation
@pytest.mark.parametrize("n", [768, 769, 800, 1701])
def test_mixed_dense_stage(ctx, n):
    p, lam0 = 170, 0.01
    X = _data(n, p)
    Xg = torch.from_numpy(X).to("cuda:0")
    ref = oracle.spmesl(X, lam0, tol=1e-11, original_scale=True)
    kw = dict(tol=1e-8, precision="mixed")
    ctx.solve(Xg[:, :40].contiguous(), 0.3, **kw)
    one = ctx.solve(Xg, lam0, max_outer=400, max_sweeps=20000, **kw)
    assert one.stats["max_working_set"] > 128 and one.stats["columns_noconv"] == 0
    two = ctx.solve_batch([Xg, Xg], lam0, **kw)
    st = torch.full((1,), 99, dtype=torch.int32, device="cuda:0")
    out = {k: torch.full_like(getattr(one, k), 5.0) for k in ("B", "sigma", "Omega")}
    na = ctx.solve_noalloc(Xg, lam0, st, out, **kw)
    torch.cuda.synchronize()
    assert int(st.item()) == 0
    for r in (one, two[0], two[1], na):
        for k in ("B", "sigma", "Omega"):  # the mixed form's bar
            assert rel_err(getattr(r, k).cpu().numpy(), ref[k]) <= 1e-4, k


def test_noalloc_many_samples(ctx):
    # a tall problem near the edge of the array
    n, p, lam0 = 441336, 2, 0.02
    rng = np.random.default_rng(3)
    X = rng.standard_normal((n, p))
    X[:, 1] += 0.3 * X[:, 0]
    st = torch.full((1,), 99, dtype=torch.int32, device="cuda:0")
    out = dict(B=torch.empty(p, p, dtype=torch.float64, device="cuda:0"),
               sigma=torch.empty(p, dtype=torch.float64, device="cuda:0"),
               Omega=torch.empty(p, p, dtype=torch.float64, device="cuda:0"))
    ctx.solve_noalloc(torch.from_numpy(X).to("cuda:0"), lam0, st, out, tol=1e-8, precision="mixed")
    torch.cuda.synchronize()
    assert int(st.item()) == 0
    ref = oracle.spmesl(X, lam0, tol=1e-12, original_scale=True)
    for k in ("B", "sigma", "Omega"):
        assert rel_err(out[k].cpu().numpy(), ref[k]) <= 1e-4, k
