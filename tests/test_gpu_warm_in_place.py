"""A capped solve resumed into its own outputs: the warm start is read before
the outputs are cleared, wherever their fill runs, so the resume does the work
and gives the results of one into other memory."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_15031_amd import spmesl
    c = spmesl.Context(0)
    yield c
    c.close()


# fills in the first kernel (up to 5 Mi elements), and beyond that beside the
# covariance kernel (double) or after the KKT pass (mixed); the data form
@pytest.mark.parametrize("share", ["result", "omega", "sigma0"])
@pytest.mark.parametrize("p,prec,data", [(2, "fp64", False), (300, "mixed", False), (300, "fp64", False),
                                         (300, "fp32", False), (2310, "fp64", False), (2310, "mixed", False),
                                         (120, "fp64", True)])
def test_resume_in_place(ctx, p, prec, data, share):
    rng = np.random.default_rng(p)
    e = rng.standard_normal((150, p + 4))
    X = torch.from_numpy(sum(e[:, i:i + p] for i in range(4))).to("cuda:0")
    kw = dict(precision=prec, data_form=data, tol=1e-8)
    lam0 = 0.2 if p < 1000 else 0.35
    capped = ctx.solve(X, lam0, max_outer=1, check=False, **kw)
    B0, s0 = capped.B.clone(), capped.sigma.clone()
    apart = ctx.solve(X, lam0, B0=B0, sigma0=s0, **kw)
    if share == "result":
        out = dict(B=B0, sigma=s0, Omega=capped.Omega)
    elif share == "omega":
        out = dict(B=capped.B, sigma=capped.sigma, Omega=B0)
    else:  # sigma0 within the cleared memory
        B = torch.empty(p, p, dtype=torch.float64, device="cuda:0")
        B.view(-1)[p * p - p:] = s0
        s0 = B.view(-1)[p * p - p:]
        out = dict(B=B, sigma=capped.sigma, Omega=capped.Omega)
    here = ctx.solve(X, lam0, B0=B0, sigma0=s0, out=out, **kw)
    for k in ("total_outer", "total_sweeps", "total_updates"):
        assert here.stats[k] == apart.stats[k], k
    for k in ("B", "sigma", "Omega"):
        assert torch.equal(getattr(here, k), getattr(apart, k)), k
    if p == 300:  # the start is used: less work than from beta = 0
        cold = ctx.solve(X, lam0, **kw)
        assert here.stats["total_updates"] < cold.stats["total_updates"]


# ... and with the placement set by hand
@pytest.mark.parametrize("split", [1, 2])
def test_resume_in_place_set_placement(ctx, split):
    rng = np.random.default_rng(7)
    e = rng.standard_normal((150, 304))
    X = torch.from_numpy(sum(e[:, i:i + 300] for i in range(4))).to("cuda:0")
    try:
        ctx.set_tuning(dict(fill_split=split))
        c = ctx.solve(X, 0.2, max_outer=1, check=False)
        B0, s0 = c.B.clone(), c.sigma.clone()
        apart = ctx.solve(X, 0.2, B0=B0, sigma0=s0)
        here = ctx.solve(X, 0.2, B0=B0, sigma0=s0, out=dict(B=B0, sigma=s0, Omega=c.Omega))
    finally:
        ctx.set_tuning(None)
    assert here.stats["total_updates"] == apart.stats["total_updates"]
    assert torch.equal(here.B, apart.B) and torch.equal(here.Omega, apart.Omega)
