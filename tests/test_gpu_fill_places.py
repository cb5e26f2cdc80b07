"""Where the outputs are cleared: batches between the totals of the first
kernel and of the large batches' rule (after the KKT pass in float and mixed,
beside the covariance tiles in double) and beyond the latter, with no shapes
set and with others than the placement set; outputs in the memory of X."""
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


def _x(n, p):
    rng = np.random.default_rng(n + p)
    return torch.from_numpy(rng.standard_normal((n, p)) + 0.3 * rng.standard_normal((n, 1))).to("cuda:0")


# totals of 5.4, 6.3 and 36 Mi elements
@pytest.mark.parametrize("prec", ["mixed", "fp32", "fp64"])
@pytest.mark.parametrize("sizes", [[(60, 2300), (50, 600)], [(70, 1801), (40, 1800), (90, 333)], [(50, 4301)] * 2],
                         ids=["5.4Mi", "6.3Mi", "36Mi"])
def test_batch_totals(ctx, prec, sizes):
    Xs = [_x(n + i, p) for i, (n, p) in enumerate(sizes)]
    lam = [float(np.sqrt(2 * np.log(p) / n)) for n, p in sizes]
    singles = [ctx.solve(X, v, tol=1e-8, precision=prec, eager=True) for X, v in zip(Xs, lam)]
    for tuning in (None, dict(dense_block=32)):
        outs = [dict(B=torch.empty_like(s.B), Omega=torch.empty_like(s.Omega), sigma=torch.empty_like(s.sigma))
                for s in singles]
        try:
            ctx.set_tuning(tuning)
            for _ in range(3):  # kernel by kernel, captured, replayed
                for o in outs:
                    o["B"].fill_(7.0)
                    o["Omega"].fill_(7.0)
                res = ctx.solve_batch(Xs, lam, tol=1e-8, precision=prec, outs=outs)
                for r, o, one in zip(res, outs, singles):
                    assert r.status == 0
                    for k in ("B", "sigma", "Omega"):
                        assert torch.equal(o[k], getattr(one, k)), k
        finally:
            ctx.set_tuning(None)


@pytest.mark.parametrize("prec,data", [("mixed", False), ("fp32", False), ("fp64", False), ("fp64", True)])
@pytest.mark.parametrize("name", ["B", "Omega"])
@pytest.mark.parametrize("at", [0, 1, 69 * 70])
def test_output_over_the_input(ctx, prec, data, name, at):
    # X begins at the output's first, second or last row's first element
    n, p = 70, 70
    X = _x(n, p)
    kw = dict(tol=1e-8, precision=prec, data_form=data)
    ref = ctx.solve(X, 0.4, **kw)
    for eager in (True, False):
        buf = torch.full((n * p + at,), 7.0, dtype=torch.float64, device="cuda:0")
        Xc = buf[at:].view(n, p)
        Xc.copy_(X)
        r = ctx.solve(Xc, 0.4, out={name: buf[:p * p].view(p, p)}, want=(name, "sigma"), eager=eager, **kw)
        assert torch.equal(r.sigma, ref.sigma) and torch.equal(getattr(r, name), getattr(ref, name))
