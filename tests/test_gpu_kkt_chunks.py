"""The row-tiled KKT pass where p takes several column chunks (beyond 3072 in
double, 5120 in float): p not a multiple of the 64-column groups, supports on
either side of the 8 entries held in registers, against the form that takes
its gradients from the data."""
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


# 1e-6 relative, the double forms' bar (both stop at 1e-10)
@pytest.mark.parametrize("prec,p", [("fp64", 3072), ("fp64", 3073), ("fp64", 6209), ("mixed", 5120),
                                    ("mixed", 5121), ("mixed", 10305)])
def test_kkt_chunks(ctx, prec, p):
    rng = np.random.default_rng(p)
    n = 600
    X = rng.standard_normal((n, p))
    X[:, 1:] += 0.7 * X[:, :-1]
    for k, m in ((3, 7), (70, 9), (p // 2, 12), (p - 1, 20)):
        X[:, k] = X[:, 100:100 + 5 * m:5].sum(1) + 0.3 * rng.standard_normal(n)
    lam0 = 0.18
    Xg = torch.from_numpy(X).to("cuda:0")
    a = ctx.solve(Xg, lam0, tol=1e-10, precision=prec, output_scale="standardized", want=("B", "sigma"))
    b = ctx.solve(Xg, lam0, tol=1e-10, precision="fp64", output_scale="standardized", want=("B", "sigma"),
                  data_form=True)
    assert int((a.B != 0).sum(0).max()) > 8
    for x, y in ((a.B, b.B), (a.sigma, b.sigma)):
        assert float((x - y).norm() / y.norm()) <= 1e-6
