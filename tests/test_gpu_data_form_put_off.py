"""The data form on more columns than its full workspace slices have
workgroups for: groups whose V outgrows the smaller slices of the first launch
go to a second one, those beyond 1024 rows are refused, and neither disturbs
the groups beside them."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from tests.parity import rel_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_15031_amd import spmesl
    return spmesl


N, P, LAM = 3000, 4200, 0.07  # 263 groups; 256 workgroups of about 700 rows


def _data(per_column, columns):
    """Columns 0 .. columns - 1 each a sum of `per_column` of the others, no two
    of them sharing one while there are enough."""
    rng = np.random.default_rng(per_column)
    X = rng.standard_normal((N, P))
    rest = np.arange(columns, P)
    rng.shuffle(rest)
    for k in range(columns):
        pick = rest[(k * per_column + np.arange(per_column)) % rest.size]
        X[:, k] = X[:, pick].sum(1) * (0.9 / np.sqrt(per_column)) + 0.4 * rng.standard_normal(N)
    return X


@pytest.mark.parametrize("warm", [False, True])
def test_groups_put_off(sp, warm):
    # groups 0 .. 3: V of about 16 x 52 = 830 rows; the others a few dozen
    X = _data(52, 64)
    Xg = torch.from_numpy(X).to("cuda:0")
    ctx = sp.Context(0)
    try:
        ref = ctx.solve(Xg, LAM, tol=1e-9, precision="fp64")
        kw = dict(B0=ref.B, sigma0=ref.sigma) if warm else {}
        for _ in range(3):  # kernel by kernel, captured, replayed
            r = ctx.solve(Xg, LAM, tol=1e-9, precision="fp64", data_form=True, **kw)
            # 1e-6: the double forms' bar
            for k in ("B", "sigma", "Omega"):
                assert rel_err(getattr(r, k).cpu().numpy(), getattr(ref, k).cpu().numpy()) <= 1e-6, k
        cols = [0, 17, 40, 63, 64, 2000, 4199]
        nnz = (ref.B != 0).sum(0).cpu().numpy()
        assert nnz[:64].min() >= 45  # the four groups' V exceed the smaller slices
        orc = oracle.spmesl_columns(X, LAM, cols, tol=1e-11)
        want = ctx.solve(Xg, LAM, tol=1e-9, precision="fp64", data_form=True, output_scale="standardized")
        assert rel_err(want.B[:, cols].cpu().numpy(), orc["B"]) <= 1e-6
        assert rel_err(want.sigma[cols].cpu().numpy(), orc["sigma"]) <= 1e-6
    finally:
        ctx.close()


def test_refused_beyond_the_full_slices(sp):
    X = torch.from_numpy(_data(75, 32)).to("cuda:0")  # V of 1200 rows
    ctx = sp.Context(0)
    try:
        with pytest.raises(sp.SpmeslError) as e:
            ctx.solve(X, 0.06, tol=1e-9, precision="fp64", data_form=True)
        assert e.value.code == sp.EWORKSET
        # the context still solves
        Y = X[:, 64:164].contiguous()
        a = ctx.solve(Y, LAM, tol=1e-9, precision="fp64", data_form=True)
        b = ctx.solve(Y, LAM, tol=1e-9, precision="fp64")
        assert rel_err(a.B.cpu().numpy(), b.B.cpu().numpy()) <= 1e-6
    finally:
        ctx.close()
