"""The mixed form's covariance kernels at the edges of their tiles.

n and p around the 16-variable operand blocks, the 64 x 64 and 256 x 256
tiles and the padding of the samples to 64, against the covariance in double;
one size on either side of the rule that picks the tile edge."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from tests.parity import standardized_cov

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_15031_amd import spmesl
    c = spmesl.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("n,p", [(2, 2), (63, 15), (64, 16), (65, 17), (129, 65), (31, 255), (200, 321),
                                 (96, 4096), (70, 4351), (33, 4609)])
def test_covariance_mixed_tile_edges(ctx, n, p):
    rng = np.random.default_rng(n + 7 * p)
    X = rng.standard_normal((n, p)) + 0.5 * rng.standard_normal((n, 1))
    Xg = torch.from_numpy(X).to("cuda:0")
    S, _, _ = ctx.covariance(Xg, "mixed")
    if p <= 400:
        ref = standardized_cov(X)
        np.fill_diagonal(ref, 1.0)
        err = np.abs(S.cpu().numpy().astype(np.float64) - ref).max()
    else:
        Z = Xg - Xg.mean(0)
        Z = Z / torch.sqrt((Z * Z).mean(0))
        ref = (Z.T @ Z) / n
        ref.fill_diagonal_(1.0)
        err = float((S.double() - ref).abs().max())
    # the bf16 split's per-entry bound plus float accumulation over n terms
    assert err <= 3 * 2.0 ** -16 + (n + 2) * 2.0 ** -24, err
    assert bool(torch.equal(S, S.T))


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("n", [2, 5, 96, 101, 230])
def test_covariance_same_bits_for_every_tile_edge(ctx, prec, n):
    """The first variables' block of S does not depend on the tile edge that
    the number of variables picks (32, 64, 128), and is the covariance."""
    rng = np.random.default_rng(n)
    full = 8200 if prec == "fp64" else 5100
    Xg = torch.from_numpy(rng.standard_normal((n, full)) + 0.5 * rng.standard_normal((n, 1))).to("cuda:0")
    ref = None
    for p in (33, 95, 705, 1001, full):
        S, _, _ = ctx.covariance(Xg[:, :p].contiguous(), prec)
        assert bool(torch.equal(S, S.T))
        m = min(p, 300)
        Z = Xg[:, :m] - Xg[:, :m].mean(0)
        Z = Z / torch.sqrt((Z * Z).mean(0))
        want = (Z.T @ Z) / n
        want.fill_diagonal_(1.0)
        # double: rounding of n products; float: that in single, and of the inputs
        tol = 1e-13 if prec == "fp64" else (n + 2) * 2.0 ** -24 + 2 * 2.0 ** -24
        assert float((S[:m, :m].double() - want).abs().max()) <= tol
        if ref is None:
            ref = S[:33, :33].clone()
        assert bool(torch.equal(S[:33, :33], ref)), p
