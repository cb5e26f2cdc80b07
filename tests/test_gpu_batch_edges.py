"""A batch's shared launches at their edges: data sets that take each width of
the fused standardisation and none, one column block and many, outputs left
out and only 8-byte aligned; bit for bit the single solves."""
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


@pytest.mark.parametrize("prec", ["mixed", "fp64", "fp32"])
def test_batch_edges(ctx, prec):
    # strips of 8 variables fit up to n = 910, of 4 up to 1638
    sizes = [(910, 9), (911, 33), (40, 2), (1638, 5), (1639, 17), (64, 301)]
    Xs, outs, singles = [], [], []
    for i, (n, p) in enumerate(sizes):
        rng = np.random.default_rng(n + p)
        X = torch.from_numpy(rng.standard_normal((n, p)) + 0.5 * rng.standard_normal((n, 1))).to("cuda:0")
        Xs.append(X)
        buf = torch.full((2 * p * p + 3,), 7.0, dtype=torch.float64, device="cuda:0")
        o = dict(B=buf[1:1 + p * p].view(p, p), Omega=buf[2 + p * p:2 + 2 * p * p].view(p, p),
                 sigma=torch.empty(p, dtype=torch.float64, device="cuda:0"), buf=buf)
        if i == 1:
            o["B"] = None
        if i == 2:
            o["Omega"] = None
        outs.append(o)
        singles.append(ctx.solve(X, 0.2, tol=1e-8, precision=prec, eager=True))
    for _ in range(3):  # kernel by kernel, captured, replayed
        for o in outs:
            o["buf"].fill_(7.0)
        res = ctx.solve_batch(Xs, 0.2, tol=1e-8, precision=prec, outs=outs)
        for (n, p), r, o, one in zip(sizes, res, outs, singles):
            assert r.status == 0
            assert torch.equal(o["sigma"], one.sigma)
            for k in ("B", "Omega"):
                if o[k] is not None:
                    assert torch.equal(o[k], getattr(one, k)), (k, n, p)
            b = o["buf"]  # nothing written beside the outputs
            keep = [0, 1 + p * p, 2 + 2 * p * p]
            assert bool((b[keep] == 7.0).all())


@pytest.mark.parametrize("p", [2, 33, 600])
def test_outputs_of_a_small_solve(ctx, p):
    # cleared by the solve's first kernel: 8-byte aligned, nothing beside them
    rng = np.random.default_rng(p)
    X = torch.from_numpy(rng.standard_normal((80, p)) + 0.5 * rng.standard_normal((80, 1))).to("cuda:0")
    ref = ctx.solve(X, 0.3, tol=1e-8, precision="mixed")
    for skip in (None, "B", "Omega"):
        buf = torch.full((2 * p * p + 3,), 7.0, dtype=torch.float64, device="cuda:0")
        out = dict(B=buf[1:1 + p * p].view(p, p), Omega=buf[2 + p * p:2 + 2 * p * p].view(p, p))
        want = [k for k in ("B", "Omega") if k != skip]
        for k in want:
            buf.fill_(7.0)
            ctx.solve(X, 0.3, tol=1e-8, precision="mixed", out={q: out[q] for q in want}, want=tuple(want))
        for k in want:
            assert torch.equal(out[k], getattr(ref, k))
        assert bool((buf[[0, 1 + p * p, 2 + 2 * p * p]] == 7.0).all())


def test_output_in_the_inputs_memory(ctx):
    # an output that overlaps X is cleared only once X has been read
    rng = np.random.default_rng(5)
    n = p = 70
    X = torch.from_numpy(rng.standard_normal((n, p))).to("cuda:0")
    ref = ctx.solve(X, 0.4, tol=1e-8, precision="mixed")
    Xc = X.clone()
    r = ctx.solve(Xc, 0.4, tol=1e-8, precision="mixed", out=dict(B=Xc, sigma=ref.sigma.clone()), want=("B", "sigma"))
    assert torch.equal(r.B, ref.B) and torch.equal(r.sigma, ref.sigma)
