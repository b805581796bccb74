"""Warm-started projections whose estimate has an empty support, of values so
large against the radius that adding it to one rounds away (r below half a
unit in the last place of max y).  No value is then above the start's bound
-lam_J = max y, nothing has a slope at the fallback's lambda_0 = -max y, and
the step from there must not lead to an infinite multiplier: x is finite, as
the multi-launch route's is, dense and sparse, waiting and queued."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

F64, F32 = torch.float64, torch.float32
BIG = {F32: 3.4028234663852886e38, F64: 1.7976931348623157e308}


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_15910_amd as cqk
    c = cqk.Context(0)
    yield c
    c.close()


def _data(case, n, dtype):
    g = np.random.default_rng(3)
    if case == "tiny_radius":
        return g.standard_normal(n), 1e-300
    if case == "large":
        return 1e30 * g.standard_normal(n), 1.0
    if case == "lowest":
        return np.full(n, -BIG[dtype]), 1.0
    # one value too large in the last block, ordinary ones in the others
    y = g.standard_normal(n)
    y[-1] = 1e30
    return y, 1.0


# one block, several, the last size of the one launch's, past it
@pytest.mark.parametrize("n", [1, 700, 70_001, 6_291_000, 12_582_913])
@pytest.mark.parametrize("case", ["tiny_radius", "large", "lowest", "one_large"])
@pytest.mark.parametrize("dtype", [F32, F64])
def test_empty_support(ctx, dtype, case, n):
    import paper_2603_15910_amd as cqk
    y, r = _data(case, n, dtype)
    t = torch.from_numpy(y).to("cuda", dtype)
    for l1 in (False, True):
        fn = ctx.project_l1 if l1 else ctx.project_simplex
        fs = ctx.project_l1_sparse if l1 else ctx.project_simplex_sparse
        for xbar in (torch.zeros_like(t), torch.full_like(t, float("nan"))):
            x, info = fn(t, r, xbar=xbar)
            _, _ = fn(t, r, xbar=xbar, out=(q := torch.full_like(t, 9.0)), sync=False, max_iter=30)
            i, v, _ = fs(t, r, xbar=xbar)
            s = torch.zeros_like(t)
            s[i] = v
            assert np.isfinite(info["lambda"])
            # x = (|y| + lambda)_+ : at most what rounding leaves of the radius
            big = float(t.abs().max())
            assert float(x.abs().max()) <= r + 2.0 * torch.finfo(dtype).eps * big
            assert torch.equal(x, q) and torch.equal(x, s)
            if l1:
                assert bool((x * t >= 0).all())
        assert cqk.cqk_set_team_wait(ctx.handle, 0) == 0
        x0, _ = fn(t, r, xbar=torch.zeros_like(t))
        assert cqk.cqk_set_team_wait(ctx.handle, 2_000_000) == 0
        if case != "one_large":   # there it may take the value's neighbours as zero or not
            assert torch.equal(x0, x)
