"""l1 projections of a y inside the ball: x = y and the outcome says so in the
same words on every route (lambda = lambda_0 = 0, no iteration, the trivial
stop), dense and sparse, cold and warm, waiting and queued."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

F64, F32 = torch.float64, torch.float32


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_15910_amd as cqk
    c = cqk.Context(0)
    yield c
    c.close()


def _says_inside(info, n, y):
    assert info["status"] == 0 and info["stop_reason"] == 5 and info["iterations"] == 0
    assert info["lambda"] == 0.0 and info["lambda0"] == 0.0
    assert info["n_free"] == int((y != 0).sum())
    assert abs(info["abs_bx"] - float(y.abs().double().sum())) <= 1e-12 * max(1.0, info["abs_bx"])
    assert info["residual"] <= 1e-12 * max(1.0, info["abs_bx"])


# one block, several, the last sizes of the one launch, past them
@pytest.mark.parametrize("n", [1, 700, 70_001, 6_291_457, 12_582_913])
@pytest.mark.parametrize("dtype", [F32, F64])
def test_inside(ctx, dtype, n):
    import paper_2603_15910_amd as cqk
    y = torch.from_numpy(np.random.default_rng(n).standard_normal(n)).to("cuda", dtype)
    y[n // 2] = 0.0
    r = 1.01 * float(y.abs().double().sum()) + 1.0
    for wait in (30_000, 0):
        assert cqk.cqk_set_team_wait(ctx.handle, wait) == 0
        for kw in ({}, dict(xbar=torch.ones_like(y))):
            x, info = ctx.project_l1(y, r, out=torch.full_like(y, 9.0), **kw)
            assert torch.equal(x, y)
            _says_inside(info, n, y)
            x, _ = ctx.project_l1(y, r, out=torch.full_like(y, 9.0), sync=False, max_iter=20, **kw)
            st, info = ctx.ctx_last_info()
            assert st == 0 and torch.equal(x, y)
            _says_inside(info, n, y)
            i, v, info = ctx.project_l1_sparse(y, r, cap=n, **kw)
            assert torch.equal(i, torch.nonzero(y)[:, 0]) and torch.equal(v, y[i])
            _says_inside(info, n, y)
    assert cqk.cqk_set_team_wait(ctx.handle, 30_000) == 0


@pytest.mark.parametrize("n", [12_582_913, 12_599_999])
@pytest.mark.parametrize("dtype", [F32, F64])
def test_long_inside_in_three_launches(ctx, dtype, n):
    """The sample, the pass over y and the launch behind it, which makes the
    copy; the end of y that is no whole vector, and y and x at any element."""
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    for off in (0, 1, 3):
        y = torch.randn(n + off, device="cuda", dtype=dtype, generator=g)[off:]
        out = torch.full((n + 2 * off,), 9.0, device="cuda", dtype=dtype)
        x, info = ctx.project_l1(y, 2.0 * n, out=out[off:off + n])
        assert torch.equal(x, y) and info["pass_launches"] == 3
        assert bool((out[:off] == 9.0).all()) and bool((out[off + n:] == 9.0).all())
        _says_inside(info, n, y)
