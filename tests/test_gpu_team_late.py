"""One-launch calls in which one block gives up at a chosen exchange, the last
one among them, after the rest of the team has its record: the call's outcome
is the multi-launch route's, waiting and queued, for the single solves, the
projections (dense and sparse) and the batched form in both directions.

The two routes add their sums in another order, so a multiplier may differ by
a few roundings of its terms; with O(1) data x is held to 1e-12 (FP64) and one
unit of the last place of values up to 8 (FP32: 5e-7), lambda to 1e-12."""
import numpy as np
import pytest

from paper_2603_15910_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

F64, F32 = torch.float64, torch.float32
WAIT = 20_000   # 0.2 ms: what the other blocks wait for the one that gave up


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_15910_amd as cqk
    c = cqk.Context(0)
    yield c
    c.close()


def _set(ctx, wait, block=0, exchange=0):
    import paper_2603_15910_amd as cqk
    assert cqk.cqk_set_team_wait(ctx.handle, wait) == 0
    assert cqk.cqk_set_team_late(ctx.handle, block, exchange) == 0


def _same(got, want, dtype):
    x, info = got
    x0, info0 = want
    tol = 1e-12 if dtype == F64 else 5e-7
    assert info["status"] == info0["status"] == 0
    assert info["n_free"] == info0["n_free"]
    assert abs(info["lambda"] - info0["lambda"]) <= 1e-12 * (1.0 + abs(info0["lambda"]))
    assert info["residual"] <= info0["residual"] + tol * max(1.0, info0["abs_bx"])
    assert float((x - x0).abs().max()) <= tol * max(1.0, float(x0.abs().max()))


def _every_exchange(ctx, call, want, dtype, block, launches, sync=True):
    """call() with the block late at exchange 1, 2, ...: as many as the launch
    has, which a waiting call tells by the number of its launches."""
    try:
        for k in range(1, 14):
            _set(ctx, WAIT, block, k)
            got = call()
            _same(got, want, dtype)
            if sync and got[1]["pass_launches"] == launches:
                break
        assert k > 3 and (not sync or got[1]["pass_launches"] == launches), k
    finally:
        _set(ctx, 2_000_000)


@pytest.mark.parametrize("sync", [True, False])
@pytest.mark.parametrize("block", [1, 255])
@pytest.mark.parametrize("l1", [False, True])
@pytest.mark.parametrize("dtype", [F32, F64])
def test_long_projection(ctx, dtype, l1, block, sync):
    """The launch behind the pass over y, every block of which writes x."""
    n = 12_600_001 if dtype == F32 else 6_300_001
    y = W.simplex_input(n, 4, "normal", np.float32 if dtype == F32 else np.float64)
    t = torch.from_numpy(y).cuda()
    fn = ctx.project_l1 if l1 else ctx.project_simplex
    _set(ctx, 0)
    want = fn(t, 1.0)

    def call():
        x, info = fn(t, 1.0, out=torch.full_like(t, 9.0), sync=sync, max_iter=30)
        if not sync:
            _, info = ctx.ctx_last_info()
        return x, info

    _every_exchange(ctx, call, want, dtype, block, 3, sync)


@pytest.mark.parametrize("sync", [True, False])
@pytest.mark.parametrize("dtype", [F32, F64])
def test_long_projection_stopped_early(ctx, dtype, sync):
    """max_iter = 1: the two routes end at different multipliers, both above
    lambda*.  Entries that the other blocks have written at the one launch's,
    the larger here, do not stay behind in the other route's x."""
    n = 12_600_001 if dtype == F32 else 6_300_001
    # one value far above the rest: the candidates of either start end far
    # from lambda*, the one launch's four further than the other's twelve
    y = np.random.default_rng(6).random(n)
    y[-1] = 3.0
    t = torch.from_numpy(y).to("cuda", dtype)
    kw = dict(max_iter=1, check=False)
    _set(ctx, WAIT)
    one = ctx.project_simplex(t, 100.0, **kw)
    _set(ctx, 0)
    want = ctx.project_simplex(t, 100.0, **kw)
    assert one[1]["status"] == want[1]["status"] == 3
    assert one[1]["n_free"] > want[1]["n_free"]
    try:
        for k in (1, 2, 3):   # the bound, the candidates, the evaluation
            _set(ctx, WAIT, 1, k)
            x, info = ctx.project_simplex(t, 100.0, out=torch.full_like(t, 9.0), sync=sync, **kw)
            if not sync:
                _, info = ctx.ctx_last_info()
            assert info["n_free"] == want[1]["n_free"]
            assert torch.equal(x, want[0])
    finally:
        _set(ctx, 2_000_000)


@pytest.mark.parametrize("sync", [True, False])
@pytest.mark.parametrize("dtype", [F32, F64])
def test_projection(ctx, dtype, sync):
    n = 300_001
    y = W.simplex_input(n, 4, "normal", np.float32 if dtype == F32 else np.float64)
    t = torch.from_numpy(y).cuda()
    _set(ctx, 0)
    want = ctx.project_simplex(t, 1.0)

    def call():
        x, info = ctx.project_simplex(t, 1.0, out=torch.full_like(t, 9.0), sync=sync, max_iter=30)
        if not sync:
            _, info = ctx.ctx_last_info()
        return x, info

    _every_exchange(ctx, call, want, dtype, 5, 1, sync)


def test_sparse_projection(ctx):
    n = 300_001
    t = torch.from_numpy(W.simplex_input(n, 4, "normal", np.float64)).cuda()
    _set(ctx, 0)
    want = ctx.project_simplex(t, 1.0)

    def call():
        i, v, info = ctx.project_simplex_sparse(t, 1.0)
        x = torch.zeros_like(t)
        x[i] = v
        assert i.numel() == info["n_free"] and bool((i[1:] > i[:-1]).all())
        return x, info

    _every_exchange(ctx, call, want, F64, 5, 1)


@pytest.mark.parametrize("sync", [True, False])
@pytest.mark.parametrize("n", [100_001, 4_400_003])
def test_solve(ctx, n, sync):
    inst = W.cqk_uniform(n, 8)
    t = [torch.from_numpy(inst[k]).cuda() for k in "dablu"]
    _set(ctx, 0)
    want = ctx.solve(*t, inst["r"])
    one = sync and n < 2_000_000   # longer inputs do not tell it in their launches

    def call():
        x, info = ctx.solve(*t, inst["r"], out=torch.full_like(t[0], 9.0), sync=sync, max_iter=20)
        if not sync:
            _, info = ctx.ctx_last_info()
        return x, info

    _every_exchange(ctx, call, want, F64, 3, 1, one)


@pytest.mark.parametrize("dtype", [F64, F32])
def test_batched(ctx, dtype):
    g = np.random.default_rng(5)
    lens = np.concatenate([[300_000, 70_001, 70_000, 20_011], g.integers(300, 9000, 60)])
    off = np.zeros(lens.size + 1, np.int64)
    np.cumsum(lens, out=off[1:])
    inst = W.cqk_uniform(int(off[-1]), 3, np.float64 if dtype == F64 else np.float32)
    t = [torch.from_numpy(inst[k]).to("cuda", dtype) for k in "dablu"]
    to = torch.from_numpy(off).cuda()
    mid = t[2].double() * (t[3].double() + t[4].double()) * 0.5
    r = torch.segment_reduce(mid, "sum", lengths=to[1:] - to[:-1])
    gr = torch.from_numpy(g.standard_normal(int(off[-1]))).to("cuda", dtype)
    tol = 1e-12 if dtype == F64 else 5e-7

    def run():
        lam = torch.full_like(r, 7.0)
        st = torch.full((r.numel(),), 9, dtype=torch.int32, device="cuda")
        x, info = ctx.solve_batched(*t, to, r, lambda_out=lam, status_out=st)
        grad_r = torch.full_like(r, 7.0)
        ga = ctx.solve_batched_backward(x, gr, t[0], t[2], t[3], t[4], to, grad_r=grad_r)
        assert not bool(st.any()) and info["status"] == 0
        return x, lam, ga, grad_r

    _set(ctx, 0)
    want = run()
    try:
        for block in (1, 130):
            for k in (1, 2, 3, 5, 8, 13):
                _set(ctx, WAIT, block, k)
                for a, b in zip(run(), want):
                    assert float((a - b).abs().max()) <= tol * 10 * max(1.0, float(b.abs().max()))
    finally:
        _set(ctx, 2_000_000)
