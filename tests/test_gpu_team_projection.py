"""The one-launch simplex and l1 projections (values kept in the compute units'
registers): sizes around each step of values per thread, dense and sparse
output, cold and warm starts, ties and full supports (a wave's list
overflows), bad values, short room, a block that gives up, queued calls and
graph replays.  Results are held to the bars of tests/parity.py against the
oracle; the multi-launch route (team wait 0) must agree on the support."""
import numpy as np
import pytest

from oracle import cqk_oracle as O
from paper_2603_15910_amd import workloads as W
from tests.parity import check_simplex

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

F64, F32 = torch.float64, torch.float32
# blocks of 4096 FP32 / 2048 FP64 values, up to 256 of them; then blocks of
# 16384 / 8192, 256 of them 4194304 / 2097152, and 2 and 3 times that
SIZES = {F32: [1, 2, 3, 5, 255, 4095, 4096, 4097, 16385, 4_194_303, 4_194_305, 8_388_609,
               12_582_911, 12_582_913],
         F64: [1, 2, 3, 5, 255, 2047, 2048, 2049, 8193, 2_097_151, 2_097_153, 4_194_305,
               6_291_455, 6_291_457]}


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_15910_amd as cqk
    c = cqk.Context(0)
    yield c
    c.close()


def _wait(ctx, ticks):
    import paper_2603_15910_amd as cqk
    assert cqk.cqk_set_team_wait(ctx.handle, ticks) == 0


def _np(dtype):
    return np.float64 if dtype == F64 else np.float32


def _oracle(y, r, l1):
    y = y.astype(np.float64)
    res = O.project_l1(y, r) if l1 else O.project_simplex(y, r)
    return res[0], res[1]


def _check(x, y, r, l1, dtype):
    xr, lam = _oracle(y, r, l1)
    check_simplex(x, y, xr, lam, r, 1e-10 if dtype == F64 else 1e-5, l1=l1)


def _both(ctx, t, r, l1, dtype, **kw):
    """Dense and sparse results of the one-launch route, equal to each other."""
    dense = ctx.project_l1 if l1 else ctx.project_simplex
    sparse = ctx.project_l1_sparse if l1 else ctx.project_simplex_sparse
    x, info = dense(t, r, out=torch.full_like(t, 9.0), **kw)
    i, v, _ = sparse(t, r, **kw)
    y = torch.zeros_like(t)
    y[i] = v
    assert bool((i[1:] > i[:-1]).all())
    assert torch.equal(x, y)
    assert int(i.numel()) == info["n_free"]
    return x, info


@pytest.mark.parametrize("l1", [False, True])
@pytest.mark.parametrize("dtype", [F32, F64])
@pytest.mark.parametrize("which", range(14))
def test_sizes(ctx, dtype, which, l1):
    n = SIZES[dtype][which]
    y = W.simplex_input(n, 3 + which, "normal" if which % 2 else "uniform", _np(dtype))
    t = torch.from_numpy(y).cuda()
    x, info = _both(ctx, t, 1.0, l1, dtype)
    last = SIZES[dtype][-1]
    assert (info["pass_launches"] == 1) == (n < last)
    _check(x.cpu().numpy(), y, 1.0, l1, dtype)


@pytest.mark.parametrize("past", [0, 1])
@pytest.mark.parametrize("dtype", [F32, F64])
def test_end_of_the_first_step(ctx, dtype, past):
    """256 blocks of 4096 FP32 / 2048 FP64 values, and the next step."""
    n = (1_048_576 if dtype == F32 else 524_288) + past
    y = W.simplex_input(n, 21, "normal", _np(dtype))
    t = torch.from_numpy(y).cuda()
    for l1 in (False, True):
        x, info = _both(ctx, t, 1.0, l1, dtype)
        assert info["pass_launches"] == 1
        _check(x.cpu().numpy(), y, 1.0, l1, dtype)


@pytest.mark.parametrize("l1", [False, True])
@pytest.mark.parametrize("dtype", [F32, F64])
@pytest.mark.parametrize("n", [700, 50_001])
def test_warm_starts(ctx, dtype, n, l1):
    y = W.simplex_input(n, 9, "normal", _np(dtype))
    t = torch.from_numpy(y).cuda()
    fn = ctx.project_l1 if l1 else ctx.project_simplex
    cold, info0 = fn(t, 1.0)
    y2 = W.perturbed(y, 4)
    t2 = torch.from_numpy(y2).cuda()
    for xbar in (cold, torch.zeros_like(cold), torch.ones_like(cold), -cold):
        x, info = _both(ctx, t2, 1.0, l1, dtype, xbar=xbar)
        assert info["pass_launches"] == 1
        _check(x.cpu().numpy(), y2, 1.0, l1, dtype)
    # the exact solution as the estimate starts at lam*
    x, info = fn(t, 1.0, xbar=cold)
    assert torch.equal(x, cold)
    assert abs(info["lambda0"] - info0["lambda"]) <= 1e-6 * max(1.0, abs(info0["lambda"]))


@pytest.mark.parametrize("dtype", [F32, F64])
@pytest.mark.parametrize("case", ["ties", "all_free", "inside", "large_r", "two_values", "tiny",
                                  "zeros", "negative", "one_big"])
def test_shapes_of_data(ctx, dtype, case):
    n = 40_003
    g = np.random.default_rng(7)
    y, r = {"ties": (np.full(n, 0.25), 1.0),
            "all_free": (1.0 + 1e-3 * g.standard_normal(n), 1000.0),
            "inside": (1e-6 * g.standard_normal(n), 1.0),
            "large_r": (g.standard_normal(n), 1e6),
            "two_values": (np.where(g.random(n) < 0.5, 1.0, 2.0), 5.0),
            "tiny": (1e-30 * g.standard_normal(n), 1e-31),
            "zeros": (np.zeros(n), 2.0),
            "negative": (-1.0 - g.random(n), 0.5),
            "one_big": (np.concatenate([g.standard_normal(n - 1), [1e6]]), 1.0)}[case]
    y = y.astype(_np(dtype))
    t = torch.from_numpy(y).cuda()
    for l1 in (False, True):
        x, info = _both(ctx, t, r, l1, dtype)
        assert info["pass_launches"] == 1
        _check(x.cpu().numpy(), y, r, l1, dtype)


@pytest.mark.parametrize("dtype", [F32, F64])
@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
def test_bad_values(ctx, dtype, bad):
    for n in (10, 60_000):
        y = W.simplex_input(n, 2, "normal", _np(dtype))
        y[n - 1] = bad
        t = torch.from_numpy(y).cuda()
        for fn in (ctx.project_simplex, ctx.project_l1):
            _, info = fn(t, 1.0, check=False)
            assert info["status"] == 2
        _, _, info = ctx.project_l1_sparse(t, 1.0, check=False)
        assert info["status"] == 2


def test_short_room(ctx):
    y = W.simplex_input(50_000, 3, "uniform", np.float32)
    t = torch.from_numpy(y).cuda()
    i0, v0, _ = ctx.project_simplex_sparse(t, 1.0)
    out = (torch.full((5,), -3, dtype=torch.int64, device="cuda"),
           torch.full((5,), -3.0, device="cuda"))
    import paper_2603_15910_amd as cqk
    st, nnz = cqk.cqk_project_simplex_sparse_f32(ctx.handle, t.numel(), t.data_ptr(), None, 1.0, 5,
                                                 out[0].data_ptr(), out[1].data_ptr())
    assert st == cqk.CQK_BUFFER_TOO_SMALL and nnz == i0.numel() > 5
    assert bool((out[0] == -3).all()) and bool((out[1] == -3.0).all())
    i, v, _ = ctx.project_simplex_sparse(t, 1.0, cap=5)   # the binding makes room
    assert torch.equal(i, i0) and torch.equal(v, v0)


def test_a_block_that_gives_up(ctx):
    y = W.simplex_input(300_000, 3, "normal", np.float64)
    t = torch.from_numpy(y).cuda()
    for sync in (True, False):
        _wait(ctx, 1)
        x, info = ctx.project_simplex(t, 1.0, out=torch.full_like(t, 9.0), sync=sync, max_iter=30)
        if not sync:
            st, info = ctx.ctx_last_info()
            assert st == 0
        i, v, _ = ctx.project_simplex_sparse(t, 1.0)
        _wait(ctx, 2_000_000)
        assert info["pass_launches"] > 1
        _check(x.cpu().numpy(), y, 1.0, False, F64)
        assert torch.equal(x[i], v) and int((x != 0).sum()) == i.numel()
        x, info = ctx.project_simplex(t, 1.0)
        assert info["pass_launches"] == 1
        _check(x.cpu().numpy(), y, 1.0, False, F64)


@pytest.mark.parametrize("l1", [False, True])
@pytest.mark.parametrize("n", [3000, 200_001])
def test_queued_and_replayed(ctx, n, l1):
    ctx.reserve(n)
    ys = [W.simplex_input(n, s, "normal", np.float32) for s in (1, 2, 3)]
    t = torch.from_numpy(ys[0]).cuda()
    x = torch.empty_like(t)
    fn = ctx.project_l1 if l1 else ctx.project_simplex
    first, info1 = fn(t, 1.0)
    again, info = fn(t, 1.0, out=torch.full_like(t, 5.0), sync=False, max_iter=30)
    st, info2 = ctx.ctx_last_info()
    assert st == 0 and torch.equal(first, again)
    for k in ("lambda", "lambda0", "iterations", "stop_reason", "n_free", "residual",
              "n_after_init"):
        assert info1[k] == info2[k], k
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        with torch.cuda.graph(graph, stream=s):
            fn(t, 1.0, out=x, max_iter=30)
    for y in ys + ys:
        t.copy_(torch.from_numpy(y))
        x.fill_(3.0)
        graph.replay()
        torch.cuda.synchronize()
        eager, _ = fn(t, 1.0)
        assert torch.equal(x, eager)


# ---- past those sizes: one launch behind the pass over y ----

LONG = {F32: 12_582_913, F64: 6_291_457}


def _long_data(case, n, g):
    if case == "few":
        return g.standard_normal(n), 1.0
    if case == "clustered":       # neighbours: a few waves hold every survivor
        y = g.standard_normal(n)
        y[1000:201_000] = 50.0 + 1e-3 * g.standard_normal(200_000)
        return y, 10_000.0
    if case == "spread":          # lists longer than LDS in every wave
        y = g.uniform(0.0, 1.0, n)
        return y, 0.45 * n * 0.45
    if case == "all_free":        # more survivors than the launch takes
        return 1.0 + 1e-3 * g.standard_normal(n), float(n)
    if case == "ties":
        return np.full(n, 0.25), 1.0
    if case == "inside":
        return 1e-9 * g.standard_normal(n), 1.0
    if case == "zeros":
        return np.zeros(n), 2.0
    return np.concatenate([g.standard_normal(n - 1), [1e6]]), 1.0   # one_big


@pytest.mark.parametrize("dtype", [F32, F64])
@pytest.mark.parametrize("case", ["few", "clustered", "spread", "all_free", "ties", "inside",
                                  "zeros", "one_big"])
def test_long_inputs(ctx, dtype, case):
    n = LONG[dtype]
    y, r = _long_data(case, n, np.random.default_rng(17))
    y = y.astype(_np(dtype))
    t = torch.from_numpy(y).cuda()
    for l1 in (False, True):
        x, info = _both(ctx, t, r, l1, dtype)
        _wait(ctx, 0)
        x0, info0 = (ctx.project_l1 if l1 else ctx.project_simplex)(t, r)
        _wait(ctx, 2_000_000)
        if case in ("few", "clustered", "one_big"):
            assert info["pass_launches"] == 3 < info0["pass_launches"]
        assert abs(info["lambda"] - info0["lambda"]) <= 1e-13 * (1.0 + abs(info0["lambda"]))
        _check(x.cpu().numpy(), y, r, l1, dtype)


@pytest.mark.parametrize("dtype", [F32, F64])
def test_long_warm_starts(ctx, dtype):
    n = LONG[dtype]
    y = W.simplex_input(n, 9, "normal", _np(dtype))
    t = torch.from_numpy(y).cuda()
    for l1 in (False, True):
        fn = ctx.project_l1 if l1 else ctx.project_simplex
        cold, _ = fn(t, 1.0)
        for xbar in (cold, torch.zeros_like(cold), torch.ones_like(cold)):
            x, info = _both(ctx, t, 1.0, l1, dtype, xbar=xbar)
            assert info["pass_launches"] == 3
            _check(x.cpu().numpy(), y, 1.0, l1, dtype)


def test_long_bad_values_and_room(ctx):
    n = LONG[F32]
    y = W.simplex_input(n, 2, "uniform", np.float32)
    t = torch.from_numpy(y).cuda()
    i0, v0, _ = ctx.project_simplex_sparse(t, 1.0)
    i, v, _ = ctx.project_simplex_sparse(t, 1.0, cap=5)
    assert torch.equal(i, i0) and torch.equal(v, v0)
    for bad in (np.nan, np.inf, -np.inf):
        t[n - 3] = float(bad)
        _, info = ctx.project_simplex(t, 1.0, check=False)
        assert info["status"] == 2
        _, _, info = ctx.project_l1_sparse(t, 1.0, check=False)
        assert info["status"] == 2


def test_long_give_up_queued_and_replayed(ctx):
    n = LONG[F64]
    ctx.reserve(n)
    y = W.simplex_input(n, 5, "normal", np.float64)
    t = torch.from_numpy(y).cuda()
    first, info1 = ctx.project_simplex(t, 1.0)
    for sync in (True, False):
        for ticks in (1, 0, 2_000_000):
            _wait(ctx, ticks)
            x, info = ctx.project_simplex(t, 1.0, out=torch.full_like(t, 9.0), sync=sync,
                                          max_iter=30)
            if not sync:
                st, info = ctx.ctx_last_info()
                assert st == 0
            _check(x.cpu().numpy(), y, 1.0, False, F64)
            i, v, _ = ctx.project_simplex_sparse(t, 1.0)
            assert torch.equal(i, torch.nonzero(first)[:, 0])
            if ticks == 2_000_000:
                assert torch.equal(x, first)
                for k in ("lambda", "lambda0", "iterations", "stop_reason", "n_free", "residual"):
                    assert info[k] == info1[k], k
    x = torch.empty_like(t)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        with torch.cuda.graph(graph, stream=s):
            ctx.project_simplex(t, 1.0, out=x, max_iter=20)
    for seed in (6, 7, 5):
        t.copy_(torch.from_numpy(W.simplex_input(n, seed, "normal", np.float64)))
        x.fill_(3.0)
        graph.replay()
        torch.cuda.synchronize()
        eager, _ = ctx.project_simplex(t, 1.0)
        assert torch.equal(x, eager)
