"""Which workgroup rows of the batched general CQK teams of blocks hold and
which are streamed: numbers of rows and lengths on both sides of each limit,
forward and backward, and calls with rows of both kinds and rows past the
longest team's.  Results are the streaming route's (team wait 0) to the
rounding of sums added in another order: with O(1) data 1e-12 (FP64), a unit
in the last place of values up to 8 (FP32: 5e-7), ten times that for the VJP,
whose terms are divided once more.  A call of few short rows is not slower for
the teams' launch."""
import time

import numpy as np
import pytest

from paper_2603_15910_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

F64, F32 = torch.float64, torch.float32
DEFAULT = 30_000


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


def _problem(lens, dtype, seed=5):
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    inst = W.cqk_uniform(int(off[-1]), seed, np.float64 if dtype == F64 else np.float32)
    t = [torch.from_numpy(inst[k]).to("cuda", dtype) for k in "dablu"]
    to = torch.from_numpy(off).cuda()
    mid = t[2].double() * (t[3].double() + t[4].double()) * 0.5
    r = torch.segment_reduce(mid, "sum", lengths=to[1:] - to[:-1], unsafe=True)
    g = torch.from_numpy(np.random.default_rng(seed).standard_normal(int(off[-1])))
    return t, to, r, g.to("cuda", dtype)


def _both(ctx, problem, **kw):
    t, to, r, g = problem
    lam = torch.full_like(r, 7.0)
    st = torch.full((r.numel(),), 9, dtype=torch.int32, device="cuda")
    x, _ = ctx.solve_batched(*t, to, r, lambda_out=lam, status_out=st, **kw)
    gr = torch.full_like(r, 7.0)
    ga = ctx.solve_batched_backward(x, g, t[0], t[2], t[3], t[4], to, grad_r=gr)
    assert not bool(st.any())
    return x, lam, ga, gr


def _compare(ctx, problem, dtype, **kw):
    _wait(ctx, 0)
    want = _both(ctx, problem, **kw)
    _wait(ctx, DEFAULT)
    tol = 1e-12 if dtype == F64 else 5e-7
    for a, b, k in zip(_both(ctx, problem, **kw), want, (1, 1, 10, 10)):
        assert float((a - b).abs().max()) <= k * tol * max(1.0, float(b.abs().max()))


# workgroup rows around the limits of each length: 512, 1024, 2048 and 4096
# forward, 256, 384, 512, 1024, 3072 backward (FP64 and FP32 between them)
@pytest.mark.parametrize("rows", [255, 256, 383, 384, 511, 512, 1023, 1024, 2047, 2048, 3072,
                                  4096])
@pytest.mark.parametrize("dtype", [F64, F32])
def test_numbers_of_rows(ctx, dtype, rows):
    lens = np.tile([513, 1023, 1024, 2047, 2048, 4095], rows // 6 + 1)[:rows]
    _compare(ctx, _problem(lens, dtype), dtype)


@pytest.mark.parametrize("lambda0", ["zero", "formula"])
@pytest.mark.parametrize("dtype", [F64, F32])
def test_both_kinds_in_a_call(ctx, dtype, lambda0):
    past = 524_288 if dtype == F64 else 1_048_576
    lens = np.array([513, 4095, 4096, 8191, 8192, 16383, 16384, 32767, 32768, past - 1, past, 0,
                     1, 64, 512, 2048, 600])
    _compare(ctx, _problem(lens, dtype), dtype, lambda0=lambda0)
    _compare(ctx, _problem(np.array([past, 700, past + 3]), dtype), dtype, lambda0=lambda0)


@pytest.mark.parametrize("schedule", [(4, 2, 1, 0), (8, 4, 0, 0)])
@pytest.mark.parametrize("rows", [40, 600])
def test_schedules(ctx, schedule, rows):
    """Wave rows first, and workgroup rows from 257 values on."""
    import paper_2603_15910_amd as cqk
    from paper_2603_15910_amd import _lib as L
    lens = np.random.default_rng(rows).integers(0, 6000, rows)
    for which in (2, 3):
        _, old = cqk.cqk_get_batch_schedule(ctx.handle, which)
        assert cqk.cqk_set_batch_schedule(ctx.handle, which, L.cqk_batch_schedule(*schedule)) == 0
    try:
        p = _problem(lens, F64)
        p[2][torch.from_numpy(lens == 0).cuda()] = 0.0
        _compare(ctx, p, F64)
    finally:
        for which in (2, 3):
            assert cqk.cqk_set_batch_schedule(ctx.handle, which, old) == 0


@pytest.mark.parametrize("lens", ["8 of 10 to 3000", "100 of 10 to 600"])
@pytest.mark.parametrize("dtype", [F64, F32])
def test_few_short_rows_are_not_slower(ctx, dtype, lens):
    n, lo, hi = {"8 of 10 to 3000": (8, 10, 3000), "100 of 10 to 600": (100, 10, 600)}[lens]
    t, to, r, g = _problem(np.random.default_rng(1).integers(lo, hi, n), dtype)
    x, ga = torch.empty_like(t[0]), torch.empty_like(t[0])
    calls = (lambda: ctx.solve_batched(*t, to, r, out=x),
             lambda: ctx.solve_batched_backward(x, g, t[0], t[2], t[3], t[4], to, grad_a=ga))

    def median(call):
        for _ in range(5):
            call()
        took = []
        for _ in range(40):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            call()
            torch.cuda.synchronize()
            took.append(time.perf_counter() - t0)
        return 1e6 * sorted(took)[20]

    for call in calls:
        us = {}
        for _ in range(3):
            for ticks in (0, DEFAULT):
                _wait(ctx, ticks)
                us[ticks] = min(us.get(ticks, 1e9), median(call))
        # the streaming route and the empty launch of the teams' kernel
        assert us[DEFAULT] <= 1.1 * us[0] + 5.0, us
