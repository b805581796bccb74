"""After a block of a one-launch call gave up, the context's next calls take
the multi-launch route at once: 16, then 32, ... while tries go on ending so.
And callers on several streams at once, whose launches compete for the compute
units, get their results without a wait per call."""
import threading
import time

import numpy as np
import pytest

from paper_2603_15910_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

DEFAULT = 30_000


@pytest.fixture()
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_15910_amd as cqk
    c = cqk.Context(0)
    yield c
    c.close()


def _late(ctx, block, exchange):
    import paper_2603_15910_amd as cqk
    assert cqk.cqk_set_team_late(ctx.handle, block, exchange) == 0


def _solve(n, seed=8):
    inst = W.cqk_uniform(n, seed)
    t = [torch.from_numpy(inst[k]).cuda() for k in "dablu"]
    return lambda c, **kw: c.solve(*t, inst["r"], **kw)


def _project(n, dtype, seed=4):
    t = torch.from_numpy(W.simplex_input(n, seed, "normal", dtype)).cuda()
    return lambda c, **kw: c.project_simplex(t, 1.0, **kw)


def _rows(seed=3):
    lens = np.random.default_rng(seed).integers(300, 60_000, 300)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    inst = W.cqk_uniform(int(off[-1]), seed)
    t = [torch.from_numpy(inst[k]).cuda() for k in "dablu"]
    to = torch.from_numpy(off).cuda()
    r = torch.segment_reduce(t[2] * (t[3] + t[4]) * 0.5, "sum", lengths=to[1:] - to[:-1])
    return lambda c, **kw: c.solve_batched(*t, to, r, **kw)


@pytest.mark.parametrize("what", ["solve", "projection", "long projection"])
def test_pause_of_waiting_calls(ctx, what):
    call, one = {"solve": (_solve(50_001), 1),
                 "projection": (_project(50_001, np.float64), 1),
                 "long projection": (_project(6_300_001, np.float64), 3)}[what]
    for pause in (16, 32):
        _late(ctx, 1, 2)
        assert call(ctx)[1]["pass_launches"] > one
        _late(ctx, 0, 0)
        for _ in range(pause):
            assert call(ctx)[1]["pass_launches"] > one
        assert call(ctx)[1]["pass_launches"] == one
    for _ in range(64):
        assert call(ctx)[1]["pass_launches"] == one
    _late(ctx, 1, 2)
    call(ctx)
    _late(ctx, 0, 0)
    for _ in range(16):
        assert call(ctx)[1]["pass_launches"] > one
    assert call(ctx)[1]["pass_launches"] == one


def test_setting_the_wait_ends_a_pause(ctx):
    import paper_2603_15910_amd as cqk
    call = _solve(50_001)
    _late(ctx, 1, 1)
    assert call(ctx)[1]["pass_launches"] > 1
    _late(ctx, 0, 0)
    assert call(ctx)[1]["pass_launches"] > 1
    assert cqk.cqk_set_team_wait(ctx.handle, DEFAULT) == 0
    assert call(ctx)[1]["pass_launches"] == 1


def test_pause_of_queued_calls(ctx):
    n = 50_001
    call = _project(n, np.float64)

    def one_launch():
        call(ctx, sync=False, max_iter=20)
        st, info = ctx.ctx_last_info()
        assert st == 0
        # x as the map of all of y, or the survivors' entries alone
        return info["finalize_bytes"] == 2.0 * 8 * n

    for pause in (16, 32):
        _late(ctx, 1, 2)
        assert not one_launch()
        _late(ctx, 0, 0)
        for _ in range(pause):
            assert not one_launch()
        assert one_launch()


def test_pause_of_batched_calls(ctx):
    call = _rows()
    want = call(ctx)[0]
    _late(ctx, 3, 2)
    got = [call(ctx)[0]]
    _late(ctx, 0, 0)
    for k in range(20):
        got.append(call(ctx, sync=k % 2 == 0)[0])
    torch.cuda.synchronize()
    for x in got:
        assert float((x - want).abs().max()) <= 1e-11


def test_one_try_of_a_set_in_a_call(ctx):
    """n past the registers: a first launch on the compacted set gives up, the
    pass kernels finish; no further launch of the call tries again."""
    call = _solve(4_400_003)
    x, info = call(ctx)
    _late(ctx, 1, 1)
    y, other = call(ctx)
    _late(ctx, 0, 0)
    assert other["status"] == 0 and other["pass_launches"] > info["pass_launches"]
    assert float((x - y).abs().max()) <= 1e-11


@pytest.mark.parametrize("kinds", [("solve",) * 4, ("long",) * 4, ("rows",) * 4,
                                   ("solve", "long", "rows", "projection")])
def test_callers_at_once(kinds):
    """Four threads with a context and a stream each.  A call alone takes 0.1
    to 0.4 ms; with a wait of 20 ms in every one, 60 of them took 1 to 3 s."""
    import paper_2603_15910_amd as cqk
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    make = {"solve": lambda i: _solve(2_000_000, i), "long": lambda i: _solve(5_000_000, i),
            "rows": _rows, "projection": lambda i: _project(10_000_000, np.float32, i)}
    calls = [make[k](i + 1) for i, k in enumerate(kinds)]
    ctxs = [cqk.Context(0) for _ in kinds]
    streams = [torch.cuda.Stream() for _ in kinds]
    torch.cuda.synchronize()
    want = []
    for call, c, s in zip(calls, ctxs, streams):
        with torch.cuda.stream(s):
            call(c)
            want.append(call(c)[0])
            s.synchronize()
    start, bad, took = threading.Barrier(len(kinds)), [], [0.0] * len(kinds)

    def work(i):
        try:
            with torch.cuda.stream(streams[i]):
                start.wait()
                t0 = time.perf_counter()
                got = [calls[i](ctxs[i])[0] for _ in range(60)]
                took[i] = time.perf_counter() - t0
                for x in got:
                    tol = 1e-11 if x.dtype == torch.float64 else 5e-7 * float(want[i].abs().max())
                    if float((x - want[i]).abs().max()) > tol:
                        bad.append(i)
        except Exception as e:   # a thread's failure has to reach the test
            bad.append(e)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(kinds))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for c in ctxs:
        c.close()
    assert not bad, bad
    assert max(took) < 0.5, took
