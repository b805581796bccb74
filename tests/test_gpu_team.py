"""The one-launch general solve (blocks of one launch exchanging their sums):
sizes around its block, value-per-thread and upper limits, every start, bad
and infeasible inputs, a block that gives up waiting, queued calls and graph
replays.  Results are held to the FP64 / FP32 bars of tests/parity.py against
the oracle."""
import numpy as np
import pytest

from oracle import cqk_oracle as O
from paper_2603_15910_amd import workloads as W
from tests.parity import check_cqk

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# one block of 4 values per thread: 2048; 256 blocks of 4, 8, 16: 524288,
# 1048576, 2097152; past that the multi-launch route
SIZES = [1, 2, 3, 511, 2047, 2048, 2049, 6145, 524_287, 524_289, 1_048_577, 2_097_151, 2_097_153]


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


def _dev(inst, dtype=torch.float64):
    return [torch.from_numpy(inst[k]).to("cuda", dtype) for k in "dablu"]


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_sizes(ctx, n, dtype):
    np_t = np.float64 if dtype == torch.float64 else np.float32
    inst = W.cqk_uniform(n, 11, np_t)
    ref = O.solve_cqk(*[inst[k] for k in "dablu"], inst["r"])
    x, info = ctx.solve(*_dev(inst, dtype), inst["r"])
    assert (info["pass_launches"] == 1) == (n <= 2_097_152)
    check_cqk(x.cpu().numpy(), inst, ref, 1e-10 if dtype == torch.float64 else 1e-5)


@pytest.mark.parametrize("start", ["formula", "user", "warm"])
@pytest.mark.parametrize("n", [777, 30_001])
def test_starts(ctx, n, start):
    inst = W.cqk_paper(n, 3, "weak")
    ref = O.solve_cqk(*[inst[k] for k in "dablu"], inst["r"])
    kw = {"formula": dict(lambda0="formula"), "user": dict(lambda0="user", lambda0_user=0.3),
          "warm": dict(xbar=torch.from_numpy(ref.x + 1e-3).cuda())}[start]
    x, info = ctx.solve(*_dev(inst), inst["r"], **kw)
    check_cqk(x.cpu().numpy(), inst, ref, 1e-10)
    # the multi-launch route's start and iterates
    _wait(ctx, 0)
    _, other = ctx.solve(*_dev(inst), inst["r"], **kw)
    _wait(ctx, 2_000_000)
    assert info["pass_launches"] == 1 and other["pass_launches"] > 1
    assert info["iterations"] == other["iterations"] and info["passes"] == other["passes"]
    # 4 is criterion 1 with phi(lam) = r to the last bit, which the order of
    # the sums decides
    assert {info["stop_reason"], other["stop_reason"]} in ({1}, {4}, {1, 4}, {2}, {3})
    assert info["n_free"] == other["n_free"]
    assert abs(info["lambda0"] - other["lambda0"]) <= 1e-12 * max(1.0, abs(other["lambda0"]))


def test_breakpoint_steps(ctx):
    # a start far from every breakpoint: slope zero, the closest-breakpoint search
    inst = W.cqk_uniform(50_001, 2)
    ref = O.solve_cqk(*[inst[k] for k in "dablu"], inst["r"])
    for lam0 in (-1e6, 1e6):
        x, info = ctx.solve(*_dev(inst), inst["r"], lambda0="user", lambda0_user=lam0)
        assert info["pass_launches"] == 1
        check_cqk(x.cpu().numpy(), inst, ref, 1e-10)


@pytest.mark.parametrize("n", [100, 9000])
def test_bad_and_infeasible(ctx, n):
    inst = W.cqk_uniform(n, 4)
    for k, v in (("d", -1.0), ("b", 0.0), ("a", np.nan), ("l", np.inf)):
        bad = dict(inst)
        bad[k] = inst[k].copy()
        bad[k][n - 1] = v
        _, info = ctx.solve(*_dev(bad), inst["r"], check=False)
        assert info["status"] == 2, k
    top = float(np.dot(inst["b"], inst["u"]))
    _, info = ctx.solve(*_dev(inst), 1.5 * abs(top) + 1.0, check=False)
    assert info["status"] == 1
    inf = dict(inst, l=np.full(n, -np.inf), u=np.full(n, np.inf))
    ref = O.solve_cqk(*[inf[k] for k in "dablu"], inst["r"])
    x, _ = ctx.solve(*_dev(inf), inst["r"])
    check_cqk(x.cpu().numpy(), inf, ref, 1e-10)


def test_views_at_any_element(ctx):
    inst = W.cqk_uniform(4099, 6)
    ref = O.solve_cqk(*[inst[k] for k in "dablu"], inst["r"])
    for off in (1, 3):
        t = [torch.cat([v[:off], v])[off:] for v in _dev(inst)]
        out = torch.full((4099 + 2 * off,), 5.0, dtype=torch.float64, device="cuda")
        ctx.solve(*t, inst["r"], out=out[off:off + 4099])
        check_cqk(out[off:off + 4099].cpu().numpy(), inst, ref, 1e-10)
        assert bool((out[:off] == 5.0).all()) and bool((out[off + 4099:] == 5.0).all())


def test_a_block_that_gives_up(ctx):
    # a wait limit of one tick (10 ns): the blocks give up at the first
    # exchange and the multi-launch route returns the solution
    inst = W.cqk_uniform(100_000, 8)
    ref = O.solve_cqk(*[inst[k] for k in "dablu"], inst["r"])
    t = _dev(inst)
    for sync in (True, False):
        _wait(ctx, 1)
        x, info = ctx.solve(*t, inst["r"], out=torch.full_like(t[0], 9.0), sync=sync, max_iter=20)
        if not sync:
            _, info = ctx.ctx_last_info()
        _wait(ctx, 2_000_000)
        assert info["pass_launches"] > 1
        check_cqk(x.cpu().numpy(), inst, ref, 1e-10)
        x, info = ctx.solve(*t, inst["r"])
        assert info["pass_launches"] == 1
        check_cqk(x.cpu().numpy(), inst, ref, 1e-10)


@pytest.mark.parametrize("n", [1500, 70_001])
def test_replays(ctx, n):
    ctx.reserve(n)
    insts = [W.cqk_uniform(n, s) for s in (1, 2, 3)]
    r = insts[0]["r"]
    t = _dev(insts[0])
    x = torch.empty_like(t[0])
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        with torch.cuda.graph(graph, stream=s):
            ctx.solve(*t, r, out=x, max_iter=20)
    for inst in insts + insts:
        for dst, k in zip(t, "dablu"):
            dst.copy_(torch.from_numpy(inst[k]))
        x.fill_(3.0)
        graph.replay()
        torch.cuda.synchronize()
        eager, info = ctx.solve(*t, r)
        assert info["pass_launches"] == 1
        assert torch.equal(x, eager)
