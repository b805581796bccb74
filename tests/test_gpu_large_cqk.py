"""The single CQK solve past the one-launch sizes: the iterations on a
compacted set in one launch (held to the oracle, the pass-by-pass route and
its iterates), the sampled set's second bracket around a predicted iterate,
and the first pass at a flat lam_0 that answers Algorithm 1's breakpoint
steps."""
import numpy as np
import pytest

from oracle import cqk_oracle as O
from paper_2603_15910_amd import workloads as W
from tests.parity import check_cqk

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

F64, F32 = torch.float64, torch.float32
N = 2_100_001


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


def _paper(n, seed, left=False):
    """The paper's weakly correlated class; from lam_0 = 0 phi is flat and
    lam* lies to the right, or, mirrored, to the left."""
    g = np.random.default_rng(seed)
    b = g.uniform(10, 25, n)
    d, a = b + g.uniform(-5, 5, n), b + g.uniform(-5, 5, n)
    p, q = g.uniform(10, 25, n), g.uniform(10, 25, n)
    l, u = np.minimum(p, q), np.maximum(p, q)
    if left:
        a, l, u = -a, -u, -l
    return dict(d=d, a=a, b=b, l=l, u=u, r=float(np.dot(b, (l + u) / 2)))


def _held(inst, dtype):
    """The instance as arrays of dtype hold it."""
    if dtype == F64:
        return inst
    out = {k: (v.astype(np.float32).astype(np.float64) if k in "dablu" else v)
           for k, v in inst.items()}
    out["r"] = float(np.dot(out["b"], (out["l"] + out["u"]) / 2))
    return out


def _arrays(inst, dtype=F64):
    return [torch.from_numpy(np.asarray(inst[k])).to("cuda", dtype) for k in "dablu"]


def _same_iterates(ctx, t, r, info, **kw):
    """lam and the number of iterations of the traced, pass-by-pass route."""
    _, traced = ctx.solve(*t, r, trace=True, **kw)
    assert abs(info["iterations"] - traced["iterations"]) <= 1
    assert abs(info["lambda"] - traced["lambda"]) <= 1e-12 * (1.0 + abs(traced["lambda"]))
    return ctx.trace()


@pytest.mark.parametrize("dtype", [F64, F32])
@pytest.mark.parametrize("gen", ["uniform", "correlated", "paper", "paper_left"])
@pytest.mark.parametrize("n", [N, 4_400_003])
def test_against_the_oracle(ctx, dtype, gen, n):
    inst = (W.cqk_uniform(n, 61) if gen == "uniform" else
            W.cqk_correlated(n, 62) if gen == "correlated" else
            _paper(n, 63, left=gen == "paper_left"))
    inst = _held(inst, dtype)
    ref = O.solve_cqk(*[inst[k] for k in "dablu"], inst["r"])
    t = _arrays(inst, dtype)
    x, info = ctx.solve(*t, inst["r"])
    check_cqk(x.cpu().numpy().astype(np.float64), inst, ref, 1e-10 if dtype == F64 else 1e-5)
    tr = _same_iterates(ctx, t, inst["r"], info)
    if n >= 1 << 22:
        ev = [e for e in tr if e["kind"] == 1]
        if gen == "correlated":
            # lam_1 far from lam*, read from the set by its second bracket
            assert ev[1]["source"] == 3 and not (
                [e for e in tr if e["kind"] == 9][0]["lo"] < ev[1]["lam"])
        if gen.startswith("paper"):
            # past the last breakpoint phi is known without a pass, and the
            # steps are those of a run without compaction
            _, off = ctx.solve(*t, inst["r"], trace=True, compaction="off")
            lams = [[e["lam"] for e in z if e["kind"] in (1, 5)] for z in (tr, ctx.trace())]
            assert abs(len(lams[0]) - len(lams[1])) <= 1
            k = min(map(len, lams))
            np.testing.assert_allclose(lams[0][:k], lams[1][:k], rtol=1e-9)
    # a warm start from the solution
    xw, winfo = ctx.solve(*t, inst["r"], xbar=x)
    check_cqk(xw.cpu().numpy().astype(np.float64), inst, ref, 1e-10 if dtype == F64 else 1e-5)


@pytest.mark.parametrize("kind", ["ties", "fixed", "infinite", "all_fixed_but_one_side", "outlier"])
@pytest.mark.parametrize("left", [False, True])
def test_flat_start_edges(ctx, kind, left):
    n = 4_200_001
    inst = _paper(n, 71)
    g = np.random.default_rng(72)
    if kind == "ties":
        # whole numbers: the first and last breakpoint belong to many indices
        inst["d"] = np.round(g.uniform(1, 3, n))
        inst["b"] = np.ones(n)
        inst["a"] = np.round(g.uniform(0, 3, n))
        inst["l"] = np.round(g.uniform(4, 6, n))
        inst["u"] = inst["l"] + np.round(g.uniform(1, 3, n))
    elif kind == "fixed":
        m = g.random(n) < 0.5
        inst["u"][m] = inst["l"][m]
    elif kind == "infinite":
        inst["u"][g.random(n) < 0.1] = np.inf
    elif kind == "all_fixed_but_one_side":
        inst["u"][: n // 2] = inst["l"][: n // 2]
    else:
        inst["u"][12345] = 1e9
    up = np.where(np.isfinite(inst["u"]) & (inst["u"] < 1e8), inst["u"], inst["l"] + 5)
    inst["r"] = float(np.dot(inst["b"], (inst["l"] + up) / 2))
    if left:
        inst["a"], inst["l"], inst["u"] = -inst["a"], -inst["u"], -inst["l"]
        inst["r"] = -inst["r"]
    ref = O.solve_cqk(*[inst[k] for k in "dablu"], inst["r"])
    t = _arrays(inst)
    x, info = ctx.solve(*t, inst["r"])
    check_cqk(x.cpu().numpy(), inst, ref, 1e-10)
    _same_iterates(ctx, t, inst["r"], info)


def test_flat_start_with_a_bad_value_and_without_a_solution(ctx):
    n = 4_200_001
    inst = _paper(n, 73)
    t = _arrays(inst)
    for bad in (np.nan, np.inf):
        t[1][n - 7] = bad
        _, info = ctx.solve(*t, inst["r"], check=False)
        assert info["status"] == 2, (bad, info)
    t = _arrays(inst)
    _, info = ctx.solve(*t, 1.01 * float(np.dot(inst["b"], inst["u"])), check=False)
    assert info["status"] == 1, info
    _, info = ctx.solve(*t, 0.99 * float(np.dot(inst["b"], inst["l"])), check=False)
    assert info["status"] == 1, info


@pytest.mark.parametrize("order", ["clustered", "shuffled"])
def test_set_longer_than_the_registers(ctx, order):
    """theta = 1 keeps every side whatever its size; sorted by breakpoint the
    survivors fill a few waves' regions, which outgrow the registers."""
    inst = W.cqk_uniform(N, 65)
    if order == "clustered":
        k = np.argsort((inst["b"] * inst["l"] - inst["b"] * inst["a"] / inst["d"])
                       / (inst["b"] ** 2 / inst["d"]))
        inst = {q: (v[k] if q in "dablu" else v) for q, v in inst.items()}
    ref = O.solve_cqk(*[inst[k] for k in "dablu"], inst["r"])
    t = _arrays(inst)
    for kw in (dict(compaction="always"), {}):
        x, info = ctx.solve(*t, inst["r"], **kw)
        check_cqk(x.cpu().numpy(), inst, ref, 1e-10)
        _same_iterates(ctx, t, inst["r"], info, **kw)


def test_leaving_the_set_goes_back_to_the_arrays(ctx):
    """Sampled tiles that are not like the rest: the bracket misses lam*, the
    launch on the set ends at the iterate that leaves it, and passes over the
    caller's arrays finish."""
    n = 4_500_007
    inst = W.cqk_uniform(n, 43)
    pos = (np.arange(16384)[:, None] * (n // 16384) + np.arange(64)[None, :]).ravel()
    inst["d"][pos] = inst["b"][pos] = 1.0
    inst["l"][pos], inst["u"][pos] = -50.0, 50.0
    target = 0.0
    for _ in range(12):
        inst["r"] = float(np.dot(inst["b"], (inst["l"] + inst["u"]) / 2))
        inst["a"][pos] = inst["r"] / n - target + np.random.default_rng(44).uniform(
            -1e-3, 1e-3, pos.size)
        c, s = inst["b"] * inst["a"] / inst["d"], inst["b"] ** 2 / inst["d"]
        lo, hi = inst["b"] * inst["l"], inst["b"] * inst["u"]
        res = np.sum(np.clip(c, lo, hi)) - inst["r"]
        m = (c > lo) & (c <= hi) if res > 0 else (c >= lo) & (c < hi)
        target = -res / s[m].sum()
    inst["r"] = float(np.dot(inst["b"], (inst["l"] + inst["u"]) / 2))
    ref = O.solve_cqk(*[inst[k] for k in "dablu"], inst["r"])
    t = _arrays(inst)
    x, info = ctx.solve(*t, inst["r"])
    check_cqk(x.cpu().numpy(), inst, ref, 1e-10)
    tr = _same_iterates(ctx, t, inst["r"], info)
    assert any(e["kind"] == 1 and e["source"] == 0 for e in tr[3:])


@pytest.mark.parametrize("gen", ["uniform", "correlated", "paper"])
def test_blocks_that_give_up_and_queued_calls(ctx, gen):
    n = 4_400_003
    inst = (W.cqk_uniform(n, 81) if gen == "uniform" else
            W.cqk_correlated(n, 81) if gen == "correlated" else _paper(n, 81))
    ref = O.solve_cqk(*[inst[k] for k in "dablu"], inst["r"])
    t = _arrays(inst)
    first, info1 = ctx.solve(*t, inst["r"])
    for sync in (True, False):
        for ticks in (1, 0, 2_000_000):
            _wait(ctx, ticks)
            x, info = ctx.solve(*t, inst["r"], out=torch.full_like(first, 7.0), sync=sync,
                                max_iter=25)
            if not sync:
                st, info = ctx.ctx_last_info()
                assert st == 0
            check_cqk(x.cpu().numpy(), inst, ref, 1e-10)
            if ticks == 2_000_000:
                assert torch.equal(x, first)
                for k in ("lambda", "iterations", "passes", "stop_reason", "n_free", "residual"):
                    assert info[k] == info1[k], k
    _wait(ctx, 2_000_000)


@pytest.mark.parametrize("gen", ["uniform", "paper"])
def test_replays(gen):
    import paper_2603_15910_amd as cqk
    n = N
    make = W.cqk_uniform if gen == "uniform" else _paper
    insts = [make(n, 91 + i) for i in range(2)]
    for i in insts:
        i["r"] = insts[0]["r"]
    c = cqk.Context(0)
    try:
        c.reserve(n, 0)
        t = _arrays(insts[0])
        x = torch.empty_like(t[0])
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.stream(s):
            with torch.cuda.graph(graph, stream=s):
                c.solve(*t, insts[0]["r"], out=x, max_iter=15)
        torch.cuda.synchronize()
        for inst in insts + insts:
            for dst, k in zip(t, "dablu"):
                dst.copy_(torch.from_numpy(inst[k]))
            x.fill_(3.0)
            graph.replay()
            torch.cuda.synchronize()
            eager, _ = cqk.solve(*t, inst["r"])
            assert torch.equal(x, eager)
    finally:
        c.close()
