"""Rows of the batched general CQK held on chip by teams of blocks: lengths
around what one block and each team size hold, more and fewer rows than
teams, every start, the backward pass, a block that gives up waiting and graph
replays.  Rows are held to the oracle with the bars of tests/parity.py; the
VJP to the oracle's within 1e-10 (FP64) and 1e-5 (FP32) of max(1, |g|_inf),
on the free set of the GPU's own x."""
import numpy as np
import pytest

from oracle import cqk_oracle as O
from paper_2603_15910_amd import workloads as W
from tests.parity import check_cqk

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

F64, F32 = torch.float64, torch.float32
# one block holds 2047 FP64 or 4095 FP32 values, 256 blocks 524287 or 1048575;
# longer rows are streamed
EDGES = [513, 600, 2047, 2048, 2049, 4095, 4096, 4097, 8191, 16385, 65536, 131071]
LONG = [524_287, 524_288, 1_048_575, 1_048_576]


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
    np_t = np.float64 if dtype == F64 else np.float32
    inst = W.cqk_uniform(int(off[-1]), seed, np_t)
    mid = inst["b"].astype(np.float64) * (inst["l"].astype(np.float64) + inst["u"]) * 0.5
    inst["r"] = np.array([float(np.sum(mid[off[s]:off[s + 1]])) for s in range(len(lens))])
    t = [torch.from_numpy(inst[k]).cuda() for k in "dablu"]
    return off, inst, t, torch.from_numpy(off).cuda(), torch.from_numpy(inst["r"]).cuda()


def _check(x, off, inst, dtype, rows=None):
    x = x.cpu().numpy()
    for s in (range(off.size - 1) if rows is None else rows):
        if off[s + 1] == off[s]:
            continue
        row = {k: inst[k][off[s]:off[s + 1]] for k in "dablu"} | {"r": inst["r"][s]}
        ref = O.solve_cqk(*[row[k] for k in "dablu"], row["r"])
        check_cqk(x[off[s]:off[s + 1]], row, ref, 1e-10 if dtype == F64 else 1e-5)


def _check_vjp(ctx, x, t, offs, off, inst, dtype):
    n = int(off[-1])
    g = torch.from_numpy(W.upstream_grad(n, 3, np.float64)).cuda().to(dtype)
    gr = torch.empty(off.size - 1, dtype=F64, device="cuda")
    ga = ctx.solve_batched_backward(x, g, t[0], t[2], t[3], t[4], offs,
                                    grad_a=torch.full_like(g, 7.0), grad_r=gr)
    want_a, want_r = O.cqk_vjp_batched(*[v.double().cpu().numpy()
                                         for v in (x, g, t[0], t[2], t[3], t[4])], off)
    bar = (1e-10 if dtype == F64 else 1e-5) * max(1.0, float(g.abs().max()))
    assert np.max(np.abs(ga.double().cpu().numpy() - want_a)) <= bar
    assert np.max(np.abs(gr.cpu().numpy() - want_r)) <= 1e-10 * max(1.0, float(g.abs().max()))


@pytest.mark.parametrize("dtype", [F64, F32])
@pytest.mark.parametrize("start", ["zero", "formula", "user"])
def test_edges(ctx, dtype, start):
    off, inst, t, offs, r = _problem(EDGES[::-1] + EDGES + [0, 3, 300], dtype)
    x, info = ctx.solve_batched(*t, offs, r, lambda0=start, lambda0_user=0.4,
                                out=torch.full_like(t[0], 9.0))
    assert info["iterations"] >= 1
    _check(x, off, inst, dtype)
    if start == "zero":
        _check_vjp(ctx, x, t, offs, off, inst, dtype)


@pytest.mark.parametrize("dtype", [F64, F32])
@pytest.mark.parametrize("n", LONG)
def test_longest_rows(ctx, dtype, n):
    off, inst, t, offs, r = _problem([n, 700], dtype)
    x, _ = ctx.solve_batched(*t, offs, r)
    _check(x, off, inst, dtype)
    _check_vjp(ctx, x, t, offs, off, inst, dtype)


@pytest.mark.parametrize("rows", [1, 5, 63, 65, 300])
def test_more_and_fewer_rows_than_teams(ctx, rows):
    off, inst, t, offs, r = _problem([20_001] * rows + [5000] * 7, F64)
    x, info = ctx.solve_batched(*t, offs, r)
    _check(x, off, inst, F64, rows=range(0, off.size - 1, 1 if rows < 10 else 17))
    _check_vjp(ctx, x, t, offs, off, inst, F64)
    # every row once: the same rows streamed take the same iterations
    _wait(ctx, 0)
    y, other = ctx.solve_batched(*t, offs, r)
    _wait(ctx, 2_000_000)
    assert info["passes"] == other["passes"] and info["iterations"] == other["iterations"]
    assert float((x - y).abs().max()) <= 1e-10 * float(x.abs().max())


@pytest.mark.parametrize("dtype", [F64, F32])
def test_breakpoints_and_bad_rows(ctx, dtype):
    lens = [700, 3000, 9000, 30_000, 9000, 3000]
    off, inst, t, offs, r = _problem(lens, dtype)
    for lam0 in (-1e6, 1e6):   # slope zero at first: the closest-breakpoint search
        x, _ = ctx.solve_batched(*t, offs, r, lambda0="user", lambda0_user=lam0)
        _check(x, off, inst, dtype)
    bad = [v.clone() for v in t]
    bad[0][int(off[2]) - 1] = -1.0          # row 1: its last d
    r2 = r.clone()
    r2[3] = 1e12                            # row 3: out of reach
    st = torch.full((len(lens),), -7, dtype=torch.int32, device="cuda")
    x, info = ctx.solve_batched(*bad, offs, r2, status_out=st, check=False)
    assert st.tolist() == [0, 2, 0, 1, 0, 0] and info["status"] == 2
    assert bool(torch.isnan(x[int(off[1]):int(off[2])]).all())
    assert bool(torch.isnan(x[int(off[3]):int(off[4])]).all())
    _check(x, off, inst, dtype, rows=[0, 2, 4, 5])


@pytest.mark.parametrize("dtype", [F64, F32])
def test_a_block_that_gives_up(ctx, dtype):
    off, inst, t, offs, r = _problem([30_000] * 40 + [700] * 9, dtype)
    _wait(ctx, 1)   # 10 ns: the teams' rows fall to the streaming kernel
    x, info = ctx.solve_batched(*t, offs, r, out=torch.full_like(t[0], 9.0))
    _check(x, off, inst, dtype, rows=[0, 1, 20, 39, 40, 48])
    _check_vjp(ctx, x, t, offs, off, inst, dtype)
    _wait(ctx, 2_000_000)
    x, other = ctx.solve_batched(*t, offs, r)
    assert info["passes"] == other["passes"]
    _check(x, off, inst, dtype, rows=[0, 39, 48])


def test_replays(ctx):
    lens = [20_000, 700, 5000, 100, 40_000]
    off, inst, t, offs, r = _problem(lens, F64)
    other = _problem(lens, F64, seed=8)
    x = torch.empty_like(t[0])
    ctx.solve_batched(*t, offs, r, out=x)   # grows the buffers before the capture
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        with torch.cuda.graph(graph, stream=s):
            ctx.solve_batched(*t, offs, r, out=x, sync=False)
    for src in (other, (off, inst, [v.clone() for v in t], offs, r.clone()), other):
        for dst, v in zip(t, src[2]):
            dst.copy_(v)
        r.copy_(src[4])
        x.fill_(3.0)
        graph.replay()
        torch.cuda.synchronize()
        eager, _ = ctx.solve_batched(*t, offs, r)
        assert torch.equal(x, eager)
