"""The batched calls' work queues: every row is handed out exactly once and
the blocks' outcomes add up, for row counts around the number of queues (32)
and the four rows of a work item.  Rows are copies of one row, so each must
return that row's solution bit for bit and the totals are multiples of its
own."""
import numpy as np
import pytest

from paper_2603_15910_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

COUNTS = [1, 4, 31, 32, 33, 127, 129, 4097]


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_15910_amd as cqk
    c = cqk.Context(0)
    yield c
    c.close()


def _offsets(nseg, n):
    return torch.arange(nseg + 1, dtype=torch.int64, device="cuda") * n


# 90: a row in one wave's registers; 700: tile by tile in the simplex call,
# a workgroup's in the general one
@pytest.mark.parametrize("n", [90, 700])
@pytest.mark.parametrize("nseg", COUNTS)
def test_cqk_rows_once_each(ctx, nseg, n):
    inst = W.cqk_uniform(n, 5)
    one = [torch.from_numpy(inst[k]).cuda() for k in "dablu"]
    x1, info1 = ctx.solve_batched(*one, _offsets(1, n),
                                  torch.tensor([inst["r"]], dtype=torch.float64, device="cuda"))
    t = [v.repeat(nseg) for v in one]
    r = torch.full((nseg,), inst["r"], dtype=torch.float64, device="cuda")
    x, info = ctx.solve_batched(*t, _offsets(nseg, n), r,
                                out=torch.full((nseg * n,), 7.0, dtype=torch.float64,
                                               device="cuda"))
    assert torch.equal(x.view(nseg, n), x1.expand(nseg, n))
    assert info["iterations"] == info1["iterations"]
    assert info["passes"] == nseg * info1["passes"]


@pytest.mark.parametrize("n", [90, 700])
@pytest.mark.parametrize("nseg", COUNTS)
def test_simplex_rows_once_each(ctx, nseg, n):
    y1 = torch.from_numpy(W.simplex_input(n, 5)).cuda()
    x1, info1 = ctx.project_simplex_batched(y1, _offsets(1, n), 1.0)
    x, info = ctx.project_simplex_batched(y1.repeat(nseg), _offsets(nseg, n), 1.0,
                                          out=torch.full((nseg * n,), 7.0, device="cuda"))
    assert torch.equal(x.view(nseg, n), x1.expand(nseg, n))
    assert info["n_after_init"] == nseg * info1["n_after_init"]
    # the backward kernel shares the queues
    g = torch.randn(n, device="cuda", generator=torch.Generator("cuda").manual_seed(3))
    g1 = ctx.project_simplex_batched_backward(x1, g, _offsets(1, n))
    gy = ctx.project_simplex_batched_backward(x, g.repeat(nseg), _offsets(nseg, n),
                                              grad_y=torch.full((nseg * n,), 7.0, device="cuda"))
    assert torch.equal(gy.view(nseg, n), g1.expand(nseg, n))


@pytest.mark.parametrize("nseg", [33, 4097])
def test_a_bad_row_is_reported(ctx, nseg):
    n = 90
    y = torch.from_numpy(W.simplex_input(n, 5)).cuda().repeat(nseg)
    y[(nseg - 2) * n + 7] = float("nan")
    _, info = ctx.project_simplex_batched(y, _offsets(nseg, n), 1.0, check=False)
    assert info["status"] == 2   # CQK_INVALID_ARG, whichever block had the row


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("small_per", [4, 8])
def test_cqk_row_lengths(ctx, dtype, small_per):
    """Wave rows around their 64-value slots and limits, against the oracle
    row by row (tests/parity.py bars)."""
    from oracle import cqk_oracle as O
    from tests.parity import check_cqk
    lens = [1, 2, 63, 64, 65, 128, 129, 192, 255, 256, 257, 320, 449, 511, 512, 513, 0, 700] * 2
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    np_t = np.float64 if dtype == torch.float64 else np.float32
    inst = W.cqk_uniform(int(off[-1]), 9, np_t)
    mid = inst["b"].astype(np.float64) * (inst["l"].astype(np.float64) + inst["u"]) * 0.5
    r = np.array([float(np.sum(mid[off[s]:off[s + 1]])) for s in range(len(lens))])
    ctx.set_batch_schedule(small_per=small_per, general=True)
    x, info = ctx.solve_batched(*[torch.from_numpy(inst[k]).cuda() for k in "dablu"],
                                torch.from_numpy(off).cuda(), torch.from_numpy(r).cuda())
    ctx.set_batch_schedule(general=True)
    x = x.cpu().numpy()
    for s, n in enumerate(lens):
        if n == 0:
            continue
        row = {k: inst[k][off[s]:off[s + 1]] for k in "dablu"} | {"r": r[s]}
        ref = O.solve_cqk(*[row[k] for k in "dablu"], r[s])
        check_cqk(x[off[s]:off[s + 1]], row, ref, 1e-10 if dtype == torch.float64 else 1e-5)
