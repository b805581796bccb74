"""A forward row that one block holds has the same bits in any batched general
CQK call of fewer than 16384 rows: alone, among many, beside a row that teams
hold, and with no teams."""
import numpy as np
import pytest

from paper_2603_15910_amd import workloads as W
from tests.test_gpu_few_rows import F32, F64, _wait

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_15910_amd as cqk
    c = cqk.Context(0)
    yield c
    c.close()


# one block holds up to 2047 FP64 or 4095 FP32 values
@pytest.mark.parametrize("dtype,n", [(F64, 513), (F64, 1200), (F64, 2047), (F32, 700), (F32, 4095)])
@pytest.mark.parametrize("ticks", [0, 2_000_000])
def test_a_row_has_the_same_bits_in_any_call(ctx, dtype, n, ticks):
    inst = W.cqk_uniform(n, 5, np.float64 if dtype == F64 else np.float32)
    one = [torch.from_numpy(inst[k]).to("cuda", dtype) for k in "dablu"]
    r = float((one[2].double() * (one[3].double() + one[4].double())).sum()) * 0.5

    def solve(rows, tail):
        long = [torch.from_numpy(v).to("cuda", dtype) for v in
                (W.cqk_uniform(tail, 6)[k] for k in "dablu")] if tail else None
        t = [torch.cat([v.repeat(rows)] + ([w] if tail else [])) for v, w in
             zip(one, long or one)]
        off = torch.tensor([k * n for k in range(rows + 1)] + ([rows * n + tail] if tail else []),
                           dtype=torch.int64, device="cuda")
        rr = torch.full((off.numel() - 1,), r, dtype=torch.float64, device="cuda")
        if tail:
            rr[-1] = float((long[2].double() * (long[3].double() + long[4].double())).sum()) * 0.5
        x, _ = ctx.solve_batched(*t, off, rr)
        return x[:rows * n].view(rows, n)

    _wait(ctx, 2_000_000)
    want = solve(1, 0)
    _wait(ctx, ticks)
    for rows, tail in ((3, 0), (600, 0), (5000, 0), (9000, 0), (2, 20_000)):
        x = solve(rows, tail)
        assert torch.equal(x, want.expand(rows, n)), (rows, tail)
    _wait(ctx, 30_000)
