"""Batched general CQK calls of uneven rows of which teams hold the longer ones
anyway: they hold the shorter workgroup rows too, so such a call takes about
what rows of one (held) length of as many values take.  Results are the
streaming route's (team wait 0) to the rounding of sums added in another order:
1e-12 (FP64), a unit in the last place of values up to 8 (FP32: 5e-7), ten
times that for the VJP."""
import time

import numpy as np
import pytest

from tests.test_gpu_few_rows import F32, F64, _compare, _problem, _wait

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


# one long row among short ones, in the list before, among and after them;
# rows past the longest team's beside held ones
@pytest.mark.parametrize("dtype", [F64, F32])
@pytest.mark.parametrize("lens", [
    [16384, 513, 600, 1024, 4095, 300, 64],
    [257, 16383, 4096, 511, 512, 513],
    [700] * 40 + [20_000] + [700] * 40 + [64] * 9,
    [1_048_577, 600, 33_000, 513, 2047, 100],
])
def test_short_rows_beside_held_ones(ctx, dtype, lens):
    _compare(ctx, _problem(lens, dtype), dtype)


def _us(fn):
    for _ in range(3):
        fn()
    ts = []
    for _ in range(40):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        fn()
        torch.cuda.synchronize()
        ts.append(time.perf_counter() - t0)
    return 1e6 * float(np.median(ts))


def test_time_of_uneven_rows(ctx):
    """The VJP of 100 rows of 5000 to 90 000 values against rows of 47 500:
    within 12 % (40 % with the rows below 16 384 streamed)."""
    _wait(ctx, 2_000_000)

    def took(lens):
        t, to, r, g = _problem(lens, F32)
        x, _ = ctx.solve_batched(*t, to, r)
        return _us(lambda: ctx.solve_batched_backward(x, g, t[0], t[2], t[3], t[4], to))

    uneven = took(np.random.default_rng(1).integers(5000, 90_000, 100))
    even = took(np.full(100, 47_500))
    _wait(ctx, 30_000)
    assert uneven < 1.12 * even, (uneven, even)
