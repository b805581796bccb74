"""Batched general CQK with many short rows: rows of up to 127 values go four
to a wave in calls of 16384 rows or more.  Against the same rows in smaller
calls (a row to a wave), and against the oracle on some of them."""
import numpy as np
import pytest

from oracle import cqk_oracle as O
from tests.parity import check_cqk

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

ROWS = 16_384 + 3
EDGES = [0, 1, 2, 15, 16, 17, 31, 32, 33, 63, 64, 65, 112, 113, 126, 127, 128, 129, 200]


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_15910_amd as cqk
    c = cqk.Context(0)
    yield c
    c.close()


def _rows(dtype, kind):
    g = np.random.default_rng(5)
    lens = g.integers(0, 140, ROWS)
    lens[:len(EDGES)] = EDGES
    if kind == "one_length":
        lens[:] = 127
    off = np.concatenate([[0], np.cumsum(lens)])
    n = int(off[-1])
    b, d = g.uniform(1, 10, n), g.uniform(1, 10, n)
    a = g.uniform(-10, 10, n)
    l, u = g.uniform(-5, 0, n), g.uniform(0, 5, n)
    if kind == "flat":            # phi flat at lam_0 = 0: breakpoint steps
        l, u = g.uniform(10, 15, n), g.uniform(15, 20, n)
    t = [np.asarray(v, np.float32).astype(np.float64) if dtype == torch.float32 else v
         for v in (d, a, b, l, u)]
    mid = t[2] * (t[3] + t[4]) / 2
    r = np.array([mid[off[i]:off[i + 1]].sum() for i in range(ROWS)])
    if kind == "bad":
        for row in (30, 31, 77):
            if lens[row]:
                t[1][off[row]] = np.nan
        r[40] = np.nan
        r[41] = 1e9                # no solution
        r[np.flatnonzero(lens == 0)[0]] = 1.0
    return t, off, r, lens


@pytest.mark.parametrize("kind", ["mixed", "one_length", "flat", "bad"])
@pytest.mark.parametrize("lambda0", ["zero", "formula"])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_against_a_row_to_a_wave(ctx, dtype, lambda0, kind):
    t, off, r, lens = _rows(dtype, kind)
    dev = [torch.from_numpy(v).to("cuda", dtype) for v in t]
    toff, tr = torch.from_numpy(off).cuda(), torch.from_numpy(r).cuda()

    def call(lo, hi):
        o = (toff[lo:hi + 1] - toff[lo]).contiguous()
        s = slice(int(off[lo]), int(off[hi]))
        lam = torch.empty(hi - lo, dtype=torch.float64, device="cuda")
        st = torch.empty(hi - lo, dtype=torch.int32, device="cuda")
        x, info = ctx.solve_batched(*[v[s].contiguous() for v in dev], o, tr[lo:hi].contiguous(),
                                    lambda_out=lam, status_out=st, check=False, lambda0=lambda0)
        return x, lam, st, info

    x, lam, st, info = call(0, ROWS)
    half = ROWS // 2
    parts = [call(0, half), call(half, ROWS)]
    assert torch.equal(st, torch.cat([p[2] for p in parts]))
    assert info["status"] == max(p[3]["status"] for p in parts)
    assert info["passes"] == pytest.approx(sum(p[3]["passes"] for p in parts), rel=1e-3)
    tol = 1e-12 if dtype == torch.float64 else 2e-7
    xp, lp = torch.cat([p[0] for p in parts]), torch.cat([p[1] for p in parts])
    torch.testing.assert_close(x, xp, rtol=tol, atol=tol, equal_nan=True)
    torch.testing.assert_close(lam, lp, rtol=1e-11, atol=1e-11, equal_nan=True)
    xh, sh = x.cpu().numpy().astype(np.float64), st.cpu().numpy()
    for row in list(range(len(EDGES))) + [500, ROWS - 1]:
        if sh[row] != 0 or lens[row] == 0:
            continue
        s = slice(int(off[row]), int(off[row + 1]))
        inst = {k: v[s] for k, v in zip("dablu", t)}
        inst["r"] = r[row]
        ref = O.solve_cqk(*[inst[k] for k in "dablu"], inst["r"])
        check_cqk(xh[s], inst, ref, 1e-10 if dtype == torch.float64 else 1e-5)
