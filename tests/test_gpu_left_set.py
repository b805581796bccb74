"""A general solve whose compacted set the one launch leaves to the passes:
they are queued together, not two and then four."""
import pytest

from oracle import cqk_oracle as O
from paper_2603_15910_amd import workloads as W
from tests.parity import check_cqk

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_launches_on_a_set_that_was_left():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_15910_amd as cqk
    n = 2_200_001
    inst = W.cqk_uniform(n, 1)
    ref = O.solve_cqk(*[inst[k] for k in "dablu"], inst["r"])
    t = [torch.from_numpy(inst[k]).cuda() for k in "dablu"]
    ctx = cqk.Context(0)
    assert cqk.cqk_set_team_late(ctx.handle, 0, 1) == 0
    x, info = ctx.solve(*t, inst["r"])
    ctx.close()
    check_cqk(x.cpu().numpy(), inst, ref, 1e-10)
    # two sample kernels, the first pass, then the next one in its two forms
    # and three more
    assert info["pass_launches"] <= 8
