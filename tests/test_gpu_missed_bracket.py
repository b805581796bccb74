"""A general solve whose first step leaves the sampled bracket: how many passes
are queued before the host looks at the state again."""
import pytest

from oracle import cqk_oracle as O
from paper_2603_15910_amd import workloads as W
from tests.parity import check_cqk

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_launches_after_a_missed_first_iterate():
    """The pass after the first one writes the set for the iterates that
    follow, one launch finishes them, and no further passes wait behind with
    nothing to do."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_15910_amd as cqk
    n = 2_200_001
    inst = W.cqk_uniform(n, 1)
    ref = O.solve_cqk(*[inst[k] for k in "dablu"], inst["r"])
    t = [torch.from_numpy(inst[k]).cuda() for k in "dablu"]
    ctx = cqk.Context(0)
    x, info = ctx.solve(*t, inst["r"], lambda0="user", lambda0_user=0.1)
    ctx.close()
    check_cqk(x.cpu().numpy(), inst, ref, 1e-10)
    # two sample kernels, the first pass, then the next one in its two forms
    # and one more
    assert info["pass_launches"] <= 6
