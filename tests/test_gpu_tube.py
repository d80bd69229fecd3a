"""Several steps per pass for tubes against single steps (the direct odd step keeps a
context in single steps): the same operations and, in FP16, the same rounding after
every step, so every population must agree bit for bit.  Cross-sections of one cell up
to the largest a window takes, tubes shorter than a window's ends up to several
windows, zero-gradient faces on each axis, and calls whose step counts leave odd steps
and short passes."""
import numpy as np
import pytest

from paper_2609_16361_amd import binding, inputs

pytestmark = pytest.mark.gpu

TUBES = [((256, 4, 4), (1, 0, 0)), ((257, 4, 4), (0, 0, 0)), ((100, 3, 5), (1, 1, 1)), ((33, 4, 4), (0, 1, 0)),
         ((5, 2, 2), (0, 0, 1)), ((1, 1, 1), (0, 0, 0)), ((3, 1, 4), (1, 0, 0)), ((2000, 1, 1), (1, 0, 0)),
         ((90, 25, 1), (0, 1, 0)), ((70, 5, 5), (0, 0, 0)), ((61, 1, 23), (1, 0, 1)), ((5000, 4, 4), (1, 0, 0))]


def solve(case, storage, passes, calls, diag_every):
    with binding.Solver(case.params, storage=storage, odd_lds=passes) as s:
        s.init(case.Q0)
        for n in calls:
            s.step(n, diag_every)
        return s.populations()[0].view(np.uint32)


@pytest.mark.parametrize("storage", [binding.LBM_STORE_F32, binding.LBM_STORE_F16])
@pytest.mark.parametrize("collision", [inputs.RLB_SENSOR, inputs.BGK])
@pytest.mark.parametrize("dims,bc", TUBES)
def test_tube_passes_are_bitwise_single_steps(dims, bc, collision, storage):
    print("tube", dims, bc, collision, storage, flush=True)
    case = inputs.random_smooth(*dims, seed=8, amp=0.05, bc=bc, collision=collision)
    for calls, diag_every in (([23], 0), ([4, 1, 6, 17], 5)):
        a = solve(case, storage, True, calls, diag_every)
        assert np.isfinite(a.view(np.float32)).all()
        assert np.array_equal(a, solve(case, storage, False, calls, diag_every))
