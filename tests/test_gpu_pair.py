"""Step pairs (two steps per pass over memory) against single steps: the same FP32
operations on the same values, so every population must agree bit for bit.  The
direct odd step (odd_lds off) keeps a context in single steps; the grids below sit at
the edges of the pair kernel's tiles: one tile per axis and several, cut last tiles,
halos that wrap onto the tile itself, zero-gradient faces on each axis, single planes
and rows, and segments of one plane."""
import numpy as np
import pytest
import torch

from paper_2609_16361_amd import binding, inputs

pytestmark = pytest.mark.gpu

GRIDS = [((64, 16, 6), (0, 0, 0)), ((111, 13, 9), (0, 0, 0)), ((70, 33, 20), (1, 0, 0)),
         ((70, 33, 20), (0, 1, 1)), ((130, 20, 17), (1, 1, 1)), ((128, 16, 2), (0, 0, 1)),
         ((65, 9, 1), (1, 1, 0)), ((513, 40, 3), (0, 0, 0)), ((30, 600, 2), (0, 1, 0)),
         ((5, 3, 2), (0, 0, 0)), ((2000, 1, 1), (1, 0, 0)), ((1, 1, 1), (0, 0, 0)), ((1, 2, 90), (0, 1, 0))]


def solve(case, pairs, calls, diag_every=0):
    with binding.Solver(case.params, odd_lds=pairs) as s:
        s.init(case.Q0)
        for n in calls:
            s.step(n, diag_every)
        f, done = s.populations()
        recs, status = s.diagnostics()
    assert status == binding.LBM_OK
    return f, done, recs


@pytest.mark.parametrize("collision", [inputs.RLB_SENSOR, inputs.BGK])
@pytest.mark.parametrize("dims,bc", GRIDS)
def test_pairs_are_bitwise_single_steps(dims, bc, collision):
    print("pairs", dims, bc, collision, flush=True)
    case = inputs.random_smooth(*dims, seed=3, amp=0.05, bc=bc, collision=collision)
    f, done, _ = solve(case, True, [13])
    g, _, _ = solve(case, False, [13])
    assert done == 13 and np.isfinite(f).all()
    assert np.array_equal(f.view(np.uint32), g.view(np.uint32))


@pytest.mark.parametrize("calls,diag_every", [([4, 4, 7, 1, 22], 0), ([5, 33], 7), ([40], 10), ([1, 4, 3, 12], 4),
                                              ([20, 3, 1, 8], 0), ([40], 20), ([2, 3, 31], 12), ([9, 6], 1), ([30], 3)])
def test_pairs_between_calls_and_diagnostics(calls, diag_every):
    print("pairs", calls, diag_every, flush=True)
    case = inputs.random_smooth(96, 20, 12, seed=4, amp=0.05)
    f, done, recs = solve(case, True, calls, diag_every)
    g, _, want = solve(case, False, calls, diag_every)
    assert done == sum(calls)
    assert np.array_equal(f.view(np.uint32), g.view(np.uint32))
    assert [r["step"] for r in recs] == [r["step"] for r in want]
    # the two odd steps cut the diagnostic sums into other blocks: FP32 summation error
    for a, b in zip(recs, want):
        for k in ("Ek", "eps_s", "eps_d"):
            assert a[k] == pytest.approx(b[k], rel=1e-5, abs=1e-12)


def test_captured_steps_are_single_and_replay():
    # a captured launch must not keep the address of a buffer that can be given up
    case = inputs.random_smooth(40, 12, 10, seed=5, amp=0.05)
    st = torch.cuda.Stream()
    with binding.Solver(case.params, stream=st.cuda_stream) as a, binding.Solver(case.params) as b:
        a.init(case.Q0)
        b.init(case.Q0)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=st):
            a.step(8)
        a_step = a.step_count
        for _ in range(3):
            g.replay()
            torch.cuda.synchronize()
        b.step(24)
        f = a.populations()[0]
        assert a_step == 8 and np.array_equal(f.view(np.uint32), b.populations()[0].view(np.uint32))


def test_second_buffers_are_given_up_for_an_allocation():
    case = inputs.random_smooth(256, 16, 16, seed=6, amp=0.05)
    with binding.Solver(case.params, odd_lds=False) as ref:
        ref.init(case.Q0)
        ref.step(18)
        want = ref.populations()[0]
    big = dict(case.params, nx=320, ny=320, nz=320)
    need = binding.lbm_state_bytes(binding.make_params(big))
    with binding.Solver(case.params) as s, binding.Solver(big) as first:
        s.init(case.Q0)
        s.step(9)
        free = torch.cuda.mem_get_info()[0]
        torch.cuda.empty_cache()
        hog = torch.empty(free - need + (512 << 20), dtype=torch.uint8, device="cuda")
        with binding.Solver(big) as second:  # fits only in place of the second buffers
            assert second.step_count == 0
        s.step(9)
        f = s.populations()[0]
        del hog, first
    torch.cuda.empty_cache()
    assert np.array_equal(f.view(np.uint32), want.view(np.uint32))
