"""Batches whose instances make several steps per pass (tubes in windows, FP32 grids in
pairs) against the same instances alone in single steps, bit for bit: mixed sizes and
storage in one batch, instances that finish inside a run and inside a graph, that are
added at any step, and runs of odd length, after which an instance is at an odd step."""
import numpy as np
import pytest

from paper_2609_16361_amd import binding, inputs

pytestmark = pytest.mark.gpu

F32, F16 = binding.LBM_STORE_F32, binding.LBM_STORE_F16
SHAPES = [((200, 4, 4), (1, 0, 0), F32), ((333, 4, 4), (1, 0, 0), F16), ((40, 36, 33), (0, 0, 0), F32),
          ((70, 9, 20), (0, 1, 1), F32), ((24, 24, 24), (0, 0, 0), F16), ((50, 5, 5), (0, 0, 1), F32),
          ((600, 1, 1), (1, 0, 0), F32), ((30, 2, 3), (0, 0, 0), F16)]


def alone(case, storage, steps):
    with binding.Solver(case.params, storage=storage, odd_lds=False) as s:
        s.init(case.Q0)
        s.step(steps)
        return s.populations()[0].view(np.uint32)


@pytest.mark.parametrize("collision", [inputs.RLB_SENSOR, inputs.BGK])
@pytest.mark.parametrize("graph_steps,runs", [(16, [16, 48, 10]), (50, [150]), (10, [7, 30, 13, 20]), (1, [30, 4, 2]),
                                              (6, [6, 6, 18])])
def test_batch_passes_are_bitwise_single_steps(graph_steps, runs, collision):
    print("batch", graph_steps, runs, collision, flush=True)
    total = sum(runs)
    cases = [inputs.random_smooth(*d, seed=20 + i, amp=0.04, bc=bc, collision=collision)
             for i, (d, bc, _) in enumerate(SHAPES)]
    # some finish early: inside a graph, at a graph's end, after an odd number of steps
    steps = [total, total - 3, total, max(2, total // 2), total, runs[0], total + 9, max(1, runs[0] - 1)]
    with binding.Batch(1 << 28, graph_steps=graph_steps) as b:
        ids = [b.add(c.params, c.Q0, n, storage=st) for c, n, (_, _, st) in zip(cases, steps, SHAPES)]
        late = None
        for i, n in enumerate(runs):
            b.run(n)
            if i == 0 and len(runs) > 1:
                late = b.add(cases[2].params, cases[2].Q0, 1000, storage=F32)
        for i, c, n, (_, _, st) in zip(ids, cases, steps, SHAPES):
            f, done = b.populations(i)
            assert done == min(n, total)
            assert np.isfinite(f).all()
            assert np.array_equal(f.view(np.uint32), alone(c, st, done)), (i, done)
        if late is not None:
            f, done = b.populations(late)
            assert done == total - runs[0]
            assert np.array_equal(f.view(np.uint32), alone(cases[2], F32, done))
