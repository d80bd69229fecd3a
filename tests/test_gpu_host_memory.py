"""Readouts and uploads of 4 MiB and more through memory and streams that take a route of
their own: pinned user memory, which the runtime copies itself, and hipStreamPerThread,
on which every copy stays in the calling thread.  The same bits as through ordinary
memory on a private stream."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2609_16361_amd import binding, inputs

pytestmark = pytest.mark.gpu
PER_THREAD = 2  # hipStreamPerThread


@pytest.mark.parametrize("storage", [binding.LBM_STORE_F32, binding.LBM_STORE_F16])
@pytest.mark.parametrize("stream", [None, PER_THREAD])
def test_pinned_memory_and_the_per_thread_stream(stream, storage):
    print("host memory", stream, storage, flush=True)
    case = inputs.random_smooth(96, 64, 65, seed=12, amp=0.05)
    with binding.Solver(case.params, storage=storage) as s:
        s.init(case.Q0)
        s.step(30)
        f, _ = s.populations()
        Q = s.moments()
    lib = binding.load()
    pinned = torch.empty(35 * case.cells, dtype=torch.float32, pin_memory=True)
    pinned_q = torch.empty(5 * case.cells, dtype=torch.float64, pin_memory=True)
    as_f = ctypes.cast(pinned.data_ptr(), ctypes.POINTER(ctypes.c_float))
    as_q = ctypes.cast(pinned_q.data_ptr(), ctypes.POINTER(ctypes.c_double))
    with binding.Solver(case.params, storage=storage, stream=stream) as s:
        pinned_q.copy_(torch.as_tensor(np.ascontiguousarray(case.Q0)).reshape(-1))
        assert lib.lbm_init_fields(s.ctx, as_q) == 0
        for again in range(3):  # the readout follows steps that are still running
            s.set_populations(f, 0) if again else None
            s.init(case.Q0)
            s.step(30)
            assert np.array_equal(s.populations()[0].view(np.uint32), f.view(np.uint32))
            assert np.array_equal(s.moments(), Q)
        step = ctypes.c_int64()
        assert lib.lbm_get_populations(s.ctx, as_f, ctypes.byref(step)) == 0 and step.value == 30
        assert np.array_equal(pinned.numpy().view(np.uint32), f.reshape(-1).view(np.uint32))
        assert lib.lbm_moments(s.ctx, as_q) == 0
        assert np.array_equal(pinned_q.numpy(), Q.reshape(-1))
        assert lib.lbm_set_populations(s.ctx, as_f, 30) == 0
        if storage == binding.LBM_STORE_F32:
            assert np.array_equal(s.populations()[0].view(np.uint32), f.view(np.uint32))
    if stream is None:
        return
    with binding.Batch(1 << 27, stream=stream) as b:
        i = b.add(case.params, case.Q0, 30, storage=storage)
        b.run(30)
        assert np.array_equal(b.populations(i)[0].view(np.uint32), f.view(np.uint32))
        assert np.array_equal(b.moments(i), Q)
