"""Host data in and out: copies cut into chunks and moved by several threads, below, at
and above the size from which that is done, and the check of initial fields, which must
name the first unphysical cell wherever its thread's share lies."""
import numpy as np
import pytest

from paper_2609_16361_amd import binding, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(7, 5, 3), (128, 117, 2), (61, 53, 37), (96, 64, 65)])
@pytest.mark.parametrize("storage", [binding.LBM_STORE_F32, binding.LBM_STORE_F16])
def test_populations_and_moments_round_trip(dims, storage):
    print("copy", dims, storage, flush=True)
    case = inputs.random_smooth(*dims, seed=9, amp=0.05)
    with binding.Solver(case.params, storage=storage) as a, binding.Solver(case.params, storage=storage) as b:
        a.init(case.Q0)
        assert np.abs(a.moments() - case.Q0).max() < (2e-6 if storage == binding.LBM_STORE_F32 else 2e-2)
        a.step(3)
        f, at = a.populations()
        b.set_populations(f, at)
        g, at2 = b.populations()
        assert at == at2 == 3
        if storage == binding.LBM_STORE_F32:
            assert np.array_equal(f.view(np.uint32), g.view(np.uint32))
            assert np.array_equal(a.moments(), b.moments())
        else:
            # the restored state picks its own power-of-two scales: subnormals may round
            assert np.abs(f - g).max() <= 2.0 ** -10 * np.abs(f).max()
    with binding.Batch(1 << 27) as b:
        i = b.add(case.params, case.Q0, 5, storage=storage)
        b.run(3)
        assert np.array_equal(b.populations(i)[0].view(np.uint32), f.view(np.uint32))


def test_first_unphysical_cell_is_named():
    case = inputs.random_smooth(90, 40, 37, seed=10, amp=0.05)
    n = case.cells
    with binding.Solver(case.params) as s:
        s.init(case.Q0)
        before = s.moments()
        for cell in (0, 4095, 4096, n // 4, n // 4 - 1, n // 2 + 5, n - 1):
            for field, value, word in ((0, -1.0, "density"), (4, 0.0, "pressure"), (2, np.nan, "finite"),
                                       (3, np.inf, "finite")):
                Q = case.Q0.reshape(5, n).copy()
                Q[field, cell] = value
                Q[0, min(n - 1, cell + 7000)] = np.nan if cell + 7000 < n else Q[0, n - 1]
                with pytest.raises(binding.LbmError) as e:
                    s.init(Q)
                assert e.value.status == binding.LBM_EINVAL
                assert word in str(e.value) and f"cell {cell} " in str(e.value) + " ", (cell, field, str(e.value))
        assert np.array_equal(s.moments(), before)
