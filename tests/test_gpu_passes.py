"""Several steps per pass on the shapes that large and flat grids take: tiles that walk many
planes, with and without zero-gradient faces, nontemporal stores (whole lines of states
beyond the Infinity Cache), tiles dealt plane by plane, single planes, slots more than
2^31 bytes apart.  Against single steps, whose kernels share no tile code with the pairs:
the same FP32 operations on the same values, so every population agrees bit for bit.  And
that passes are taken at all, here and on the shapes of the tests of small grids."""
import math

import pytest
import torch

from paper_2609_16361_amd import binding, inputs
from test_gpu_batch_passes import SHAPES
from test_gpu_pair import GRIDS
from test_gpu_tube import TUBES

pytestmark = pytest.mark.gpu
F32, F16 = binding.LBM_STORE_F32, binding.LBM_STORE_F16


def fields(prm, seed):
    """Smooth conserved fields, periodic, with phases from the seed, on the device."""
    d = dict(dtype=torch.float64, device="cuda")
    g = torch.Generator().manual_seed(seed)
    nx, ny, nz = prm["nx"], prm["ny"], prm["nz"]
    ax = [torch.arange(n, **d) * (2.0 * math.pi / n) for n in (nx, ny, nz)]
    Q = torch.empty((5, nz, ny, nx), **d)
    for k in range(5):
        p = (torch.rand(3, generator=g, dtype=torch.float64) * 6.28).tolist()
        wave = (torch.sin(ax[0] + p[0])[None, None, :] * torch.cos(ax[1] + p[1])[None, :, None] *
                torch.cos(ax[2] + p[2])[:, None, None])
        Q[k] = {0: prm["rho_ref"], 4: prm["E_ref"]}.get(k, 0.0) + 0.05 * (1.0 if k in (0, 4) else 0.3) * wave
        del wave
    return Q


def digest(F):
    """A sum of all words, each times an odd number of its own, modulo 2^64."""
    out = 0
    for at in range(0, F.numel(), 1 << 26):
        w = F[at:at + (1 << 26)].to(torch.int64)
        i = torch.arange(at, at + w.numel(), dtype=torch.int64, device="cuda")
        out += int((w * (2 * (i * 0x9E3779B97F4A7 % 0x7FFFFFFF) + 1)).sum())
    return out % (1 << 64)


def compare(dims, bc, collision, steps, diag_every=0, seed=1):
    base = inputs.random_smooth(8, 8, 8, seed=seed, amp=0.05, bc=bc, collision=collision).params
    prm = dict(base, nx=dims[0], ny=dims[1], nz=dims[2])
    p = binding.make_params(prm)
    size = binding.lbm_state_bytes(p)
    out = []
    for passes in (True, False):
        Q = fields(prm, seed)
        F = torch.zeros(size // 4, dtype=torch.int32, device="cuda")
        torch.cuda.synchronize()
        ctx = binding.lbm_create_in(p, F.data_ptr(), size)
        try:
            binding.lbm_set_passes(ctx, passes)
            binding.lbm_init_fields_device(ctx, Q.data_ptr())
            binding.lbm_moments_device(ctx, Q.data_ptr())
            torch.cuda.synchronize()
            assert bool((Q[0] > 0.5 * prm["rho_ref"]).all())
            del Q
            torch.cuda.empty_cache()  # the second buffer needs room to spare
            for n in steps:
                binding.lbm_step(ctx, n, diag_every)
            recs = binding.lbm_diagnostics(ctx)
            made = binding.lbm_get_passes(ctx)
            assert made["steps"] == sum(steps)
            assert (made["passes"] < sum(steps) - 2) == passes and (made["second_bytes"] == size) == passes
        finally:
            binding.lbm_destroy(ctx)
        torch.cuda.synchronize()
        assert all(bool(torch.isfinite(part.view(torch.float32)).all()) for part in F.split(1 << 28))
        out.append((digest(F), recs))
        del F
        torch.cuda.empty_cache()
    assert out[0] == out[1]


@pytest.mark.parametrize("collision", [inputs.RLB_SENSOR, inputs.BGK])
@pytest.mark.parametrize("dims,bc", [((128, 96, 86), (0, 0, 0)), ((128, 96, 86), (0, 0, 1)),
                                     ((111, 111, 111), (0, 0, 0)), ((111, 111, 111), (1, 1, 1)),
                                     ((128, 128, 128), (0, 0, 0)), ((128, 128, 128), (1, 1, 1)),
                                     ((64, 64, 1), (0, 0, 0)), ((64, 64, 1), (1, 1, 0)), ((300, 40, 1), (0, 1, 0))])
def test_pairs_over_many_planes(dims, bc, collision):
    print("planes", dims, bc, collision, flush=True)
    compare(dims, bc, collision, [13, 4, 22], 10)


@pytest.mark.parametrize("dims,bc", [((256, 256, 128), (0, 0, 0)), ((256, 256, 128), (1, 0, 1)),
                                     ((288, 288, 288), (0, 0, 0)), ((288, 288, 288), (0, 1, 1)),
                                     ((200, 200, 200), (0, 0, 0))])
def test_pairs_of_large_states(dims, bc):
    print("large", dims, bc, flush=True)
    compare(dims, bc, inputs.RLB_SENSOR, [9, 12])


def test_pairs_with_slots_beyond_2_to_31_bytes():
    # 458752000 cells, near the limit of 2^29: a slot is 1.8 GB, a plane 0.9 GB, and the
    # 32-bit offset from one slot to the next one's last cell of a plane 2.75 GB
    print("slots", flush=True)
    torch.cuda.empty_cache()
    free = torch.cuda.mem_get_info()[0]
    if free < 220 << 30:
        pytest.skip(f"{free >> 30} GiB free, 220 wanted")
    compare((16384, 14000, 2), (0, 1, 0), inputs.RLB_SENSOR, [9])


def test_small_grids_and_batches_take_passes():
    for shapes, storages in ((GRIDS, (F32,)), (TUBES, (F32, F16))):
        for dims, bc in shapes:
            case = inputs.random_smooth(*dims, seed=3, amp=0.05, bc=bc)
            for st in storages:
                with binding.Solver(case.params, storage=st) as s:
                    s.init(case.Q0)
                    s.step(23)
                    assert s.passes()["passes"] < 16, (dims, bc, st)
    with binding.Batch(1 << 28) as b:
        for i, (dims, bc, st) in enumerate(SHAPES):
            case = inputs.random_smooth(*dims, seed=20 + i, amp=0.04, bc=bc)
            b.add(case.params, case.Q0, 1000, storage=st)
        b.run(40)
        assert b.passes()["fast_steps"] == 40


def test_a_first_pass_beside_a_capture_leaves_it_whole():
    # the step that takes the second buffer allocates while another stream is captured
    case = inputs.random_smooth(40, 36, 33, seed=5, amp=0.05)
    Q = torch.as_tensor(case.Q0).cuda()
    x = torch.zeros(1000, device="cuda")
    side = torch.cuda.Stream()
    with binding.Solver(case.params) as s, binding.Solver(case.params, passes=False) as ref:
        binding.lbm_init_fields_device(s.ctx, Q.data_ptr())
        binding.lbm_init_fields_device(ref.ctx, Q.data_ptr())
        ref.step(9)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=side):
            x.add_(1.0)
            s.step(9)
            x.mul_(2.0)
        assert s.passes()["second_bytes"] > 0 and s.passes()["passes"] == 5
        for want in (2.0, 6.0, 14.0):
            g.replay()
            torch.cuda.synchronize()
            assert bool((x == want).all())
        assert (s.populations()[0] == ref.populations()[0]).all()
