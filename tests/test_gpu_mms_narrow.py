"""GPU: the manufactured source on lattices whose rows fill a small part of a tile, which
evaluate it per cell, on both sides of that rule, against the FP64 oracle; and the longest
rows, whose coordinates come near 2^31.

Bar: as at the tiles' edges, 2^-23 of each field's largest |S|.  On the longest rows the
argument K x has a rounding of its own: up to 2^31 K 2^-52 and as much from K, 2^-20 in
all at K = 2 pi / 64; S changes by at most about four times that of its largest value.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_16361_amd import binding, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(1, 64, 2100), (6, 100, 400), (1, 1, 40000), (40000, 1, 1), (1, 40000, 1),
                                  (14, 64, 700), (15, 64, 700), (3, 5, 7), (70, 1, 9000)])
def test_source_on_narrow_lattices(dims):
    case = inputs.mms(n=64)
    nx, ny, nz = dims
    print("mms source", dims, flush=True)
    guard = 4096
    S = torch.full((5 * nx * ny * nz + guard,), -7.0, dtype=torch.float32, device="cuda")
    binding.lbm_mms_source(case.meta["mms"], nx, ny, nz, 37.5, S.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert bool((S[-guard:] == -7.0).all())
    got = S[:-guard].cpu().numpy().reshape(5, nz, ny, nx).astype(np.float64)
    want = oracle.mms_source(dict(case.params, nx=nx, ny=ny, nz=nz), case.meta["mms"], 37.5)
    for k in range(5):
        err = np.abs(got[k] - want[k]).max() / np.abs(want[k]).max()
        assert err <= 2.0 ** -23, (dims, k, err)


def test_source_near_2_to_31_cells_along_one_axis():
    case = inputs.mms(n=64)  # period 64
    n = 2 ** 31 - 1
    print("mms source", n, flush=True)
    S = torch.full((5, n + 64), -7.0, dtype=torch.float32, device="cuda").reshape(-1)
    stream = torch.cuda.current_stream().cuda_stream
    for dims in ((n, 1, 1), (1, n, 1), (1, 1, n)):
        binding.lbm_mms_source(case.meta["mms"], *dims, 37.5, S.data_ptr(), stream)
        torch.cuda.synchronize()
        assert bool((S[5 * n:] == -7.0).all())
        small = tuple(min(d, 64) for d in dims)
        want = oracle.mms_source(dict(case.params, nx=small[0], ny=small[1], nz=small[2]), case.meta["mms"],
                                 37.5).reshape(5, 64)
        at = (n - 64) % 64
        for k in range(5):
            got = S[k * n + n - 64:k * n + n].cpu().numpy().astype(np.float64)
            first = S[k * n:k * n + 64].cpu().numpy().astype(np.float64)
            scale = np.abs(want[k]).max()
            assert np.abs(first - want[k]).max() <= 2.0 ** -23 * scale
            assert np.abs(got - np.roll(want[k], -at)).max() <= 2.0 ** -18 * scale, (dims, k)
