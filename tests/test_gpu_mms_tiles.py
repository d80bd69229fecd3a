"""GPU: the manufactured source on lattices at the edges of its tiles (64 cells by 8 or
16 rows by 1, 2 or 4 planes), against the FP64 oracle.

Bar: the kernel evaluates in FP64 and stores FP32, so a value is off by its rounding,
2^-24 of itself, and the FP64 sums' own error, some 1e-13 of the field's largest: 2^-23
of each field's largest |S|.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_16361_amd import binding, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(1, 1, 1), (63, 17, 2), (65, 9, 3), (24, 24, 24),
                                  (64, 64, 64),       # 8 rows, 1 plane, whole tiles
                                  (200, 130, 33),     # 16 rows, 2 planes, remainders on every axis
                                  (130, 129, 130)])   # 16 rows, 4 planes, remainders on every axis
def test_source_at_tile_edges(dims):
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
