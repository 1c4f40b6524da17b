"""Rows of 1024 and 2048 points through the band-limited row pass, transformed in
parts of 512 points or whole by n and precision: the diffusion against the FP64
oracle to 1e-13 / 2e-6 (the bars of test_gpu_plane_pass.py), for bands that fit the
lowest eighth of a part, half of it, both halves of one, and every mode kept; and a
step reproduces the iterate.
"""
import numpy as np
import pytest

import oracle
from paper_1711_01365_amd import inputs

pytestmark = pytest.mark.gpu

F64, F32, FB = 0, 1, 2
PLANS = [(1, 1024, F64), (2, 1024, FB), (3, 1024, FB), (4, 1024, F32), (2, 1024, F64), (3, 1024, F64), (4, 1024, F64),
         (1, 2048, F32), (2, 2048, F64), (3, 2048, FB), (4, 2048, FB)]


@pytest.mark.parametrize("n,L,prec", PLANS)
def test_long_rows(n, L, prec):
    import torch
    from paper_1711_01365_amd import mbo
    dt = torch.float64 if prec == F64 else torch.float32
    grid = (64, L)
    A = torch.tensor(inputs.normal_field(n, grid, 71), dtype=dt, device="cuda")
    A64 = A.double().cpu().numpy()
    bands = []
    for tau in (2e-3, 1e-4, 2e-5, 8e-6, 1e-8):
        p = mbo.Plan(grid, n, tau, precision=prec)
        bands.append(p.path()[1])
        ref = oracle.heat(A64.reshape((n * n,) + grid), tau, 2)[0].reshape(A64.shape)
        D = p.diffuse(A).double().cpu().numpy()
        assert np.abs(D - ref).max() <= (1e-13 if prec == F64 else 2e-6), tau
        X = A.clone()
        p.iterate(X, 1)
        assert torch.equal(X, p.step(A)), tau
        p.close()
    assert bands[0] < 64 and bands[-1] == L // 2
    assert any(64 <= c < 256 for c in bands) and any(256 <= c < 512 for c in bands)
