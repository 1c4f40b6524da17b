"""The 3-D plane pass at the edges of what it takes: the smallest planes (several
in one wave, the last workgroup part empty), planes of one wave, the largest plane
that a double fits in the LDS and the smallest that does not, sides of 8 to 128 (64 or 128 in float),
rows of 8 to 512 points, n = 1..4, two fields with every mode or a band kept.

The diffusion against the FP64 oracle (every path within 1e-13 in double, 2e-6 in
float), then three steps against the general passes, each from the same iterate.
Two diffusions within e of the exact one give polar factors within
4 e / (sigma_{n-1} + sigma_n) of each other (twice the first-order bound) away
from det ties, |det H| <= 2 n e |cof H|.  Energies: relative 1e-12 / 1e-5 with the
rounding of the identity's term, 8 n u / tau.
"""
import numpy as np
import pytest

import oracle
from paper_1711_01365_amd import inputs

pytestmark = pytest.mark.gpu

F64, F32, FB = 0, 1, 2
CASES = [((8, 8, 8), 2, F64, 4e-3, True), ((8, 8, 16), 3, F64, 2e-3, True), ((16, 16, 64), 1, F64, 1e-3, True),
         ((16, 8, 512), 3, F64, 1e-4, True), ((32, 16, 32), 4, F64, 1e-3, True), ((16, 64, 16), 3, F64, 1e-3, True),
         ((32, 32, 128), 3, F64, 5e-4, True), ((8, 128, 32), 4, F64, 5e-4, True), ((128, 8, 64), 2, F64, 5e-4, True),
         ((32, 64, 128), 2, F64, 1e-3, True), ((64, 128, 16), 3, F64, 5e-4, True), ((128, 64, 8), 1, F64, 5e-4, True),
         ((64, 64, 8), 3, FB, 5e-4, True), ((128, 64, 32), 2, F32, 5e-4, True), ((32, 64, 16), 3, FB, 5e-4, False),
         ((128, 128, 8), 2, F64, 5e-4, False), ((8, 256, 8), 2, FB, 5e-4, False)]


def points(H):
    n = H.shape[0]
    return np.moveaxis(H.reshape(n, n, -1), -1, 0)


@pytest.mark.parametrize("grid,n,prec,tau,served", CASES)
def test_plane_pass(grid, n, prec, tau, served):
    import torch
    from paper_1711_01365_amd import mbo
    dt = torch.float64 if prec == F64 else torch.float32
    u, e = (2.0 ** -53, 1e-13) if prec == F64 else (2.0 ** -24, 2e-6)
    A = np.stack([inputs.normal_field(n, grid, 51), inputs.uniform_field(n, grid, 52)])
    t = torch.tensor(A, dtype=dt, device="cuda")
    A = t.double().cpu().numpy()
    pb = mbo.Plan(grid, n, tau, precision=prec, batch=2)
    pg = mbo.Plan(grid, n, tau, precision=prec, batch=2)
    pg.set_path(mbo.PATH_GENERIC)
    assert (pb.path()[0] != mbo.PATH_GENERIC) == served
    # diffusion
    H = pb.diffuse(t).double().cpu().numpy()
    for b in range(2):
        ref, _ = oracle.heat(A[b].reshape((n * n,) + grid), tau, 3)
        assert np.abs(H[b] - ref.reshape(A[b].shape)).max() <= e
    # steps
    for _ in range(3):
        Hg = pg.diffuse(t).double().cpu().numpy()
        nb, ng = pb.step(t), pg.step(t)
        x = t.clone()
        lb = pb.iterate(x, 1)
        assert torch.equal(x, nb)  # a step reproduces the iterate
        lg = pg.iterate(t.clone(), 1)
        for b in range(2):
            s = np.linalg.svd(points(Hg[b]), compute_uv=False)
            gap = s[:, -2] + s[:, -1] if n > 1 else 2 * s[:, 0]
            cof = np.sqrt(sum(np.prod(np.delete(s, j, axis=1), axis=1) ** 2 for j in range(n)))
            ok = np.prod(s, axis=1) > 2 * n * 2 * (e + 8 * u) * cof
            err = np.abs(points((nb - ng)[b].double().cpu().numpy())).max(axis=(1, 2))
            assert np.all(err[ok] <= np.maximum(32 * u, 4 * (2 * e + 8 * u) / gap[ok]))
            Eb, Eg = lb["energy"][b], lg["energy"][b]
            noise = 8 * n * 2 * u / tau
            assert abs(Eb[0] - Eg[0]) <= (1e-12 if prec == F64 else 1e-5) * abs(Eg[0]) + noise
        t = ng
    # the logs, and the same iterates from a replayed graph
    runs = []
    for _ in range(3):
        x = t.clone()
        lb = pb.iterate(x, 4)
        runs.append((x, lb["energy"].copy(), lb["flips"].copy()))
    for r in runs[1:]:
        assert torch.equal(r[0], runs[0][0])
        assert np.array_equal(r[1], runs[0][1]) and np.array_equal(r[2], runs[0][2])
    pb.close()
    pg.close()
