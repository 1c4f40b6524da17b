"""The volume-preserving iteration through the band-limited passes against the
general passes (mbo_plan_set_path GENERIC), which test_gpu_volume.py checks
against the oracle.

Shapes: the shortest and longest rows and columns of the passes, several rows
per workgroup, rows beyond 512 points, n = 1..4, two fields.  The smooth fields
have domains of both determinants, so every step reassigns points near the cut.
The constant field with the caller's own volume makes Delta E equal along whole
rows from the second step on (exactly: a constant row has one nonzero mode), so
the cut falls inside a run of equal values and goes by index, at every kind of
rank (first, last, inside, none, all).

Double: both paths solve the same step to rounding, 1e-10 as in
test_gpu_volume.py; flips and counts equal.  Float: each path is within 1e-5 of
the FP64 step where sigma_{n-1} + sigma_n >= 0.1 (these fields), so two of them
within 2e-5 for one step.
"""
import numpy as np
import pytest

import oracle
from paper_1711_01365_amd import inputs

pytestmark = pytest.mark.gpu

F64, F32, FB = 0, 1, 2
P_OFF = 2  # percent of the points


def domains(n, grid, seed):
    """Smooth rotations near the identity, determinant -1 in a disc and a strip."""
    X, Y = np.meshgrid(np.arange(grid[0]) / grid[0], np.arange(grid[1]) / grid[1], indexing="ij")
    rng = np.random.default_rng(seed)
    S = np.zeros(grid + (n, n))
    for i in range(n):
        for j in range(i):
            p, q = rng.uniform(size=2)
            S[..., i, j] = 0.3 * np.sin(2 * np.pi * (X + p)) + 0.3 * np.cos(2 * np.pi * (Y + q))
            S[..., j, i] = -S[..., i, j]
    Id = np.eye(n)
    Q = np.linalg.solve(Id + S, Id - S)
    disc = (np.sin(np.pi * (X - 0.31)) ** 2 + np.sin(np.pi * (Y - 0.57)) ** 2) / np.pi ** 2 < 0.02
    strip = np.abs(X - 0.71) < 0.07 + 0.03 * np.sin(2 * np.pi * Y)
    Q[disc | strip, :, -1] *= -1
    return np.ascontiguousarray(np.moveaxis(Q, (2, 3), (0, 1)))


def both(A, tau, prec, K, n_plus):
    import torch
    from paper_1711_01365_amd import mbo
    dt = torch.float64 if prec == F64 else torch.float32
    B, n, grid = A.shape[0], A.shape[1], A.shape[3:]
    out = []
    for path in (mbo.PATH_BANDED, mbo.PATH_GENERIC):
        p = mbo.Plan(grid, n, tau, precision=prec, batch=B)
        p.set_path(path)
        assert (p.path()[0] == mbo.PATH_GENERIC) == (path == mbo.PATH_GENERIC)
        runs = []
        for _ in range(2):  # the second pass replays the captured graph
            X = torch.tensor(A, dtype=dt, device="cuda")
            logs = p.iterate_volume(X, K, n_plus)
            runs.append((X.double().cpu().numpy(), logs))
        assert np.array_equal(runs[0][0], runs[1][0])
        out.append(runs[1])
        p.close()
    return out


def check(got, ref, tol, etol):
    assert np.abs(got[0] - ref[0]).max() <= tol
    assert np.array_equal(got[1]["flips"], ref[1]["flips"])
    assert np.array_equal(got[1]["n_plus"], ref[1]["n_plus"])
    assert np.abs(got[1]["energy"] - ref[1]["energy"]).max() <= etol * np.abs(ref[1]["energy"]).max()


@pytest.mark.parametrize("n,grid", [(1, (64, 64)), (2, (64, 8)), (2, (2048, 16)), (2, (128, 1024)), (2, (64, 2048)),
                                    (3, (64, 32)), (3, (128, 512)), (3, (64, 1024)), (4, (64, 64)), (4, (64, 256))])
@pytest.mark.parametrize("given", [False, True])
def test_f64(n, grid, given):
    A = np.stack([domains(n, grid, 5 + b) for b in range(2)])
    # the caller's own volume: a little off that of the field (far inside a domain
    # of n = 2 rotations sigma_1 = sigma_2 to rounding, and the closest reflection
    # is any)
    near = np.array([(oracle.det_sign(a) > 0).sum() for a in A])
    n_plus = near + np.array([P_OFF, -P_OFF]) * (grid[0] * grid[1]) // 100 if given else None
    got, ref = both(A, 8.0 / min(max(grid), 256) ** 2, F64, 4, n_plus)
    check(got, ref, 1e-10, 1e-9)


@pytest.mark.parametrize("n,grid,prec", [(2, (64, 16), FB), (3, (64, 64), F32), (3, (256, 512), FB), (3, (64, 2048), FB),
                                         (4, (128, 128), FB)])
def test_f32_one_step(n, grid, prec):
    A = domains(n, grid, 9)[None].astype(np.float32)
    got, ref = both(A, 8.0 / min(max(grid), 256) ** 2, prec, 1, None)
    check(got, ref, 2e-5, 1e-5)


@pytest.mark.parametrize("n,grid", [(2, (64, 64)), (3, (64, 16)), (3, (64, 512))])
@pytest.mark.parametrize("count", [0, 1, 37, "third", "all but one", "all"])
def test_equal_values(n, grid, count):
    P = grid[0] * grid[1]
    n_plus = {"third": P // 3 + 5, "all but one": P - 1, "all": P}.get(count, count)
    A = np.zeros((1, n, n) + grid)
    for i in range(n):
        A[:, i, i] = 1.0
    got, ref = both(A, 2e-3, F64, 3, n_plus)
    assert int((np.linalg.det(np.moveaxis(got[0][0].reshape(n, n, -1), -1, 0)) > 0).sum()) == n_plus
    check(got, ref, 1e-10, 1e-9)
