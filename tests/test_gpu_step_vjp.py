"""mbo_step_vjp through the band-limited passes, against the FP64 oracle's chain
(heat, projection VJP, heat; <G~, d/dtau heat A> for the tau term).

Shapes: the shortest and longest rows and columns of the passes, rows shorter
than a workgroup (several rows per workgroup), rows of more than 512 points,
every mode kept (large tau / N would drop some; 8-point rows keep all), two
fields.  Fields: smooth orthogonal ones, and diag(1, 1, s) with s a sine of
small amplitude, a quarter step off its zeros: points below and above the double
threshold (at s = 0 itself the projection jumps, and the sign of a float
rounding decides on every path).

Tolerance: a point's VJP is |G| / gap large and moves by |G| d / gap^2 when its
input moves by d (gap = sigma_{n-1} + sigma_n), as in test_gpu_adjoint.py: 64 u
(1 + |G| (1/gap + 1/gap^2)), here with the largest |G| and smallest gap of the
field because the last heat step mixes the points.  The tau term sums G~ dA/dtau: that
bound on every G~ times the sum of |dA/dtau|, and 64 u of the largest |dA/dtau|
times the sum of |G~|.
"""
import numpy as np
import pytest

import oracle
from paper_1711_01365_amd import inputs

pytestmark = pytest.mark.gpu

F64, F32, FB = 0, 1, 2


def heat(A, tau):
    n, grid = A.shape[0], A.shape[2:]
    return oracle.heat(A.reshape((n * n,) + grid), tau, 2)[0].reshape(A.shape)


def smooth_field(n, grid, seed):
    return oracle.project(heat(inputs.normal_field(n, grid, seed), 4e-3))[0]


def thin_field(n, grid, amp):
    A = np.zeros((n, n) + grid)
    for i in range(n - 1):
        A[i, i] = 1.0
    x = (np.arange(grid[0])[:, None] + 0.25) / grid[0] + np.zeros(grid)
    A[n - 1, n - 1] = amp * np.sin(2 * np.pi * x)
    return A


CASES = [(n, g, p, "smooth") for n, g, p in
         [(2, (64, 8), F64), (2, (64, 8), FB), (2, (256, 1024), F32), (2, (128, 2048), FB), (2, (64, 1024), F64),
          (3, (64, 8), F32), (3, (64, 64), FB), (3, (128, 16), F64), (3, (512, 128), FB), (3, (64, 512), F64),
          (3, (128, 1024), FB), (3, (64, 2048), F32), (3, (2048, 32), F64), (3, (1024, 64), FB),
          (4, (64, 64), FB), (4, (128, 256), F64), (1, (64, 64), FB)]]
CASES += [(n, (64, 64), p, "thin") for n in (2, 3, 4) for p in (F64, F32, FB)]


@pytest.mark.parametrize("n,grid,prec,kind", CASES)
def test_step_vjp_banded(n, grid, prec, kind):
    import torch
    from paper_1711_01365_amd import mbo
    tau = 1e-3
    dt, npdt = (torch.float64, np.float64) if prec == F64 else (torch.float32, np.float32)
    u = 2.0 ** -53 if prec == F64 else 2.0 ** -24
    B = 2 if kind == "smooth" else 1
    A = [smooth_field(n, grid, 11 + b) if kind == "smooth" else thin_field(n, grid, 5e-3) for b in range(B)]
    A = [a.astype(npdt).astype(np.float64) for a in A]
    G = [inputs.normal_field(n, grid, 31 + b).astype(npdt).astype(np.float64) for b in range(B)]
    p = mbo.Plan(grid, n, tau, precision=prec, batch=B)
    assert p.path()[0] != mbo.PATH_GENERIC
    Ad = torch.tensor(np.stack(A), dtype=dt, device="cuda")
    Gd = torch.tensor(np.stack(G), dtype=dt, device="cuda")
    G2 = Gd.clone()
    dtau = torch.zeros(B, dtype=torch.float64, device="cuda")
    dtau += 1.0  # the term is added
    p.step_vjp(Ad, Gd, dtau)
    p.step_vjp(Ad, G2)  # without the tau term
    got, dtau = Gd.double().cpu().numpy(), dtau.cpu().numpy() - 1.0
    for b in range(B):
        At = heat(A[b], tau)
        if n == 1:
            Gt, worst = np.zeros_like(At), 1.0
        else:
            Gt = oracle.project_vjp(At, G[b])
            s = np.linalg.svd(np.moveaxis(At.reshape(n, n, -1), -1, 0), compute_uv=False)
            gap = (s[:, -2] + s[:, -1]).min()
            worst = np.abs(G[b]).max() * (1 / gap + 1 / gap ** 2)
        ref = heat(Gt, tau)
        dA = oracle.heat_dtau(A[b].reshape((n * n,) + grid), tau, 2).reshape(At.shape)
        bound = 64 * u * (1 + worst)
        err = np.abs(got[b] - ref).max()
        et = abs(dtau[b] - (Gt * dA).sum())
        bound_t = bound * np.abs(dA).sum() + 64 * u * np.abs(Gt).sum() * np.abs(dA).max()
        print("n=%d %s prec=%d %s: err %.2e (bound %.2e), dtau err %.2e (bound %.2e)" % (n, grid, prec, kind, err,
                                                                                      bound, et, bound_t), flush=True)
        assert err <= bound
        assert et <= bound_t
        assert np.abs(G2[b].double().cpu().numpy() - got[b]).max() <= bound
