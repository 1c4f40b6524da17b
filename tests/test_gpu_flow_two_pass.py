"""The relaxed flows through the two passes of mbo_iterate against the general passes
(mbo_plan_set_path GENERIC), which test_gpu_relaxed.py checks against the oracle.

Shapes: the shortest and longest rows and columns of the passes, several rows per
workgroup, rows beyond 512 points, n = 1..4, two fields, GD-1 and GD-3, one step
and several.  The field is smooth (every sigma_n near 1, the polar factor well
conditioned), eps = inf leaves the implicit diffusion alone.  With r the relative
rounding of one transform pass (about log2 of the points, u each), K steps differ by
at most K (1 + 2 c) r; 64 u K holds that with margin for every shape here.
Non-finite points are refused on both.  n = 4 takes the general passes on every path.
"""
import numpy as np
import pytest

import oracle
from paper_1711_01365_amd import inputs

pytestmark = pytest.mark.gpu

F64, F32, FB = 0, 1, 2
CASES = [((64, 8), 1, F64), ((64, 16), 2, F32), ((128, 64), 3, FB), ((256, 32), 4, FB), ((64, 512), 3, F64),
         ((512, 256), 3, F32), ((64, 1024), 4, F64), ((1024, 16), 4, F64), ((64, 2048), 3, FB), ((2048, 8), 3, F64),
         ((2048, 16), 2, FB), ((64, 2048), 2, F64)]


@pytest.mark.parametrize("grid,n,prec", CASES)
def test_flow_two_pass(grid, n, prec):
    import torch
    from paper_1711_01365_amd import mbo
    dt = torch.float64 if prec == F64 else torch.float32
    u = 2.0 ** -53 if prec == F64 else 2.0 ** -24
    A = np.stack([oracle.heat(np.eye(n)[:, :, None, None] + 0.2 * inputs.uniform_field(n, grid, 60 + b), 1e-3, 2)[0]
                  for b in range(2)])
    A = A.reshape((2, n, n) + grid)
    runs = {}
    for path in (mbo.PATH_BANDED, mbo.PATH_GENERIC):
        p = mbo.Plan(grid, n, 1e-3, precision=prec, batch=2)
        p.set_path(path)
        assert (p.path()[0] == mbo.PATH_GENERIC) == (path == mbo.PATH_GENERIC)
        for kind in (mbo.GD1, mbo.GD3):
            for eps, K in ((0.1, 1), (0.1, 4), (np.inf, 2)):
                outs = []
                for _ in range(2):  # the second replays the captured graph
                    X = torch.tensor(A, dtype=dt, device="cuda")
                    p.relaxed_flow(X, K, kind, eps, 1e-3)
                    outs.append(X.double().cpu().numpy())
                assert np.array_equal(outs[0], outs[1])
                runs.setdefault((kind, eps, K), []).append(outs[1])
        X = torch.tensor(A, dtype=dt, device="cuda")
        X[1, 0, 0, 3, 5] = float("nan")
        with pytest.raises(mbo.MboError):
            p.relaxed_flow(X, 1, mbo.GD1, 0.1, 1e-3)
        p.close()
    for (kind, eps, K), (a, b) in runs.items():
        assert np.abs(a - b).max() <= 64 * u * K * np.abs(b).max(), (kind, eps, K)
