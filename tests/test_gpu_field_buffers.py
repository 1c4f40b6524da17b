"""One plan, several live fields: the captured iterations read the field's pointer from a
device word, so a call on another buffer replays the same graph.  Every call has to
leave the other buffers alone and give what a plan of its own gives, bit for bit,
whatever ran on the plan before."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

F64, F32, FB = 0, 1, 2


def field(n, grid, batch, dt, seed):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn((batch, n, n) + tuple(grid), device="cuda", dtype=dt, generator=g)


@pytest.mark.parametrize("n,grid,prec,batch", [(2, (64, 64), F64, 1), (3, (64, 128), FB, 2), (3, (64, 1024), FB, 1),
                                               (2, (16, 32, 64), F64, 1), (3, (64, 64, 64), F32, 1), (2, (32, 64), F32, 1)])
@pytest.mark.parametrize("call", ["iterate", "volume", "flow"])
def test_alternating_buffers(n, grid, prec, batch, call):
    import torch
    from paper_1711_01365_amd import mbo
    dt = torch.float64 if prec == F64 else torch.float32
    tau = 1e-3

    def run(p, A):
        if call == "iterate":
            return p.iterate(A, 3)
        if call == "volume":
            return p.iterate_volume(A, 3, None)
        p.relaxed_flow(A, 3, mbo.GD1, 0.1, 1e-4)
        return {}

    start = [field(n, grid, batch, dt, s) for s in range(3)]
    ref = []
    for A in start:
        p = mbo.Plan(grid, n, tau, precision=prec, batch=batch)
        X = A.clone()
        logs = run(p, X)
        ref.append((X, logs))
        p.close()
    p = mbo.Plan(grid, n, tau, precision=prec, batch=batch)
    live = [A.clone() for A in start]
    for k in (0, 1, 0, 2, 1, 1, 2, 0):
        live[k].copy_(start[k])
        before = [x.clone() for x in live]
        logs = run(p, live[k])
        # the host's own work and synchronisations between the replays
        junk = [field(n, grid, batch, dt, 9) for _ in range(2)]
        torch.cuda.synchronize()
        for j in range(3):
            assert torch.equal(live[j], ref[j][0] if j == k else before[j])
        for key in ("flips", "energy", "n_plus", "fallbacks"):
            if key in logs:
                assert np.array_equal(logs[key], ref[k][1][key])
        del junk
    p.close()
