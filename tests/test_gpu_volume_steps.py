"""Steps of the volume-preserving iteration that a longer run takes: the field
between two steps of one call is the field that a call of one step returns.

The fields hold, point by point in a checkerboard, the rotations by +phi and -phi
of the last two axes (times a reflection in part of the domain).  Diffusion leaves
their mean, so the two smallest singular values are |cos phi| each, from 0 (a strip
with phi = pi/2) to 1: the points that the selection moves have rank n - 2 up to
rounding, where the polar factor and the vectors of the smallest singular value are
any that rounding makes them, and the moved point has to be formed from the very
factor that the others of its row were.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

F64, F32, FB = 0, 1, 2


def checkered(n, grid):
    """The field above; det -1 in a disc, which diffusion shrinks."""
    i, j = np.meshgrid(np.arange(grid[0]), np.arange(grid[1]), indexing="ij")
    x, y = i / grid[0], j / grid[1]
    phi = 0.5 * np.pi * np.minimum(1.0, 0.4 + 1.2 * np.sin(np.pi * x) ** 2)
    phi = np.where((i + j) % 2 == 0, phi, -phi)
    A = np.zeros((n, n) + tuple(grid))
    for k in range(n - 2):
        A[k, k] = 1.0
    side = np.where((x - 0.3) ** 2 + (y - 0.55) ** 2 > 0.08, 1.0, -1.0)
    A[n - 2, n - 2], A[n - 2, n - 1] = np.cos(phi), -np.sin(phi) * side
    A[n - 1, n - 2], A[n - 1, n - 1] = np.sin(phi), np.cos(phi) * side
    return A


def diffused(A, tau):
    k = [np.fft.fftfreq(N, 1.0 / N) for N in A.shape[2:]]
    s = np.exp(-4 * np.pi ** 2 * tau * (k[0][:, None] ** 2 + k[1][None, :] ** 2))
    return np.real(np.fft.ifft2(np.fft.fft2(A) * s))


def points(A):
    return np.moveaxis(A.reshape(A.shape[0], A.shape[1], -1), -1, 0)


@pytest.mark.parametrize("n,grid,prec", [(2, (64, 64), FB), (2, (64, 64), F64), (3, (64, 64), F32), (3, (64, 64), FB),
                                         (3, (128, 512), FB), (3, (64, 1024), FB), (3, (64, 64), F64), (4, (64, 64), F32),
                                         (4, (64, 256), FB), (4, (64, 64), F64)])
def test_two_steps_are_one_and_one(n, grid, prec):
    import torch
    from paper_1711_01365_amd import mbo
    dt = torch.float64 if prec == F64 else torch.float32
    tau = 2.0 / 64 ** 2
    p = mbo.Plan(grid, n, tau, precision=prec)
    assert p.path()[0] != mbo.PATH_GENERIC
    A0 = torch.tensor(checkered(n, grid)[None], dtype=dt, device="cuda")
    X = A0.clone()
    two = p.iterate_volume(X, 2, None)
    Y = A0.clone()
    one = p.iterate_volume(Y, 1, None)
    A1 = Y.double().cpu().numpy()[0]
    more = p.iterate_volume(Y, 1, None)
    p.close()

    # the first step moved points off the side of their determinant
    B = points(diffused(A0.double().cpu().numpy()[0], tau))
    moved = (np.sign(np.linalg.det(points(A1))) != np.sign(np.linalg.det(B))).sum()
    assert moved >= 10
    err = np.abs(np.matmul(np.moveaxis(points(A1), 1, 2), points(A1)) - np.eye(n)).max()
    # a few roundings per entry
    assert err <= (2e-15 if prec == F64 else 1e-6) * n * n

    # Two runs of one step from fields equal to rounding: each within 1e-5 (1e-11 in
    # double) of the exact step where sigma_{n-1} - sigma_n >= 0.1 (the condition of the
    # candidate of the other determinant; the sum is that of the polar factor), on the same side
    # away from the cut.
    tol = 2e-11 if prec == F64 else 2e-5
    assert two["flips"][0][0] == one["flips"][0][0]
    assert np.array_equal(two["n_plus"], more["n_plus"])
    e = np.abs(two["energy"][0] - np.append(one["energy"][0][:1], more["energy"][0]))
    assert e.max() <= tol * np.abs(two["energy"]).max()
    H = points(diffused(A1, tau))
    s = np.linalg.svd(H, compute_uv=False)
    x, y = points(X.double().cpu().numpy()[0]), points(Y.double().cpu().numpy()[0])
    same = np.sign(np.linalg.det(x)) == np.sign(np.linalg.det(y))
    assert (~same).sum() <= 0.01 * same.size
    good = same & (s[:, -2] - s[:, -1] >= 0.1)
    assert good.sum() >= 0.25 * good.size
    assert np.abs(x - y)[good].max() <= tol


def flipped(n, grid, share, seed):
    """Smooth rotations near the identity, the last column negated at a random share of
    the points: most of them change side in the first step, in every row."""
    rng = np.random.default_rng(seed)
    X, Y = np.meshgrid(np.arange(grid[0]) / grid[0], np.arange(grid[1]) / grid[1], indexing="ij")
    S = np.zeros(tuple(grid) + (n, n))
    for i in range(n):
        for j in range(i):
            p, q = rng.uniform(size=2)
            S[..., i, j] = 0.3 * np.sin(2 * np.pi * (X + p)) + 0.3 * np.cos(2 * np.pi * (Y + q))
            S[..., j, i] = -S[..., i, j]
    Q = np.linalg.solve(np.eye(n) + S, np.eye(n) - S)
    Q[..., -1] *= np.where(rng.random(tuple(grid)) < share, -1.0, 1.0)[..., None]
    return np.ascontiguousarray(np.moveaxis(Q, (2, 3), (0, 1)))


# every row length of volume_redo, whole lines and parts, with all and with the kept modes
@pytest.mark.parametrize("n,L,prec", [(n, L, F64) for n in (1, 2, 3, 4) for L in (8, 16, 32, 64, 128, 256, 512, 1024)] +
                         [(1, 2048, F64), (2, 2048, F64)] +
                         [(n, L, FB) for n in (1, 2, 3, 4) for L in (8, 64, 512, 1024, 2048)])
def test_rows_transformed_again(n, L, prec):
    import torch
    from paper_1711_01365_amd import mbo
    dt = torch.float64 if prec == F64 else torch.float32
    grid = (64, L)
    tau = (6.0 / max(grid)) ** 2 / 2
    A0 = torch.tensor(np.stack([flipped(n, grid, 0.3, 5), flipped(n, grid, 0.6, 6)]), dtype=dt, device="cuda")
    p = mbo.Plan(grid, n, tau, precision=prec, batch=2)
    assert p.path()[0] != mbo.PATH_GENERIC
    X, Y = A0.clone(), A0.clone()
    two = p.iterate_volume(X, 2, None)
    one = p.iterate_volume(Y, 1, None)
    more = p.iterate_volume(Y, 1, None)
    # more than the 64 per row_fast workgroup that are added by direct sums
    assert one["flips"].min() > 0.2 * 64 * L
    tol = 2e-11 if prec == F64 else 2e-5
    e = np.abs(two["energy"] - np.concatenate([one["energy"][:, :1], more["energy"]], axis=1))
    assert e.max() <= tol * np.abs(two["energy"]).max()
    assert np.array_equal(two["n_plus"], more["n_plus"])
    x, y = X.double().cpu().numpy(), Y.double().cpu().numpy()
    if prec == F64:
        assert np.array_equal(two["flips"][:, 1], more["flips"][:, 0])
        p.set_path(mbo.PATH_GENERIC)
        Z = A0.clone()
        ref = p.iterate_volume(Z, 2, None)
        assert np.array_equal(two["flips"], ref["flips"])
        z = Z.cpu().numpy()
    p.close()
    for b in range(2):
        u, v = points(x[b]), points(y[b])
        same = np.sign(np.linalg.det(u)) == np.sign(np.linalg.det(v))
        assert (~same).sum() <= 0.01 * same.size
        s = np.linalg.svd(points(diffused(one_step(A0[b], tau, prec, n, grid), tau)), compute_uv=False)
        good = same & ((s[:, -2] - s[:, -1] >= 0.1) if n > 1 else (s[:, 0] >= 0.1))
        assert np.abs(u - v)[good].max() <= tol
        if prec == F64:
            assert np.abs(u - points(z[b]))[good].max() <= 1e-10


def one_step(A, tau, prec, n, grid):
    from paper_1711_01365_amd import mbo
    p = mbo.Plan(grid, n, tau, precision=prec)
    X = A[None].clone()
    p.iterate_volume(X, 1, None)
    p.close()
    return X.double().cpu().numpy()[0]
