"""The Gauss-Newton iteration of Eq. (3) runs to a step below 1e-14 also where it
converges slowly: shift sets of 5 to 7 ROIs with residuals of tens of pixels, whose
steps shrink by a factor of at most 0.77 each, against the minimiser in extended
precision.  Needs an MI355X.

Bar: behind a step below 1e-14 at most 1e-14 x 0.77 / (1 - 0.77) = 3.4e-14 is left
(a stop at a step of 1e-13 leaves ten times that); the normalisation to det 1
scales F by less than 2 here, and rounding of the FP64 normal equations adds less than
3e-14: 1e-13."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

PCS = (127.5, 127.5, 179.2)
SEEDS = [14042, 32656, 1297, 18605, 31147, 46883, 24293, 48164, 1484, 22759, 51086, 16065]


@pytest.fixture(scope="module")
def E():
    from paper_1907_05993_amd import ebsd
    ebsd.lib()
    return ebsd


def shift_set(seed):
    """(centres, shifts) of 5 + seed % 3 ROIs."""
    rng = np.random.default_rng(seed)
    nr = 5 + seed % 3
    a = 2 * np.pi * np.arange(nr) / nr
    c = np.stack([np.round(PCS[0] + 76.8 * np.cos(a)) + 0.5, np.round(PCS[1] + 76.8 * np.sin(a)) + 0.5], 1)
    c[0] = PCS[0]
    return c, rng.normal(size=(nr, 2)).astype(np.float32) * np.float32(40)


def solve_linear(A, b):
    A, b = A.copy(), b.copy()
    n = len(b)
    for k in range(n):
        p = k + int(np.abs(A[k:, k]).argmax())
        A[[k, p]], b[[k, p]] = A[[p, k]], b[[p, k]]
        for i in range(k + 1, n):
            m = A[i, k] / A[k, k]
            A[i, k:] -= m * A[k, k:]
            b[i] -= m * b[k]
    x = np.zeros_like(b)
    for k in range(n - 1, -1, -1):
        x[k] = (b[k] - A[k, k + 1:] @ x[k + 1:]) / A[k, k]
    return x


def minimiser(c, q, stop=1e-17, dtype=np.longdouble):
    """F (det 1) by the same start and iteration, to a step below `stop`."""
    r = ((c - np.array(PCS[:2])) / PCS[2]).astype(dtype)
    p = r + q.astype(dtype) / dtype(PCS[2])
    z, o = np.zeros(len(r), dtype), np.ones(len(r), dtype)
    a = np.stack([r[:, 0], r[:, 1], o, z, z, z, -p[:, 0] * r[:, 0], -p[:, 0] * r[:, 1]], 1)
    b = np.stack([z, z, z, r[:, 0], r[:, 1], o, -p[:, 1] * r[:, 0], -p[:, 1] * r[:, 1]], 1)
    f = solve_linear(a.T @ a + b.T @ b, a.T @ p[:, 0] + b.T @ p[:, 1])
    for _ in range(400):
        i = 1 / (f[6] * r[:, 0] + f[7] * r[:, 1] + 1)
        u, v = (f[0] * r[:, 0] + f[1] * r[:, 1] + f[2]) * i, (f[3] * r[:, 0] + f[4] * r[:, 1] + f[5]) * i
        ju = np.stack([r[:, 0] * i, r[:, 1] * i, i, z, z, z, -u * r[:, 0] * i, -u * r[:, 1] * i], 1)
        jv = np.stack([z, z, z, r[:, 0] * i, r[:, 1] * i, i, -v * r[:, 0] * i, -v * r[:, 1] * i], 1)
        d = solve_linear(ju.T @ ju + jv.T @ jv, ju.T @ (u - p[:, 0]) + jv.T @ (v - p[:, 1]))
        f = f - d
        if np.sqrt(d @ d) < stop:
            break
    F = np.append(f, dtype(1)).reshape(3, 3)
    det = F[0, 0] * (F[1, 1] * F[2, 2] - F[1, 2] * F[2, 1]) - F[0, 1] * (F[1, 0] * F[2, 2] - F[1, 2] * F[2, 0]) + \
        F[0, 2] * (F[1, 0] * F[2, 1] - F[1, 1] * F[2, 0])
    return F / np.cbrt(det)


@pytest.mark.parametrize("seed", SEEDS)
def test_slow_fits_run_to_the_stated_step(E, seed):
    c, q = shift_set(seed)
    want = minimiser(c, q)
    print("case: slow fit", seed, len(q), flush=True)
    F = E.stage_solve(torch.from_numpy(q[None].repeat(3, 0)).cuda(), torch.from_numpy(c[:, 0].copy()),
                      torch.from_numpy(c[:, 1].copy()), PCS)[0]
    torch.cuda.synchronize()
    d = np.abs(F.cpu().numpy().reshape(3, 3, 3) - want[None]).max()
    print("  max |dF| %.2e" % d)
    assert d <= 1e-13
