"""Demons on levels of more than 2^24 pixels, whose pixel indices an FP32
number does not hold: one iteration from a zero field against the formula in
FP64 with torch, and the kernels of several iterations against one iteration
per launch bit for bit.  Needs an MI355X.

Bar of one iteration: reference, test and gradient differ by at most
d = 4 x 2^-24 max|image| from the FP64 ones (normalisation and one difference
each), and du = a g / (a^2 + |g|^2) moves by at most 1 / sqrt(a^2 + |g|^2) for
each of the three, so a pixel's bar is 3 d / sqrt(den) plus 8 x 2^-24 of its own
arithmetic (|du| <= 1/2), where sqrt(den) is above 1e-3 max|image|; elsewhere
the full range, 1.  The smoothing averages the bar as it averages du, and adds
16 roundings of at most 2^-25 each."""
import math

import pytest
import torch
import torch.nn.functional as F

pytestmark = pytest.mark.gpu

SHAPES = [(4100, 4100), (16384, 1028)]


@pytest.fixture(scope="module")
def E():
    from paper_1907_05993_amd import ebsd
    ebsd.lib()
    return ebsd


def images(H, W):
    g = torch.Generator(device="cuda").manual_seed(H + W)
    return [torch.rand(1, H, W, generator=g, device="cuda") for _ in range(2)]


def call(E, H, W, iters, sigma, tol=0.0, fused=0, rule=True):
    refs, tests = images(H, W)
    reg = E.Registrar(E.Params(levels=1, iters=(iters,), sigma_px=sigma, tol_px=tol, roi_size=32, n_roi=5,
                               roi_radius_frac=0.002, second_pass=0))
    reg.set_resident(rule)
    if fused:
        reg.set_fused_height(H, W, fused)
    out = reg.register(refs, tests)
    torch.cuda.synchronize()
    field, it = out["field"].clone(), out["iters"].clone()
    reg.close()
    return field, it


def smooth(v, sigma):
    r = int(math.floor(3 * sigma + 0.5))
    if r == 0:
        return v
    w = torch.exp(-torch.arange(-r, r + 1, dtype=torch.float64) ** 2 / (2 * sigma * sigma))
    w = (w / w.sum()).tolist()
    for dim, pad in ((-1, (r, r, 0, 0)), (-2, (0, 0, r, r))):
        p = F.pad(v[None], pad, mode="replicate")[0]
        v = sum(wj * p.narrow(dim, j, v.shape[dim]) for j, wj in enumerate(w))
    return v


def one_iteration(H, W, sigma):
    R, T = [((x := i[0].double()) - x.mean()) / x.std(unbiased=False) for i in images(H, W)]
    M = float(torch.maximum(R.abs().max(), T.abs().max()))
    gx, gy = torch.empty_like(R), torch.empty_like(R)
    gx[:, 1:-1] = (R[:, 2:] - R[:, :-2]) / 2
    gx[:, 0], gx[:, -1] = R[:, 1] - R[:, 0], R[:, -1] - R[:, -2]
    gy[1:-1] = (R[2:] - R[:-2]) / 2
    gy[0], gy[-1] = R[1] - R[0], R[-1] - R[-2]
    a = R - T
    den = a * a + gx * gx + gy * gy
    q = a / den
    root = den.sqrt()
    eps = 2.0 ** -24
    bar = torch.where(root > 1e-3 * M, 3 * 4 * eps * M / root + 8 * eps, torch.ones_like(root))
    return (torch.stack([smooth(q * gx, sigma), smooth(q * gy, sigma)]), smooth(bar, sigma) + 16 * eps / 2)


@pytest.mark.parametrize("H,W", SHAPES)
@pytest.mark.parametrize("sigma", [0.0, 1.0])
def test_one_iteration_of_a_large_level(E, H, W, sigma):
    print("case: one iteration", H, W, sigma, flush=True)
    want, bar = one_iteration(H, W, sigma)
    for kw in ({}, {"rule": False}, {"rule": False, "fused": 32}):
        got, _ = call(E, H, W, 1, sigma, **kw)
        d = (got[0].double() - want).abs()
        print("  ", kw, "max |d|", float(d.max()), "largest of its bar", float((d / bar).max()), flush=True)
        assert bool((d <= bar).all()), kw


@pytest.mark.parametrize("H,W", SHAPES)
@pytest.mark.parametrize("sigma,tol", [(0.0, 0.0), (1.0, 0.0), (1.0, 0.3)])
def test_several_iterations_of_a_large_level(E, H, W, sigma, tol):
    print("case: several iterations", H, W, sigma, tol, flush=True)
    want, its = call(E, H, W, 6, sigma, tol, rule=False)
    for kw in ({}, {"fused": 32}):
        got, it = call(E, H, W, 6, sigma, tol, **kw)
        assert torch.equal(it, its) and torch.equal(got, want), kw
