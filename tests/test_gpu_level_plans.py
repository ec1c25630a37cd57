"""Every kernel that a pyramid level can run on, forced with ebsd_set_level_plan,
against one iteration per launch: fields, iteration counts and status equal bit
for bit at all smoothing radii, at the sizes where strips, segments and regions
can go wrong, with and without a tolerance, and with the host ending the issue of
launches early.  Needs an MI355X."""
import pytest
import torch

pytestmark = pytest.mark.gpu

SIGMAS = [0.4, 0.7, 1.0, 1.3]  # radius 1 .. 4


@pytest.fixture(scope="module")
def E():
    from paper_1907_05993_amd import ebsd
    ebsd.lib()
    return ebsd


def pairs(E, n, H, W, deg=5.0):
    from paper_1907_05993_amd import synth as S
    return E.gen_pairs([S.make_spec(86, i, H, W, mis_deg=(0.0, deg)) for i in range(n)], labels=False)[:2]


def call(E, refs, tests, plans, resident=False, chunk=0, levels=1, **kw):
    """plans: {(h, w): (kind, rows)}, {} for one iteration per launch."""
    W = refs.shape[2]
    reg = E.Registrar(E.Params(levels=levels, roi_size=32, n_roi=5, roi_radius_frac=0.3 / W, second_pass=0, **kw))
    reg.set_resident(resident)
    reg.set_gating(chunk)
    for (h, w), (kind, rows) in plans.items():
        reg.set_level_plan(h, w, kind, rows)
    out = reg.register(refs, tests)
    torch.cuda.synchronize()
    counts = reg.launch_counts()
    reg.close()
    return {k: out[k].clone() for k in ("field", "iters", "status")}, counts


def equal(a, b, what):
    for k in a:
        assert torch.equal(a[k], b[k]), (k, what)


def launches(kind, sigma, rows, iters):
    per = {"rows": 1, "rows2": 2, "march": 2, "regions": 3 if sigma == 1.3 and rows < 80 else 4}[kind]
    return -(-iters // per)


def check(E, refs, tests, sigma, plan, runs):
    H, W = refs.shape[1:]
    for iters, tol in runs:
        a, _ = call(E, refs, tests, {}, iters=(iters,), sigma_px=sigma, tol_px=tol)
        b, (issued, planned) = call(E, refs, tests, {(H, W): plan}, iters=(iters,), sigma_px=sigma, tol_px=tol)
        equal(a, b, (plan, iters, tol))
        assert issued[0] == planned[0]
        want = launches(plan[0], sigma, plan[1], iters)
        assert planned[0] - want == 0 if tol == 0.0 else planned[0] - want in (0, 1)


RUNS = ((1, 0.0), (2, 0.0), (9, 0.0), (12, 0.0), (40, 0.2), (31, 0.05), (8, 0.02))


# two columns per lane (up to 128 px) and four; lanes past the last column; two and
# three segments; strips of the least height, of heights that leave a last one of a row
# or two, and one strip
# (four columns per lane up to radius 3)
@pytest.mark.parametrize("sigma,n,H,W", [(s, *c) for s in SIGMAS for c in
                                         [(3, 66, 66), (2, 90, 126), (2, 82, 128), (2, 73, 132), (2, 50, 260),
                                          (1, 65, 500)] if s < 1.3 or c[2] <= 128])
def test_march(E, n, H, W, sigma):
    print("case: march", n, H, W, sigma, flush=True)
    refs, tests = pairs(E, n, H, W)
    for rows in (9, 16, H - 1, H):
        check(E, refs, tests, sigma, ("march", rows), RUNS if rows in (9, 16) else RUNS[2:5])


# regions of 32, 64 and 80 rows: a column or row past a tile, one region only, several
# across, a last tile of one row or column
@pytest.mark.parametrize("n,H,W", [(3, 65, 66), (2, 72, 41), (1, 41, 129), (2, 100, 257), (2, 150, 150)])
@pytest.mark.parametrize("rows", [32, 64, 80])
@pytest.mark.parametrize("sigma", SIGMAS)
def test_regions(E, n, H, W, rows, sigma):
    print("case: regions", n, H, W, rows, sigma, flush=True)
    refs, tests = pairs(E, n, H, W)
    check(E, refs, tests, sigma, ("regions", rows), RUNS)


# every level of flat patterns, down to 4 rows, on one kind: strips and regions that
# hold both the first and the last row, with fewer rows than the smoothing has taps
@pytest.mark.parametrize("kind,rows", [("march", 9), ("march", 16), ("regions", 32), ("regions", 64), ("regions", 80),
                                       ("rows2", 16)])
@pytest.mark.parametrize("sigma", SIGMAS)
@pytest.mark.parametrize("H,W,levels", [(32, 1024, 4), (40, 480, 3), (32, 256, 4)])
def test_flat_levels(E, kind, rows, sigma, H, W, levels):
    if kind == "march" and sigma == 1.3:
        W, levels = 128, min(levels, 4)  # two columns per lane only
    print("case: flat levels", kind, rows, sigma, H, W, levels, flush=True)
    refs, tests = pairs(E, 2, H, W)
    sizes = [E.level_size(H, W, l) for l in range(levels)]
    for iters, tol in ((1, 0.0), (5, 0.0), (12, 0.0), (20, 0.1), (15, 0.01)):
        kw = dict(iters=(iters,) * levels, sigma_px=sigma, tol_px=tol, levels=levels)
        a, _ = call(E, refs, tests, {}, **kw)
        b, _ = call(E, refs, tests, {s: (kind, rows) for s in sizes}, **kw)
        equal(a, b, (iters, tol))


# the host stops issuing launches once no pair iterates: chunks of one and three launches
@pytest.mark.parametrize("sigma,kind,rows,H,W", [(s, *c) for s in (0.7, 1.0, 1.3) for c in
                                                 [("march", 16, 96, 128), ("march", 32, 96, 256),
                                                  ("regions", 32, 96, 128), ("regions", 64, 96, 256),
                                                  ("regions", 80, 96, 256), ("rows2", 16, 96, 256)]
                                                 if s < 1.3 or c[0] != "march" or c[3] <= 128])
def test_gated_levels(E, kind, rows, H, W, sigma):
    print("case: gated", kind, rows, H, W, sigma, flush=True)
    refs, tests = pairs(E, 5, H, W, deg=2.0)
    for iters, tol in ((150, 0.1), (150, 0.03), (10, 0.05)):
        kw = dict(iters=(iters,), sigma_px=sigma, tol_px=tol)
        a, _ = call(E, refs, tests, {}, **kw)
        _, (all_issued, _) = call(E, refs, tests, {(H, W): (kind, rows)}, **kw)
        for chunk in (1, 3):
            b, (issued, planned) = call(E, refs, tests, {(H, W): (kind, rows)}, chunk=chunk, **kw)
            equal(a, b, (iters, tol, chunk))
            assert planned[0] == all_issued[0] >= issued[0]
            if int(a["iters"].max()) < 50 and iters == 150:
                assert issued[0] < planned[0]
