"""Several demons iterations per launch by rule (2-D tiles for small batches,
marching wavefronts for larger ones, all iterations of a level at once
without smoothing) against one iteration per launch: fields, iteration counts and status equal bit for bit at the
sizes where the tiling can go wrong.  Needs an MI355X."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def call(E, refs, tests, multi, **kw):
    reg = E.Registrar(E.Params(levels=1, roi_size=32, n_roi=5, roi_radius_frac=0.002, **kw))
    reg.set_resident(multi)
    out = reg.register(refs, tests)
    torch.cuda.synchronize()
    counts = reg.launch_counts()
    reg.close()
    return out, counts


# one column / row past a tile, a last tile of one row or column, several tiles
# across, one region only; 20 pairs of 150 px take the regions of 64 rows (radius 3 and 4)
@pytest.mark.parametrize("n,H,W", [(1, 65, 66), (2, 72, 41), (1, 41, 129), (1, 97, 640), (2, 300, 70), (20, 150, 150)])
@pytest.mark.parametrize("sigma", [0.4, 0.7, 1.0, 1.3])  # radius 1 .. 4
def test_tiles_equal_single_iterations(E, n, H, W, sigma):
    from paper_1907_05993_amd import synth as S
    print("case: tiles", n, H, W, sigma, flush=True)
    refs, tests, _ = E.gen_pairs([S.make_spec(81, i, H, W, mis_deg=(0.0, 5.0)) for i in range(n)], labels=False)
    stops = set()
    for iters, tol in ((1, 0.0), (9, 0.0), (12, 0.0), (40, 0.3), (40, 0.1), (7, 0.02), (8, 0.02)):
        a, (ia, _) = call(E, refs, tests, False, iters=(iters,), sigma_px=sigma, tol_px=tol)
        b, (ib, _) = call(E, refs, tests, True, iters=(iters,), sigma_px=sigma, tol_px=tol)
        for k in ("field", "iters", "q1"):
            assert torch.equal(a[k], b[k]), (k, iters, tol)
        if iters > 4:
            assert ib[0] < ia[0]
        stops.update(int(v) % 4 for v in a["iters"].flatten() if v < iters)
    print("  stops (iteration mod 4):", sorted(stops))


# batches that the wide regions take without a tolerance (radius 1 the last, 2 and 3
# the first two, 4 the first and last): one region across with an odd width, several
# across, a last region of one row or column; with a tolerance the rule goes by it too
@pytest.mark.parametrize("n,H,W", [(60, 120, 127), (16, 257, 241), (110, 123, 127)])
@pytest.mark.parametrize("sigma", [0.4, 0.7, 1.0, 1.3])  # radius 1 .. 4
def test_wide_regions_equal_single_iterations(E, n, H, W, sigma):
    from paper_1907_05993_amd import synth as S
    print("case: wide regions", n, H, W, sigma, flush=True)
    refs, tests, _ = E.gen_pairs([S.make_spec(84, i, H, W, mis_deg=(0.0, 5.0)) for i in range(n)], labels=False)
    for iters, tol in ((1, 0.0), (9, 0.0), (12, 0.0), (40, 0.1), (7, 0.02), (30, 1e-3)):
        a, (ia, _) = call(E, refs, tests, False, iters=(iters,), sigma_px=sigma, tol_px=tol)
        b, (ib, _) = call(E, refs, tests, True, iters=(iters,), sigma_px=sigma, tol_px=tol)
        for k in ("field", "iters", "q1"):
            assert torch.equal(a[k], b[k]), (k, iters, tol)
        if iters > 4 and not tol:
            assert ib[0] < ia[0]


# batches that the marching wavefronts take: two and four columns per lane, lanes
# past the last column, two and three segments, strips that do not divide the
# height (the last of a few rows)
@pytest.mark.parametrize("n,H,W", [(1024, 90, 126), (1000, 66, 128), (200, 110, 132), (128, 128, 256), (160, 100, 260),
                                   (64, 140, 700)])
@pytest.mark.parametrize("sigma", [0.7, 1.0])
def test_marching_wavefronts_equal_single_iterations(E, n, H, W, sigma):
    from paper_1907_05993_amd import synth as S
    print("case: marching wavefronts", n, H, W, sigma, flush=True)
    refs, tests, _ = E.gen_pairs([S.make_spec(83, i, H, W, mis_deg=(0.0, 5.0)) for i in range(n)], labels=False)
    for iters, tol in ((1, 0.0), (9, 0.0), (12, 0.0), (40, 0.2), (31, 0.05)):
        a, (ia, _) = call(E, refs, tests, False, iters=(iters,), sigma_px=sigma, tol_px=tol)
        b, (ib, _) = call(E, refs, tests, True, iters=(iters,), sigma_px=sigma, tol_px=tol)
        for k in ("field", "iters", "q1"):
            assert torch.equal(a[k], b[k]), (k, iters, tol)
        if iters > 4:
            assert ib[0] < ia[0]


@pytest.mark.parametrize("n,H,W", [(1, 40, 37), (2, 65, 513), (1, 70, 1000)])
def test_points_equal_single_iterations(E, n, H, W):
    from paper_1907_05993_amd import synth as S
    print("case: points", n, H, W, flush=True)
    refs, tests, _ = E.gen_pairs([S.make_spec(82, i, H, W, mis_deg=(0.0, 5.0)) for i in range(n)], labels=False)
    for iters in (0, 1, 25):
        a, _ = call(E, refs, tests, False, iters=(iters,), sigma_px=0.0)
        b, (issued, planned) = call(E, refs, tests, True, iters=(iters,), sigma_px=0.0)
        for k in ("field", "iters", "q1"):
            assert torch.equal(a[k], b[k]), (k, iters)
        if W > 64:
            assert issued[0] == planned[0] == (1 if iters else 0)


@pytest.fixture(scope="module")
def E():
    from paper_1907_05993_amd import ebsd
    ebsd.lib()
    return ebsd


# The stop decisions of a launch are taken by every workgroup of a pair, also by
# those that start (in a later round of the device) after the first one has
# written the stop: strips of a few rows over several rounds, repeated calls
@pytest.mark.parametrize("n,H,W", [(257, 519, 519), (900, 135, 150), (700, 66, 128)])
def test_stops_over_several_rounds(E, n, H, W):
    from paper_1907_05993_amd import synth as S
    print("case: stops", n, H, W, flush=True)
    m = 64
    refs, tests, _ = E.gen_pairs([S.make_spec(85, i, H, W, mis_deg=(0.0, 8.0)) for i in range(m)], labels=False)
    refs, tests = (x.repeat(-(-n // m), 1, 1)[:n].contiguous() for x in (refs, tests))
    p = dict(levels=1, iters=(12,), sigma_px=1.0, tol_px=0.1, roi_size=32, n_roi=5, roi_radius_frac=0.002)
    one, _ = call(E, refs, tests, False, **{k: v for k, v in p.items() if k in ("iters", "sigma_px", "tol_px")})
    for ty in (0, 32, 64, 128):
        reg = E.Registrar(E.Params(**p))
        if ty:
            reg.set_fused_height(H, W, ty)
        for _ in range(6):
            out = reg.register(refs, tests)
            torch.cuda.synchronize()
            assert torch.equal(one["iters"], out["iters"]), ty
            assert torch.equal(one["field"], out["field"]), ty
        reg.close()
