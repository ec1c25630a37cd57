"""ebsd_autotune measures every kernel that a level can run on and later calls
run what it measured, and the tuning cache carries it to the next handle.
Needs an MI355X."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def E():
    from paper_1907_05993_amd import ebsd
    ebsd.lib()
    return ebsd


def pairs(E, n, H, W):
    from paper_1907_05993_amd import synth as S
    return E.gen_pairs([S.make_spec(91, i, H, W, mis_deg=(0.0, 6.0)) for i in range(n)], labels=False)[:2]


def params(E, **kw):
    return E.Params(levels=3, iters=(12,) * 3, sigma_px=1.0, roi_size=32, n_roi=8, **kw)


# what a tuning table says was measured is what runs: 12 iterations as 12 launches (one
# per launch), 6 (two) or 3 (four), also where the prediction prefers another kernel
@pytest.mark.parametrize("kind,fused,launches", [("rows", 0, 12), ("rows2", 32, 6), ("march", 0, 6), ("regions", 0, 3)])
def test_measured_kernel_runs(E, tmp_path, monkeypatch, kind, fused, launches):
    print("case: measured kernel", kind, flush=True)
    path = tmp_path / "tune.txt"
    k = E.PLAN_KINDS.index(kind)
    path.write_text("".join(f"gfx950 {s} {s} 64 {fused},{k},48\n" for s in (256, 128)))
    monkeypatch.setenv("EBSD_TUNE_CACHE", str(path))
    reg = E.Registrar(params(E))
    monkeypatch.delenv("EBSD_TUNE_CACHE")
    plain = E.Registrar(params(E))
    refs, tests = pairs(E, 48, 256, 256)
    a, b = plain.register(refs, tests), reg.register(refs, tests)
    torch.cuda.synchronize()
    issued, planned = reg.launch_counts()
    for level in (0, 1):
        assert reg.level_plan(256, 256, level, 48)[0] == kind
        assert issued[level] == planned[level] == launches
    for key in ("field", "iters", "F", "status"):
        assert torch.equal(a[key], b[key]), key
    # for a quarter to four times as many pairs; others go by prediction
    for n in (12, 48, 192):
        assert reg.level_plan(256, 256, 0, n)[0] == kind
    assert plain.level_plan(256, 256, 0, 1)[0] == "regions" and plain.level_plan(256, 256, 0, 4096)[0] == "march"
    assert reg.level_plan(256, 256, 0, 1)[0] == "regions" and reg.level_plan(256, 256, 0, 4096)[0] == "march"
    plain.close()
    reg.close()


@pytest.mark.parametrize("n,H,W,sigma,tol", [(48, 256, 256, 1.0, 0.0), (3, 200, 260, 0.7, 0.05), (20, 150, 171, 1.3, 0.0),
                                             (2, 300, 600, 1.0, 0.0)])
def test_autotune_keeps_what_it_measured(E, tmp_path, monkeypatch, n, H, W, sigma, tol):
    print("case: autotune", n, H, W, sigma, tol, flush=True)
    path = tmp_path / "tune.txt"
    monkeypatch.setenv("EBSD_TUNE_CACHE", str(path))
    p = E.Params(levels=3, iters=(24,) * 3, sigma_px=sigma, tol_px=tol, roi_size=32, n_roi=8,
                 roi_radius_frac=0.1)
    refs, tests = pairs(E, n, H, W)
    plain = E.Registrar(p)
    reg = E.Registrar(p)
    reg.autotune(refs, tests)
    lines = {tuple(x.split()[1:3]): x.split()[4] for x in path.read_text().splitlines()}
    again = E.Registrar(p)
    outs = [r.register(refs, tests) for r in (plain, reg, again)]
    torch.cuda.synchronize()
    for level in range(3):
        h, w = E.level_size(H, W, level)
        kind, rows = reg.level_plan(H, W, level, n)
        print("  level", level, (h, w), kind, rows, "by rule:", plain.level_plan(H, W, level, n), flush=True)
        assert again.level_plan(H, W, level, n) == (kind, rows)
        if kind == "resident":
            assert lines[str(h), str(w)].isdigit()
        else:
            assert lines[str(h), str(w)].split(",")[1:] == [str(E.PLAN_KINDS.index(kind)), str(n)]
    for o in outs[1:]:
        for key in ("field", "iters", "F", "status"):
            assert torch.equal(o[key], outs[0][key]), key
    # the measured kernel is not slower than the others by more than what timings of
    # levels of a few launches scatter by
    if tol == 0.0:
        kind, _ = reg.level_plan(H, W, 0, n)
        ms = {}
        for k, rows in (("rows", 64), ("rows", 16), ("rows2", 32), ("march", 32), ("march", 64), ("regions", 32),
                        ("regions", 64), ("regions", 80)):
            t = E.Registrar(p)
            try:
                t.set_level_plan(H, W, k, rows)
            except E.EbsdError:
                continue
            t.set_timing()
            for _ in range(4):
                t.register(refs, tests)
                ms[k, rows] = min(ms.get((k, rows), 1e9), float(t.timing()[0][0]))
            t.close()
        reg.set_timing()
        for _ in range(4):
            reg.register(refs, tests)
            ms["tuned"] = min(ms.get("tuned", 1e9), float(reg.timing()[0][0]))
        print("  ms of level 0:", {k: round(v, 4) for k, v in ms.items()}, flush=True)
        assert ms["tuned"] <= 1.3 * min(ms.values())
    for r in (plain, reg, again):
        r.close()


def test_plans_that_a_level_does_not_support_are_refused(E):
    reg = E.Registrar(params(E))
    for level, kind, rows in (((256, 255), "march", 32), ((256, 256), "march", 8), ((256, 256), "regions", 48),
                              ((256, 256), "points", 0), ((256, 256), "rows", 0), ((256, 256), "rows2", 8),
                              ((256, 256), "resident", 0), ((5000, 5000), "march", 64), ((5000, 5000), "regions", 80),
                              ((0, 256), "rows", 64), ((256, 256), "march", 1 << 30)):
        with pytest.raises(E.EbsdError) as ei:
            reg.set_level_plan(*level, kind, rows)
        assert ei.value.code == -1, (level, kind, rows)
    reg.set_level_plan(256, 256, "regions", 64)
    assert reg.level_plan(256, 256, 0, 1000) == ("regions", 64)
    reg.set_fused_height(256, 256, 32)  # the last one counts
    assert reg.level_plan(256, 256, 0, 1000) == ("rows2", 32)
    reg.set_level_plan(256, 256, "march", 16)
    assert reg.level_plan(256, 256, 0, 1000) == ("march", 16)
    reg.set_level_plan(256, 256, None)
    assert reg.level_plan(256, 256, 0, 1000) == ("rows2", 32)
    assert reg.level_plan(256, 256, 2, 1000) == ("resident", 0)
    for bad in ((256, 256, 3, 10), (256, 256, -1, 10), (256, 256, 0, 0), (0, 256, 0, 10)):
        with pytest.raises(E.EbsdError):
            reg.level_plan(*bad)
    reg.close()
