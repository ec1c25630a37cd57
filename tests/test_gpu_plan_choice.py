"""The kernel that the rule picks for a level is not slower than one iteration per
launch, which every level ran on before there was a rule: levels whose pairs stop
on a coarse tolerance after a few iterations (a launch of several runs on past the
stop and repeats it), large batches of little smoothing (irregular fields, whose
gathers bind the row and marching kernels) and of the widest.  Needs an MI355X."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def E():
    from paper_1907_05993_amd import ebsd
    ebsd.lib()
    return ebsd


# pairs, size, smoothing, tolerance, iterations: where the rule took 1.3 to 3.8 times as
# long as one iteration per launch, or 1.5 to 1.9 times as long as the best kernel
CASES = [(31, 1024, 1244, 1.3, 0.1, 60), (885, 300, 301, 1.0, 0.1, 60), (487, 153, 161, 1.0, 0.1, 60),
         (487, 153, 161, 0.7, 0.1, 60), (62, 1024, 1244, 1.0, 0.1, 60), (132, 300, 301, 1.0, 0.1, 60),
         (885, 300, 301, 1.3, 0.0, 24), (250, 400, 400, 0.4, 0.0, 24), (610, 256, 256, 0.4, 0.0, 24)]


@pytest.mark.parametrize("n,H,W,sigma,tol,iters", CASES)
def test_rule_is_not_slower_than_single_iterations(E, n, H, W, sigma, tol, iters):
    from paper_1907_05993_amd import synth as S
    m = min(n, 24)
    refs, tests, _ = E.gen_pairs([S.make_spec(95, i, H, W, mis_deg=(0.0, 8.0)) for i in range(m)], labels=False)
    at = torch.arange(n, device="cuda") % m
    refs, tests = refs[at].contiguous(), tests[at].contiguous()
    p = E.Params(levels=3, iters=(iters,) * 3, sigma_px=sigma, tol_px=tol, roi_size=32, n_roi=5, roi_radius_frac=0.01,
                 second_pass=0)

    def level_ms(resident, plan=None):
        reg = E.Registrar(p)
        reg.set_gating(0)
        reg.set_resident(resident)
        if plan:
            reg.set_level_plan(H, W, *plan)
        reg.set_timing()
        ms = []
        for _ in range(4):
            reg.register(refs, tests, want_field=False)
            ms.append(float(reg.timing()[0][0]))
        kind = reg.level_plan(H, W, 0, n)
        reg.close()
        return min(ms[1:]), kind

    (rule, kind), (single, _) = level_ms(True), level_ms(False)
    regions, _ = level_ms(True, ("regions", 64))
    print(f"case: {n} x {H} x {W}, sigma {sigma}, tolerance {tol}: rule {kind} {rule:.3f} ms, one iteration "
          f"{single:.3f}, regions {regions:.3f}", flush=True)
    assert rule <= 1.15 * min(single, regions)
