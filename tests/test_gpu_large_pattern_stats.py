"""Statistics of few large patterns by 16 workgroups each (patterns of at least 2^17
pixels at 16-byte addresses) against those by one workgroup each, which the same
patterns one pixel off such an address take: fields, shifts and status bit for bit,
also with tails of one to three pixels, flagged patterns and the pre-filter.  Needs an
MI355X."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def E():
    from paper_1907_05993_amd import ebsd
    ebsd.lib()
    return ebsd


def at_offset(x, off):
    """Copies of the patterns of x, each `off` floats past a 16-byte address."""
    out = []
    for p in x:
        buf = torch.zeros(p.numel() + 8, device="cuda")
        v = buf[off:off + p.numel()].view(p.shape)
        v.copy_(p)
        assert v.data_ptr() % 16 == 4 * off
        out.append(v)
    return out


@pytest.mark.parametrize("n,H,W", [(2, 512, 256), (1, 363, 363), (2, 331, 398), (3, 365, 363), (2, 512, 1025),
                                   (1, 1024, 1244)])
@pytest.mark.parametrize("bandpass", [(0.0, 0.0), (1.0, 12.0)])
def test_statistics_of_few_large_patterns(E, n, H, W, bandpass):
    print("case: large pattern statistics", n, H, W, bandpass, flush=True)
    g = torch.Generator(device="cuda").manual_seed(H * W)
    refs, tests = (1e3 + 400 * torch.rand(n + 4, H, W, generator=g, device="cuda") for _ in range(2))
    tests[n, H // 2, 3] = float("nan")
    refs[n + 1, -1, -1] = float("inf")
    tests[n + 2].fill_(7.0)  # no contrast
    refs[n + 3, 0, 0] = 3e38  # squares far out of range of FP32
    outs = []
    for off in (0, 1):
        reg = E.Registrar(E.Params(levels=2, iters=(3, 3), sigma_px=1.0, roi_size=64, n_roi=6, roi_radius_frac=0.05,
                                   bandpass=bandpass))
        outs.append(reg.register(at_offset(refs, off), at_offset(tests, off)))
        torch.cuda.synchronize()
        reg.close()
    a, b = outs
    assert torch.equal(a["status"], b["status"])
    st = a["status"].cpu().tolist()
    print("  status:", st, flush=True)
    assert all(s == st[0] for s in st[:n])
    for k in ("q1", "q2", "F", "peak_height"):
        assert torch.equal(a[k][:n], b[k][:n]), k
        assert torch.equal(torch.nan_to_num(a[k]), torch.nan_to_num(b[k])), k
    for x, y in zip(a["field"], b["field"]):
        assert torch.equal(torch.nan_to_num(x), torch.nan_to_num(y))
