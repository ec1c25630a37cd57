"""The second pass's remap (two quotients of each pixel's ray from one
reciprocal) against the stand-alone remap (two divisions): the shifts and peak
heights of ebsd_second_pass_batch equal, bit for bit, those of the cross-correlation
of the ROIs cut from ebsd_stage_remap's image.  Among the rotations are those by a
right angle, which turn the rays of one column or row (at an integer pattern
centre) parallel to the detector.  Needs an MI355X."""
import numpy as np
import pytest
import torch
from scipy.spatial.transform import Rotation

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def E():
    from paper_1907_05993_amd import ebsd
    ebsd.lib()
    return ebsd


# right angles as whole numbers: the third component of R^T r is exactly 0 in a
# column (first four) or in a row
RIGHT = [[[0, 0, s], [0, 1, 0], [-s, 0, 0]] for s in (1, -1)] + [[[0, 0, s], [0, -1, 0], [s, 0, 0]] for s in (1, -1)] + \
    [[[1, 0, 0], [0, 0, s], [0, -s, 0]] for s in (1, -1)] + [[[-1, 0, 0], [0, 0, s], [0, s, 0]] for s in (1, -1)]


@pytest.mark.parametrize("H,W,N", [(128, 128, 32), (128, 192, 64), (300, 280, 128), (320, 336, 256)])
@pytest.mark.parametrize("interp", [3, 1])
def test_second_pass_equals_stage_remap(E, H, W, N, interp):
    print("case: second pass remap", H, W, N, interp, flush=True)
    tilted = [Rotation.from_rotvec(v).as_matrix() for v in
              ([0.01, -0.02, 0.03], [0.3, 0.1, -0.2], [0.0, 1.2, 0.0], [-1.4, 0.1, 0.0], [2.0, 0.5, 0.1])]
    R = torch.tensor(np.array(RIGHT + tilted, dtype=np.float64), device="cuda")
    n = R.shape[0]
    g = torch.Generator(device="cuda").manual_seed(H + W + N)
    refs, tests = (torch.rand(n, H, W, generator=g, device="cuda") for _ in range(2))
    pc = ((W // 2 + 0.5) / W, (H // 2 + 0.5) / H, 0.7)  # xs = W / 2, ys = H / 2
    p = E.Params(levels=1, roi_size=N, n_roi=5, roi_radius_frac=0.02, pc=pc, remap_interp=interp)
    pcs = (pc[0] * W - 0.5, pc[1] * H - 0.5, pc[2] * W)
    assert pcs[0] == W // 2 and pcs[1] == H // 2
    reg = E.Registrar(p)
    out = reg.second_pass(refs, tests, R)
    torch.cuda.synchronize()
    norm = [E.stage_normalize(x)[0] for x in (refs, tests)]
    image, _ = E.stage_remap(norm[0], R, pcs, interp=interp)
    _, _, x0, y0 = E.roi_layout(p, H, W)
    for j in range(5):
        a, b = (im[:, y0[j]:y0[j] + N, x0[j]:x0[j] + N].contiguous() for im in (image, norm[1]))
        q, ph = E.stage_xcf(a, b)
        torch.cuda.synchronize()
        assert torch.equal(out["q2"][:, j], q), (j, (out["q2"][:, j] - q).abs().max(dim=1))
        assert torch.equal(out["peak_height"][:, j], ph), j
    reg.close()
