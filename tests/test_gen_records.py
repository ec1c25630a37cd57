"""The pattern specs as the library takes them (ebsd.gen_pairs): orientations,
deformations, gradients and counts of any array or tensor kind and shape of nine
elements, against a record filled field by field.  CPU only."""
import numpy as np
import pytest
import torch

from paper_1907_05993_amd import ebsd
from paper_1907_05993_amd import synth as S


def by_field(spec):
    r = ebsd.CGenSpec()
    G, F = [float(v) for v in list(spec.G.ravel())], [float(v) for v in list(spec.F.ravel())]
    for j in range(9):
        r.G[j], r.F[j] = G[j], F[j]
    r.gx, r.gy, r.counts = float(spec.gxy[0]), float(spec.gxy[1]), float(spec.counts)
    r.key[0], r.key[1] = int(spec.seeds[0]) & 0xFFFFFFFF, int(spec.seeds[1]) & 0xFFFFFFFF
    r.noise, r.bands = int(bool(spec.noise)), 1
    return bytes(r)


def grad(a):
    return torch.tensor(a, requires_grad=True)


@pytest.mark.parametrize("kinds", [(np.asarray,), (np.float32,), (np.ravel,), (lambda a: a[None],), (np.asfortranarray,),
                                   (lambda a: np.append(a, 7.0),), (torch.tensor,), (grad,),
                                   (np.asarray, np.ravel, grad)])
def test_records_equal_field_by_field(kinds):
    specs = []
    for i in range(7):
        s = S.make_spec(3, i, 64, 64, mis_deg=(0.0, 9.0))
        kind = kinds[i % len(kinds)]
        s.G, s.F = kind(s.G), kind(s.F)
        s.seeds = (2 ** 40 + 5, -i)
        if kind in (torch.tensor, grad):
            s.gxy, s.counts = kind(np.asarray(s.gxy)), kind(s.counts)
        specs.append(s)
    assert ebsd._gen_records(specs).tobytes() == b"".join(by_field(s) for s in specs)


@pytest.mark.parametrize("n", [1, 4])
def test_too_few_elements_are_refused(n):
    specs = [S.make_spec(3, i, 64, 64) for i in range(n)]
    for s in specs:
        s.G = np.ones(1)
    with pytest.raises(IndexError):
        ebsd._gen_records(specs)
