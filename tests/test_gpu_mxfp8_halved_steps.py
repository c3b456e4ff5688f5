"""MX-FP8 projections whose waves halve every depth step (128 x 192 tiles), at
last groups of one to four steps, ragged rows and more than one
round of tiles: against float64 products of the decoded operands, and bit for
bit the same with scale rows on 16 bytes and not."""
import pytest
import torch

from tests.gpu_util import need_gpu, plans
from tests.test_gpu_mxfp8_small_tiles import EPS, decoded, quantized

import paper_2410_05437_amd as espace

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R,C,D", [(4096, 1536, 1536), (4001, 1500, 1537), (4090, 1441, 1700), (3970, 1530, 1800),
                                   (2048, 2458, 2500), (8100, 1500, 9000)])
def test_project(capfd, R, C, D):
    need_gpu()
    got = []
    for pad16 in (True, False):
        g = torch.Generator(device="cuda").manual_seed(R + C + D)
        X, Pt = quantized(R, D, g, pad16), quantized(C, D, g, pad16)
        Z = espace.mx_empty(R, C, "cuda")
        Z.codes.fill_(0x7F)
        Z.scales.fill_(0xFF)
        _, (p,) = plans(capfd, lambda: espace.espace_project_mxfp8(Pt, X, Z=Z))
        assert p["small"] < 0 and p["tile"] == 2, p
        got.append(Z)
    assert torch.equal(got[0].codes, got[1].codes)
    assert torch.equal(got[0].scales[:, :(C + 127) // 128 * 4], got[1].scales[:, :(C + 127) // 128 * 4])
    assert not Z.codes[:, C:].any() and not Z.scales[:, (C + 31) // 32:(C + 127) // 128 * 4].any()
    ref, mag = decoded(X) @ decoded(Pt).t(), decoded(X).abs() @ decoded(Pt).abs().t()
    amax = torch.nn.functional.pad(ref, (0, -C % 32)).abs().view(R, -1, 32).amax(-1).repeat_interleave(32, 1)[:, :C]
    # half an E4M3 step or the clamp, and the accumulation: two instructions per step
    bound = 2.0 ** -3 * ref.abs() + 2.0 ** -16 * amax + (2 * ((D + 127) // 128) + 1) * EPS * mag
    assert bool(((decoded(Z) - ref).abs() <= bound).all())
    assert ((decoded(Z) - ref).norm() / ref.norm()).item() < 4e-2
