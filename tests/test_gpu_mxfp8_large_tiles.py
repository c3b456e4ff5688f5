"""MX-FP8 projections of many tokens on 128 x 192 tiles (scale rows on 16 bytes
and not), ragged, against float64 products of the decoded operands; the padding
columns up to a multiple of 128 are written as zeros."""
import pytest
import torch

from tests.gpu_util import need_gpu, plans
from tests.test_gpu_mxfp8_small_tiles import EPS, decoded, quantized

import paper_2410_05437_amd as espace

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R,C,D", [(4096, 1536, 1600), (2048, 2458, 2500), (4001, 1500, 1537), (2481, 1921, 1959),
                                   (2454, 1556, 1936)])
@pytest.mark.parametrize("pad16", [True, False])
def test_project(capfd, R, C, D, pad16):
    need_gpu()
    g = torch.Generator(device="cuda").manual_seed(R + C + D)
    X, Pt = quantized(R, D, g, pad16), quantized(C, D, g, pad16)
    Z = espace.mx_empty(R, C, "cuda")
    Z.codes.fill_(0x7F)
    Z.scales.fill_(0xFF)
    _, (p,) = plans(capfd, lambda: espace.espace_project_mxfp8(Pt, X, Z=Z))
    assert p["small"] < 0 and p["tile"] == 2, p                 # 128 x 192
    assert not Z.codes[:, C:].any() and not Z.scales[:, (C + 31) // 32:].any()
    ref, mag = decoded(X) @ decoded(Pt).t(), decoded(X).abs() @ decoded(Pt).abs().t()
    amax = torch.nn.functional.pad(ref, (0, -C % 32)).abs().view(R, -1, 32).amax(-1).repeat_interleave(32, 1)[:, :C]
    # as for the small tiles: half an E4M3 step or the clamp, and the accumulation
    bound = 2.0 ** -3 * ref.abs() + 2.0 ** -16 * amax + ((D + 127) // 128 + 1) * EPS * mag
    assert bool(((decoded(Z) - ref).abs() <= bound).all())
    assert ((decoded(Z) - ref).norm() / ref.norm()).item() < 4e-2
