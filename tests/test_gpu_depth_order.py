"""Tiles whose XCDs all walk the depth in one order (192 x 192, and 256 x 256 at
depths or operands past the Infinity Cache): equal tokens give equal results bit for
bit wherever their tiles run."""
import pytest
import torch

from tests.gpu_util import need_gpu, plans

import paper_2410_05437_amd as espace

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R,C,D,tile", [(2163, 3992, 5504, "192x192"), (4096, 4096, 16384, "256x256"),
                                        (4096, 4096, 17000, "256x256")])
def test_equal_tokens(capfd, R, C, D, tile):
    need_gpu()
    g = torch.Generator(device="cuda").manual_seed(D)
    x = espace.padded_empty(R, D, torch.bfloat16, "cuda")
    x.copy_(torch.randn(1, D, generator=g, device="cuda").expand(R, D))
    W = espace.padded_empty(C, D, torch.bfloat16, "cuda")
    W.copy_(torch.randn(C, D, generator=g, device="cuda"))
    Y, (p,) = plans(capfd, lambda: espace.espace_dense_linear(x, W))
    assert p["kind"] == "tiled" and p["tile"] == tile and p["splits"] == 1 and p["rows1"] == 0
    assert bool((Y == Y[:1]).all())
