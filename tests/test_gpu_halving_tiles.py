"""Products on the tiles whose waves halve every depth step (128 x 192 at long
depths, 192 x 192, 256 x 160), ragged in every dimension, against a float64
product; sizes for which the planner takes them with 256 CUs."""
import pytest
import torch

from tests.gpu_util import need_gpu, plans

import paper_2410_05437_amd as espace

pytestmark = pytest.mark.gpu

# (rows, columns, depth), tile, depth ranges: 128 x 192 at long depths, 192 x 192, 256 x 160
SIZES = [(4090, 1530, 3080, "128x192", 1), (4090, 1530, 3077, "128x192", 1), (12280, 1533, 3901, "192x192", 1),
         (380, 24500, 2405, "192x192", 1), (8190, 2555, 3100, "256x160", 1), (8190, 2555, 3077, "256x160", 1),
         (1025, 135, 12726, "128x192", 4), (2748, 515, 9277, "128x192", 3),
         (10996, 289, 3160, "192x192", 2), (3208, 823, 4007, "192x192", 3), (5426, 258, 4501, "192x192", 4),
         (8644, 388, 3049, "256x160", 2), (8218, 275, 3751, "256x160", 3), (6376, 263, 4820, "256x160", 4)]


def mat(rows, cols, g):
    """rows x cols bfloat16 with NaN in the padding columns."""
    ld = (cols + 7) // 8 * 8
    t = torch.full((rows, ld), float("nan"), device="cuda", dtype=torch.bfloat16)
    t[:, :cols] = torch.randn(rows, cols, generator=g, device="cuda")
    return t[:, :cols]


@pytest.mark.parametrize("R,C,D,tile,splits", SIZES)
def test_product(capfd, R, C, D, tile, splits):
    need_gpu()
    g = torch.Generator(device="cuda").manual_seed(R + C + D)
    X, W = mat(R, D, g), mat(C, D, g)
    Y = espace.padded_empty(R, C, torch.bfloat16, X.device)
    whole = torch.as_strided(Y, (R, Y.stride(0)), (Y.stride(0), 1)).fill_(float("nan"))
    _, (p,) = plans(capfd, lambda: espace.espace_dense_linear(X, W, Y=Y))
    assert (p["kind"], p["tile"], p["splits"], p["pair"], p["rows1"]) == ("tiled", tile, splits, 0, 0), p
    ref, mag = X.double() @ W.double().t(), X.double().abs() @ W.double().abs().t()
    # exact products, fp32 sums of D terms in any order, one rounding to bfloat16
    bound = 2.0 ** -8 * ref.abs() + (1 + 2.0 ** -8) * (D + 16) * 2.0 ** -23 * mag
    assert bool(((Y.double() - ref).abs() <= bound).all())
    assert bool(whole[:, C:].isnan().all())          # nothing written past a row
    assert torch.equal(espace.espace_dense_linear(X, W), Y)


@pytest.mark.parametrize("M,K,L,N,tile", [(12288, 4090, 1530, 4090, "128x192"), (6144, 3100, 2555, 8190, "256x160")])
def test_layer_projection(capfd, M, K, L, N, tile):
    """Z handed on in row pairs gives what projection and expansion give."""
    need_gpu()
    g = torch.Generator(device="cuda").manual_seed(N)
    X, Pt, Wf = mat(N, K, g), mat(L, K, g), mat(M, L, g)
    Y, ps = plans(capfd, lambda: espace.espace_projected_linear(X, Pt, Wf))
    assert ps[0]["tile"] == tile and ps[0]["splits"] == 1 and ps[0]["rows1"] == 0, ps
    assert torch.equal(Y, espace.espace_expand(espace.espace_project(Pt, X), Wf))
