"""The bfloat16 product on small tiles (a few to a few hundred tokens) at its
edges: ragged tokens, rows and depths, a depth split, and the layer whose
projection runs on them while its expansion is tiled."""
import pytest
import torch

from tests.gpu_util import need_gpu, plans

import paper_2410_05437_amd as espace

pytestmark = pytest.mark.gpu

# (rows of the weight, depth): fewer than a chunk, a chunk that straddles the
# depth, whole steps, more waves than steps, few rows and a long depth (split)
WEIGHTS = [(1, 1), (37, 5), (300, 129), (1537, 515), (2458, 1000), (1000, 12000), (5001, 72)]
TOKENS = [3, 8, 9, 16, 17, 33, 48, 49, 100, 201, 333]


def mat(rows, cols, g):
    """rows x cols bfloat16 with NaN in the padding columns."""
    ld = (cols + 7) // 8 * 8
    t = torch.full((rows, ld), float("nan"), device="cuda", dtype=torch.bfloat16)
    t[:, :cols] = torch.randn(rows, cols, generator=g, device="cuda")
    return t[:, :cols]


def check(Y, X, W):
    ref = X.double() @ W.double().t()
    mag = X.double().abs() @ W.double().abs().t()
    # exact products, fp32 sums of D terms in any order, one rounding to bfloat16
    bound = 2.0 ** -8 * ref.abs() + (1 + 2.0 ** -8) * (X.shape[1] + 16) * 2.0 ** -23 * mag
    assert bool(((Y.double() - ref).abs() <= bound).all())


@pytest.mark.parametrize("C,D", WEIGHTS)
def test_small_tiles(C, D):
    need_gpu()
    g = torch.Generator(device="cuda").manual_seed(C * 7 + D)
    W = mat(C, D, g)
    for R in TOKENS:
        X = mat(R, D, g)
        Y = espace.padded_empty(R, C, torch.bfloat16, X.device)
        whole = torch.as_strided(Y, (R, Y.stride(0)), (Y.stride(0), 1))
        whole.fill_(float("nan"))
        espace.espace_dense_linear(X, W, Y=Y)
        check(Y, X, W)
        assert bool(whole[:, C:].isnan().all())      # nothing written past a row


# (tokens, rows, depth): every tile configuration in the kernel's order, ragged
# everywhere, a partial last tile both ways
CONFIGS = [(3, 41, 157), (9, 42, 161), (17, 41, 159), (3, 4125, 164), (3, 9054, 151), (3, 12347, 150), (3, 17142, 155),
           (3, 21471, 158), (716, 161, 155), (18, 6497, 155), (17, 10596, 159), (17, 13090, 158), (17, 17597, 166),
           (17, 21803, 173), (516, 350, 158), (35, 7211, 164), (33, 8911, 166), (33, 13139, 183), (34, 17684, 159),
           (36, 21335, 151), (763, 325, 153), (957, 527, 151), (98, 5509, 155), (52, 13156, 159), (49, 16599, 167),
           (162, 7050, 150), (66, 6823, 150), (145, 5303, 153), (69, 12397, 169), (67, 16417, 157), (267, 2706, 196),
           (954, 1177, 159), (91, 12650, 162), (100, 10651, 154)]


@pytest.mark.parametrize("config", range(len(CONFIGS)))
def test_every_tile(capfd, config):
    need_gpu()
    R, C, D = CONFIGS[config]
    g = torch.Generator(device="cuda").manual_seed(config)
    X, W = mat(R, D, g), mat(C, D, g)
    Y = espace.padded_empty(R, C, torch.bfloat16, X.device)
    whole = torch.as_strided(Y, (R, Y.stride(0)), (Y.stride(0), 1)).fill_(float("nan"))
    _, (p,) = plans(capfd, lambda: espace.espace_dense_linear(X, W, Y=Y))
    assert (p["kind"], p["tile"], p["splits"]) == ("small", config, 1), p
    check(Y, X, W)
    assert bool(whole[:, C:].isnan().all())


@pytest.mark.parametrize("M,K,L,N", [(12288, 4096, 1536, 333), (22016, 4096, 1530, 201), (24576, 1000, 700, 511)])
def test_layer_with_tiled_expansion(M, K, L, N):
    """Z handed from the small tiles to the tiled expansion (row pairs) gives
    what projection and expansion give by themselves."""
    need_gpu()
    g = torch.Generator(device="cuda").manual_seed(N)
    X, Pt, Wf = mat(N, K, g), mat(L, K, g), mat(M, L, g)
    Y = espace.espace_projected_linear(X, Pt, Wf)
    Z = espace.espace_project(Pt, X)
    check(Z, X, Pt)
    assert torch.equal(Y, espace.espace_expand(Z, Wf))
