"""MX-FP8 products on small tiles (up to about a thousand tokens) at their
edges, against float64 products of the decoded operands, with scale rows at
the smallest leading dimension and padded to 16 bytes."""
import pytest
import torch

from tests.gpu_util import need_gpu, plans

import paper_2410_05437_amd as espace

pytestmark = pytest.mark.gpu

# (tokens, weight rows, depth): ragged everywhere, one step, more waves than
# steps, several rounds, and a depth only the narrow tiles' scales fit
SIZES = [(1, 1, 1), (8, 300, 130), (13, 1537, 515), (17, 129, 4096), (48, 2500, 700), (100, 1000, 11008),
         (201, 5001, 384), (333, 640, 2458), (640, 1536, 1000), (5, 200, 24576)]
EPS = 2.0 ** -10        # per block-scaled instruction, of |C| + sum |a·b| (about 3x the largest measured)


def quantized(rows, cols, g, pad16):
    A = espace.padded_empty(rows, cols, torch.bfloat16, "cuda")
    A.copy_(torch.randn(rows, cols, generator=g, device="cuda") *
            torch.exp(torch.randn(rows, cols, generator=g, device="cuda")))
    out = espace.mx_empty(rows, cols, A.device)
    if not pad16:
        cp = out.codes.shape[1]
        out.scales = torch.empty((rows, cp // 32), dtype=torch.uint8, device=A.device)
    return espace.espace_quantize_mxfp8(A, out=out)


def decoded(m):
    v = m.codes.view(torch.float8_e4m3fn).double()
    s = torch.exp2(m.scales.double() - 127).repeat_interleave(32, dim=1)[:, :v.shape[1]]
    return (v * s)[:, :m.cols]


@pytest.mark.parametrize("R,C,D", SIZES)
def test_expand(R, C, D):
    need_gpu()
    got = []
    for pad16 in (True, False):
        g = torch.Generator(device="cuda").manual_seed(R + C + D)
        T, W = quantized(R, D, g, pad16), quantized(C, D, g, pad16)
        Y = espace.padded_empty(R, C, torch.bfloat16, "cuda")
        whole = torch.as_strided(Y, (R, Y.stride(0)), (Y.stride(0), 1))
        whole.fill_(float("nan"))
        espace.espace_expand_mxfp8(T, W, Y=Y)
        assert bool(whole[:, C:].isnan().all())
        got.append(Y)
    assert torch.equal(got[0], got[1])
    ref, mag = decoded(T) @ decoded(W).t(), decoded(T).abs() @ decoded(W).abs().t()
    # the chain of instructions errs by at most EPS per instruction of the
    # magnitude so far, and a wave's chain has at most D / 128 of them
    n = (D + 127) // 128
    bound = 2.0 ** -8 * ref.abs() + (n + 1) * EPS * mag
    assert bool(((Y.double() - ref).abs() <= bound).all())
    assert ((Y.double() - ref).norm() / ref.norm()).item() < 4e-3


@pytest.mark.parametrize("R,C,D", [s for s in SIZES if s[1] <= s[2]])
def test_project(R, C, D):
    need_gpu()
    got = []
    for pad16 in (True, False):
        g = torch.Generator(device="cuda").manual_seed(R + C + D)
        X, Pt = quantized(R, D, g, pad16), quantized(C, D, g, pad16)
        Z = espace.mx_empty(R, C, "cuda")
        Z.codes.fill_(77)
        Z.scales.fill_(77)
        espace.espace_project_mxfp8(Pt, X, Z=Z)
        assert not Z.codes[:, C:].any() and not Z.scales[:, (C + 31) // 32:].any()   # the padding is zero
        got.append(Z)
    assert torch.equal(got[0].codes, got[1].codes) and torch.equal(got[0].scales, got[1].scales)
    ref, mag = decoded(X) @ decoded(Pt).t(), decoded(X).abs() @ decoded(Pt).abs().t()
    amax = torch.nn.functional.pad(ref, (0, -C % 32)).abs().view(R, -1, 32).amax(-1).repeat_interleave(32, 1)[:, :C]
    # E4M3 after scaling: half a step of 2^-4 for normal values, up to 2^-3 where
    # a value between 448 and 512 is clamped; 2^-9 2^S <= 2^-17 of the block's
    # largest for subnormal ones
    bound = 2.0 ** -3 * ref.abs() + 2.0 ** -16 * amax + ((D + 127) // 128 + 1) * EPS * mag
    assert bool(((decoded(Z) - ref).abs() <= bound).all())
    assert ((decoded(Z) - ref).norm() / ref.norm()).item() < 4e-2


# every tile configuration in the kernel's order, and those with MX-FP8 output
CONFIGS = [(1, 41, 153), (1, 4187, 151), (1, 8477, 150), (1, 12555, 153), (1, 17011, 258), (826, 139, 154), (17, 6227, 155),
           (17, 8615, 161), (68, 4924, 157), (221, 3298, 170), (848, 202, 165), (33, 6517, 163), (67, 5501, 157),
           (241, 2063, 150), (194, 3497, 277), (354, 2703, 261), (294, 1628, 155), (306, 2373, 154), (345, 2590, 271),
           (197, 4897, 390), (150, 5275, 266), (232, 5217, 391), (267, 2706, 242), (265, 4065, 274)]
MX_CONFIGS = {1: (1, 41, 300), 3: (385, 530, 582), 4: (1013, 267, 301), 6: (523, 135, 326), 8: (821, 387, 414),
              9: (1015, 663, 710), 11: (722, 266, 303), 13: (810, 518, 543), 15: (960, 1061, 1063), 18: (868, 785, 878),
              21: (1014, 1026, 1103)}


@pytest.mark.parametrize("config", range(len(CONFIGS)))
def test_every_tile(capfd, config):
    _, ps = plans(capfd, lambda: test_expand(*CONFIGS[config]))
    assert len(ps) == 2 and all(p["out_mx"] == 0 and p["small"] == config for p in ps), ps


@pytest.mark.parametrize("config", MX_CONFIGS)
def test_every_tile_project(capfd, config):
    _, ps = plans(capfd, lambda: test_project(*MX_CONFIGS[config]))
    assert len(ps) == 2 and all(p["out_mx"] == 1 and p["small"] == config for p in ps), ps


@pytest.mark.parametrize("M,K,L,N", [(2200, 1500, 700, 8), (22016, 1024, 640, 201), (24576, 2000, 1000, 512)])
def test_layer(M, K, L, N):
    """The layer (Z in plain rows or row pairs) equals projection, then expansion."""
    need_gpu()
    g = torch.Generator(device="cuda").manual_seed(N)
    X, Pt, Wf = (quantized(r, c, g, True) for r, c in ((N, K), (L, K), (M, L)))
    Y = espace.espace_projected_linear_mxfp8(X, Pt, Wf)
    assert torch.equal(Y, espace.espace_expand_mxfp8(espace.espace_project_mxfp8(Pt, X), Wf))
