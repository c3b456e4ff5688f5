"""The float32 product at the edges of its kernels: each tile shape with
ragged rows, columns and depths, against a float64 product."""
import pytest
import torch

from tests.gpu_util import need_gpu

import paper_2410_05437_amd as espace

pytestmark = pytest.mark.gpu

# (tokens, output columns, depth); with 256 CUs: 128 x 128 tiles (272 and 256 of
# them), 64 x 64 tiles (176, 128), 32 x 32 blocks (175, 160) and 16 x 16 blocks
SHAPES = [(2049, 1930, 37), (2048, 2048, 64), (700, 1000, 70), (512, 1024, 33), (130, 1100, 100), (160, 1020, 257),
          (17, 300, 66), (16, 4099, 31), (5000, 7, 40), (1, 1, 1), (1, 2049, 1023), (33, 16, 520),
          # many columns or rows against up to 16 (16 x 16 blocks), up to 32 (32 x 32
          # blocks; 64 x 64 tiles at shallow depths) and up to 64 of the other
          (1, 33001, 300), (33001, 7, 300), (17, 9001, 290), (9001, 32, 290), (24, 40003, 130), (40003, 30, 64),
          (50, 40003, 70), (40003, 64, 70)]


def mat(rows, cols, g):
    """rows x cols with NaN in the padding columns."""
    ld = (cols + 3) // 4 * 4
    t = torch.full((rows, ld), float("nan"), device="cuda")
    t[:, :cols] = torch.randn(rows, cols, generator=g, device="cuda")
    return t[:, :cols]


@pytest.mark.parametrize("R,C,D", SHAPES)
def test_f32_product(R, C, D):
    need_gpu()
    g = torch.Generator(device="cuda").manual_seed(R * 31 + C)
    X, W = mat(R, D, g), mat(C, D, g)
    Y = espace.padded_empty(R, C, torch.float32, X.device, 4)
    whole = torch.as_strided(Y, (R, Y.stride(0)), (Y.stride(0), 1))
    whole.fill_(float("nan"))
    espace.espace_dense_linear(X, W, Y=Y)
    ref = X.double() @ W.double().t()
    # fp32 products and sums in any order: D + 8 roundings of at most 2^-24 each
    bound = (D + 8) * 2.0 ** -24 * (X.double().abs() @ W.double().abs().t())
    assert bool(((Y.double() - ref).abs() <= bound).all())
    assert bool(whole[:, C:].isnan().all())      # nothing written past a row


@pytest.mark.parametrize("R,C", [(1, (1 << 26) + 5), ((1 << 26) + 5, 1)])
def test_f32_more_blocks_than_a_launch(R, C):
    need_gpu()
    X = torch.randn(R, 4, device="cuda")
    W = torch.randn(C, 4, device="cuda")
    Y = espace.padded_empty(R, C, torch.float32, "cuda", 4).fill_(float("nan"))
    espace.espace_dense_linear(X, W, Y=Y)
    ref = X.double() @ W.double().t()
    assert bool(((Y.double() - ref).abs() <= 12 * 2.0 ** -24 * (X.double().abs() @ W.double().abs().t())).all())


@pytest.mark.parametrize("R,C,D", [(700, 1000, 70), (130, 1100, 100), (17, 300, 66)])
def test_f32_special_values(R, C, D):
    """Subnormal, infinite and NaN entries give what float32 arithmetic gives."""
    need_gpu()
    g = torch.Generator(device="cuda").manual_seed(5)
    X, W = mat(R, D, g).clone(), mat(C, D, g).clone()
    X[0] = 0.0
    X[0, D - 1] = 2.0 ** -140                    # subnormal times 1, 3: exact in float32
    W[:, D - 1] = 1.0
    W[1, D - 1] = 3.0
    X[1, 2] = float("inf")
    X[2, D - 2] = float("nan")
    pad = lambda t: espace.padded_empty(t.shape[0], t.shape[1], t.dtype, t.device, 4).copy_(t)  # noqa: E731
    Y = espace.espace_dense_linear(pad(X), pad(W))
    assert Y[0, 0].item() == 2.0 ** -140 and Y[0, 1].item() == 3 * 2.0 ** -140
    assert bool((Y[1] == torch.sign(W[:, 2]) * float("inf")).all())
    assert bool(Y[2].isnan().all())
    assert bool(Y[3:].isfinite().all())
