"""Which kernel a bfloat16 product runs on where two were measured far apart (256 CUs,
operands rotated through HBM), and its result against a float64 product."""
import pytest
import torch

from tests.gpu_util import need_gpu, plans

import paper_2410_05437_amd as espace

pytestmark = pytest.mark.gpu

# rows, columns, depth; kernel, tile, depth ranges, pair; us there and on the kernel
# that an earlier rule took
CASES = [
    (512, 6144, 3686, "tiled", "128x192", 2, 1),        # 45, small tiles 57
    (128, 22016, 1536, "tiled", "128x192", 2, 1),       # 25, small tiles 30
    (201, 11392, 2688, "tiled", "128x192", 2, 1),       # 29, small tiles 36
    (48, 12288, 4096, "small", None, 1, 0),             # 23, 128 x 192 tiles in four ranges 30
    (282, 7701, 384, "tiled", "128x192", 1, 0),         # 9, small tiles 12
    (772, 8832, 20736, "tiled", "192x192", 1, 0),       # 318, 128 x 256 tiles 420
    (6702, 11008, 12032, "tiled", "256x256", 1, 0),     # 1542, 192 x 192 tiles 1636
    (6457, 640, 4736, "tiled", "128x128", 2, 1),        # 53, 128 x 192 tiles 58
    (4096, 1536, 11008, "tiled", "128x192", 1, 0),      # 130, pairs of 256 x 192 tiles 156
    (12288, 1536, 4096, "tiled", "192x192", 1, 0),      # 142, two launches by rows 149
    (1, 512, 8192, "gemv", None, 1, 0),                 # 4.6, small tiles 6.6
    (1, 5120, 8192, "gemv", None, 1, 0),                # 17.8, small tiles 18.8
    (1, 640, 12231, "gemv", None, 1, 0),                # 8.0, small tiles 10.1
    (1, 6144, 24576, "small", None, 1, 0),              # 54, in four ranges 60, streamed 58
    (1, 1536, 11008, "small", None, 1, 0),              # 10.0, streamed 10.7
    (2, 6144, 3686, "gemv", None, 1, 0),                # 12.0, small tiles 13.4
    (2, 16384, 8192, "gemv", None, 1, 0),               # 49.9, small tiles 52.2
    (2, 4096, 11008, "small", None, 1, 0),              # 18.6, streamed 25.4
    (3, 24576, 2458, "stream", None, 1, 0),             # 24.0, small tiles 25.9
    (8, 6144, 3686, "stream", None, 1, 0),              # 13.1, small tiles 14.9
    (16, 14336, 5000, "stream", None, 1, 0),            # small tiles 13% more
    (16, 24576, 1000, "stream", None, 1, 0),            # small tiles 7% more
    (16, 4096, 4096, "small", None, 1, 0),              # 9.0, streamed 11.1
    (8, 24600, 6144, "stream", None, 1, 0),             # the deepest it takes
    (16, 28000, 1536, "stream", None, 1, 0),            # 17.8, small tiles 19.8
]


def mat(rows, cols, g):
    """rows x cols bfloat16 with NaN in the padding columns."""
    ld = (cols + 7) // 8 * 8
    t = torch.full((rows, ld), float("nan"), device="cuda", dtype=torch.bfloat16)
    t[:, :cols] = torch.randn(rows, cols, generator=g, device="cuda")
    return t[:, :cols]


@pytest.mark.parametrize("R,C,D,kind,tile,splits,pair", CASES)
def test_plan(capfd, R, C, D, kind, tile, splits, pair):
    need_gpu()
    g = torch.Generator(device="cuda").manual_seed(R + C + D)
    X, W = mat(R, D, g), mat(C, D, g)
    Y, (p,) = plans(capfd, lambda: espace.espace_dense_linear(X, W))
    assert p["kind"] == kind and p["splits"] == splits and p["pair"] == pair and p["rows1"] == 0, p
    assert tile is None or p["tile"] == tile, p
    ref, mag = X.double() @ W.double().t(), X.double().abs() @ W.double().abs().t()
    # exact products, fp32 sums of D terms in any order, one rounding to bfloat16
    bound = 2.0 ** -8 * ref.abs() + (1 + 2.0 ** -8) * (D + 16) * 2.0 ** -23 * mag
    assert bool(((Y.double() - ref).abs() <= bound).all())
