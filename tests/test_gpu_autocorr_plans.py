"""The bfloat16 autocorrelation update at the edges of its plans: small tiles
of every width, 256 x 192 and 256 x 256 tiles, several depth ranges."""
import pytest
import torch

from tests.gpu_util import need_gpu

import paper_2410_05437_amd as espace

pytestmark = pytest.mark.gpu

# (K, tokens): small tiles from one block to many, ragged; tiles of 256 rows
SIZES = [(1, 1), (17, 33), (65, 5), (130, 700), (333, 64), (513, 9000), (700, 1000), (900, 300), (1537, 2500),
         (2000, 150), (2050, 3000), (2700, 515), (4100, 130)]


@pytest.mark.parametrize("K,N", SIZES)
@pytest.mark.parametrize("normalize", [False, True])
def test_update(K, N, normalize):
    need_gpu()
    g = torch.Generator(device="cuda").manual_seed(K + N)
    ld = (K + 7) // 8 * 8
    X = torch.full((N, ld), float("nan"), device="cuda", dtype=torch.bfloat16)[:, :K]
    X.copy_(torch.randn(N, K, generator=g, device="cuda"))
    C0 = torch.randn(K, K, generator=g, device="cuda")
    C0 = C0 + C0.t()
    C = espace.padded_empty(K, K, torch.float32, X.device, 4)
    whole = torch.as_strided(C, (K, C.stride(0)), (C.stride(0), 1)).fill_(float("nan"))
    C.copy_(C0)
    espace.espace_autocorrelation_update(X, C, 0.25, normalize=normalize)
    x = X.double()
    if normalize:
        x = x / x.norm(dim=1, keepdim=True)
    ref, mag = C0.double() + 0.25 * x.t() @ x, x.abs().t() @ x.abs()
    # fp32 sums of N exact products, the scaling and the addition to C; unit
    # tokens are rounded to bfloat16 first
    bound = 2.0 ** -23 * ref.abs() + 0.25 * ((N + 8) * 2.0 ** -24 + (2.0 ** -7 if normalize else 0.0)) * mag + 2.0 ** -23 * C0.abs()
    assert bool(((C.double() - ref).abs() <= bound).all())
    assert torch.equal(C, C.t())                     # exactly symmetric
    assert bool(whole[:, K:].isnan().all())


@pytest.mark.parametrize("K,N,limit", [(1069, 5679, 1.4e-7), (583, 5988, 1.15e-7), (648, 13694, 1.1e-7)])
def test_accuracy(K, N, limit):
    """The error against float64 on normal data grows with the length of a sum: 1.29e-7
    at K = 1069 in 18 steps of 64 tokens, 1.48e-7 in 23 (limits between the two)."""
    need_gpu()
    g = torch.Generator(device="cuda").manual_seed(K)
    X = espace.padded_empty(N, K, torch.bfloat16, "cuda")
    X.copy_(torch.randn(N, K, generator=g, device="cuda"))
    C = espace.padded_empty(K, K, torch.float32, "cuda", 4).zero_()
    espace.espace_autocorrelation_update(X, C, 1.0)
    ref = X.double().t() @ X.double()
    err = ((C.double() - ref).norm() / ref.norm()).item()
    print(f"K={K} N={N} {err:.3e}")
    assert err < limit
