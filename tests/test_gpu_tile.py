"""The large-tile Linear (k_tile.hip) against gemm_kernel's 64-row form, which sums in the same order: the results are the same
bits.  Shapes are ones whose own choice is a large tile (192 x 128 .. 256 x 256), rows and columns cut, one round of tiles and
several, K-tiles from 17 (more than the stages, an odd number) to 44."""
import pytest
import torch
from paper_2404_13528_amd import binding as sm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K,act,res,rope", [
    (4147, 928, 1088, "none", True, None),           # 128 x 192
    (834, 4672, 1088, "swiglu", False, None),
    (1292, 5440, 1280, "gelu", False, None),         # 128 x 256
    (4685, 832, 1088, "none", True, None),           # 192 x 128
    (5705, 656, 1088, "gelu", True, None),
    (1677, 4680, 1088, "gelu", False, None),         # 192 x 192
    (3335, 2368, 1088, "geglu", True, None),
    (2148, 4096, 1088, "swiglu", False, None),       # 192 x 256
    (5436, 1544, 1088, "gelu", True, None),          # 256 x 192
    (2041, 8184, 1088, "none", True, None),          # 256 x 256, one round
    (2041, 6144, 1088, "none", False, (4096, 128, 700, 10000.0)),
    (4100, 9984, 1088, "swiglu", True, None),        # several rounds
    (333, 5632, 2816, "swiglu", False, None),        # few rows
    (6304, 2304, 768, "none", True, None),           # a short K
])
def test_tile_linear_is_the_tiled_kernel(M, N, K, act, res, rope):
    g = torch.Generator().manual_seed(M + N + K)
    A, W = torch.randn(M, K, generator=g).bfloat16().cuda(), (torch.randn(N, K, generator=g) * K ** -0.5).bfloat16().cuda()
    b = None if rope else torch.randn(N, generator=g).bfloat16().cuda()
    R = torch.randn(M, N // 2 if "glu" in act else N, generator=g).bfloat16().cuda() if res else None
    got = sm.linear(A, W, b, residual=R, act=act, rope=rope)
    again = sm.linear(A, W, b, residual=R, act=act, rope=rope)
    try:
        sm.gemm_tuning(64, 2)
        want = sm.linear(A, W, b, residual=R, act=act, rope=rope)
    finally:
        sm.gemm_tuning(0, 0)
    assert torch.isfinite(want.float()).all()
    assert torch.equal(got, want) and torch.equal(again, want)
