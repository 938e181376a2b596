"""GPU: split precision's 4M tiles keep the cross products' sums apart.

A = 1 + 2^-9 + 2^-16 (hi = 1, lo the rest), B = 1, K = 16384: the hi hi
products add up exactly in one sum (integers), the cross products exactly in
another (multiples of 2^-16 below 2^6), so the result is off by one rounding.
Added to the hi hi sum as they come, each MFMA's 16 (2^-9 + 2^-16) loses its
last bits there once the sum passes 2^12: 2^-16 of the result in the end.
"""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2606_01852_amd import tnc  # noqa: E402

X, K = 1 + 2.0 ** -9 + 2.0 ** -16, 16384


@pytest.fixture(scope="module")
def ctx():
    c = tnc.Context(0, arena_bytes=64 << 20)
    yield c
    c.close()


# every tile but 256 x 128, which has one sum; then what a call gets by
# itself, among them sizes that fill the chip with 256-row tiles
@pytest.mark.parametrize("variant, m, n", [(v, 300, 130) for v in (0, 1, 2, 4, 5, 6)] +
                         [(-1, 1024, 1024), (-1, 2048, 1024), (-1, 4096, 2048), (-1, 4096, 4096)], ids=str)
def test_cross_products_have_their_own_sum(ctx, variant, m, n):
    A = torch.full((m, K), X, dtype=torch.complex64, device="cuda")
    B = torch.full((n, K), 1.0, dtype=torch.complex64, device="cuda")
    C = torch.full((m, n), float("nan"), dtype=torch.complex64, device="cuda")
    torch.cuda.synchronize()
    print(variant, m, n, flush=True)
    tnc.tnc_ctx_set_gemm_variant(ctx.handle, variant)
    try:
        tnc.tnc_batched_cgemm(ctx.handle, 1, m, n, K, A.data_ptr(), 0, B.data_ptr(), 0, C.data_ptr(), tnc.PREC_BF16X3,
                              tnc.GEMM_4M)
        ctx.sync()
    finally:
        tnc.tnc_ctx_set_gemm_variant(ctx.handle, -1)
    r = torch.view_as_real(C).double()
    assert float((r[..., 0] - K * X).abs().max()) <= 2.0 ** -24 * K * X
    assert not bool(r[..., 1].any())
