"""GPU: split precision (bf16 hi + lo) on the 4M kernels' tile shapes and on
the shapes for few tiles, and complex64 in the 3M form on the same kernels.

Split precision is checked at the edges of tiles and of K stages (8 complex)
against the elementwise bound of its arithmetic; the 3M form of complex64
gives bitwise what its 4M form gives.
"""
import numpy as np
import pytest

from tests.gpu_util import from_dev, gemm_elem_bound, rel_fro, split_elem_bound, to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2606_01852_amd import tnc  # noqa: E402


@pytest.fixture(scope="module")
def ctx():
    c = tnc.Context(0, arena_bytes=64 << 20)
    yield c
    c.close()


def operands(h, m, n, k):
    rng = np.random.Generator(np.random.PCG64(m * 31 + n * 7 + k))
    z = [(rng.standard_normal(s + (2,), dtype=np.float32) * np.float32(np.sqrt(0.5))).view(np.complex64).reshape(s)
         for s in ((h, m, k), (h, n, k))]
    return z[0], z[1]


def gemm(ctx, A, B, prec, form, variant=-1):
    (h, m, k), n = A.shape, B.shape[1]
    Ad, Bd = to_dev(torch, A), to_dev(torch, B)
    Cd = torch.full((h, m, n, 2), float("nan"), dtype=torch.float32, device="cuda")
    torch.cuda.synchronize()
    tnc.tnc_ctx_set_gemm_variant(ctx.handle, variant)
    try:
        tnc.tnc_batched_cgemm(ctx.handle, h, m, n, k, Ad.data_ptr(), m * k, Bd.data_ptr(), n * k, Cd.data_ptr(), prec, form)
        ctx.sync()
    finally:
        tnc.tnc_ctx_set_gemm_variant(ctx.handle, -1)
    return from_dev(Cd).view(np.complex64).reshape(h, m, n)


# the seven tiles at their edges; then, by default, the shapes with few tiles
# (eight waves share K out in stages of 8): a K shorter than the waves' first
# round, one that ends inside a stage, and one element more
TILES = [(v, s) for v in range(7) for s in ((96, 65, 33, 17), (40, 129, 63, 24), (2, 300, 161, 8 * 33 + 1), (3, 257, 129, 136))]
FEW = [(-1, s) for s in ((1, 64, 32, 129), (3, 90, 50, 321), (1, 512, 512, 24), (1, 500, 509, 67), (8, 1000, 61, 130), (1, 33, 47, 4099))]


@pytest.mark.parametrize("variant, shape", TILES + FEW, ids=str)
def test_split_precision(ctx, variant, shape):
    h, m, n, k = shape
    A, B = operands(h, m, n, k)
    print(f"variant {variant} {shape}", flush=True)
    got = gemm(ctx, A, B, tnc.PREC_BF16X3, tnc.GEMM_4M, variant).astype(np.complex128)
    ref = np.matmul(A.astype(np.complex128), B.astype(np.complex128).transpose(0, 2, 1))
    assert np.all(np.isfinite(got))
    # hi and lo hold 16 bits: each product is off by some 2^-17 of itself, in random directions
    assert rel_fro(got, ref) <= 2.0 ** -16 + 2 * np.sqrt(k) * 2.0 ** -24
    assert np.all(np.abs(got - ref) <= split_elem_bound(A, B) + gemm_elem_bound(A, B))


@pytest.mark.parametrize("shape", [(2, 300, 161, 265), (8, 1000, 61, 130), (96, 65, 33, 17)], ids=str)
def test_complex64_form_is_one(ctx, shape):
    A, B = operands(*shape)
    print(shape, flush=True)
    got = [gemm(ctx, A, B, tnc.PREC_C64, form) for form in (tnc.GEMM_4M, tnc.GEMM_3M)]
    np.testing.assert_array_equal(got[0].view(np.float32), got[1].view(np.float32))
