"""GPU: the complex64 4M GEMM on the bf16 pipe (exact three-way split).

Every element lies within the float32 accumulation bound 8 sqrt(k) 2^-24
||A_i|| ||B_j|| of the complex128 product on every tile shape, at the edges
of tiles and of K stages (8 complex), and inputs that the split cannot hold
(infinities, NaNs, values that round up to infinity in bf16, values whose
low bits bf16 cannot hold) give what float32 arithmetic gives.
"""
import numpy as np
import pytest

from tests.gpu_util import assert_gemm_close, from_dev, gemm_elem_bound, to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2606_01852_amd import tnc  # noqa: E402


@pytest.fixture(scope="module")
def ctx():
    c = tnc.Context(0, arena_bytes=64 << 20)
    yield c
    c.close()


def cn(rng, shape):
    z = rng.standard_normal(shape + (2,), dtype=np.float32) * np.float32(np.sqrt(0.5))
    return z.view(np.complex64).reshape(shape)


def gemm(ctx, A, B, variant=-1, form=tnc.GEMM_4M):
    (h, m, k), n = A.shape, B.shape[1]
    Ad, Bd = to_dev(torch, A), to_dev(torch, B)
    Cd = torch.full((h, m, n, 2), float("nan"), dtype=torch.float32, device="cuda")
    torch.cuda.synchronize()
    tnc.tnc_ctx_set_gemm_variant(ctx.handle, variant)
    try:
        tnc.tnc_batched_cgemm(ctx.handle, h, m, n, k, Ad.data_ptr(), m * k, Bd.data_ptr(), n * k, Cd.data_ptr(),
                              tnc.PREC_C64, form)
        ctx.sync()
    finally:
        tnc.tnc_ctx_set_gemm_variant(ctx.handle, -1)
    return from_dev(Cd).view(np.complex64).reshape(h, m, n)


def exact(A, B):
    return np.matmul(A.astype(np.complex128), B.astype(np.complex128).transpose(0, 2, 1))


@pytest.mark.parametrize("variant", range(7))
@pytest.mark.parametrize("shape", [(128, 64, 32, 16), (96, 65, 33, 17), (64, 127, 31, 23), (40, 129, 63, 25), (2, 300, 161, 8 * 33 + 1),
                                   (3, 257, 129, 136)], ids=str)
def test_every_tile_shape_at_its_edges(ctx, variant, shape):
    h, m, n, k = shape
    rng = np.random.Generator(np.random.PCG64(m * 131 + k))
    A, B = cn(rng, (h, m, k)), cn(rng, (h, n, k))
    print(f"variant {variant} {shape}", flush=True)
    got = gemm(ctx, A, B, variant)
    # six products a term, one rounding of the running sum per 16 terms: no
    # more than half of the float32 chain's 2 sqrt(k) 2^-24 in norm
    assert_gemm_close(got, exact(A, B), A, B, tol=2 * np.sqrt(k) * 2.0 ** -24 + 2.0 ** -24)
    real = gemm(ctx, A.real.astype(np.complex64), B.real.astype(np.complex64), variant)
    assert not np.any(real.imag)   # 4M: products of real operands are real


@pytest.mark.parametrize("variant", [0, 2, 3, 6])
def test_values_the_split_cannot_hold(ctx, variant):
    h, m, n, k = 8, 300, 150, 40
    rng = np.random.Generator(np.random.PCG64(5))
    A, B = cn(rng, (h, m, k)), cn(rng, (h, n, k))
    top = np.finfo(np.float32).max
    A[0, 3, 5] = np.inf
    A[1, 200, 1] = complex(1.0, np.nan)
    A[2, 299, :] = 0
    A[2, 299, k - 1] = top                    # rounds to a bf16 infinity
    B[2] *= np.float32(2.0 ** -30)
    A[3, 64:128] *= np.float32(2.0 ** -118)   # the last bits are below bf16's smallest
    B[3] *= np.float32(2.0 ** 60)
    A[4, 10, :] = 0
    A[4, 10, 7] = np.float32(2.0 ** -140)     # a subnormal, against a large value
    B[4, 20, 7] = np.float32(2.0 ** 100)
    A[5, 17] = 0                              # zeros are nothing special
    print(f"variant {variant}", flush=True)
    got = gemm(ctx, A, B, variant)
    a, b = A.astype(np.complex128), B.astype(np.complex128).transpose(0, 2, 1)
    with np.errstate(all="ignore"):
        re = np.matmul(a.real, b.real) - np.matmul(a.imag, b.imag)
        im = np.matmul(a.real, b.imag) + np.matmul(a.imag, b.real)
    finite_rows = np.ones((h, m), dtype=bool)
    finite_rows[0, 3] = finite_rows[1, 200] = False
    assert np.all(np.isnan(got[1, 200].real)) and np.all(np.isnan(got[1, 200].imag))
    np.testing.assert_array_equal(got[0, 3].real, re[0, 3].astype(np.float32))
    np.testing.assert_array_equal(got[0, 3].imag, im[0, 3].astype(np.float32))
    assert np.all(np.isfinite(got[finite_rows].view(np.float32)))
    A0 = np.where(np.isfinite(A), A, 0)
    bound = gemm_elem_bound(A0, B) + k * 2.0 ** -148
    with np.errstate(all="ignore"):
        within = np.abs(got - (re + 1j * im)) <= bound
    assert np.all(within[finite_rows])
    assert got[4, 10, 20] == np.complex64(2.0 ** -40)
    assert not np.any(got[5, 17])


# the shapes with few tiles (32 x 16, 32 x 32, 64 x 32 complex; eight waves
# share K out in stages of 8): edges of the tiles, a K shorter than the waves'
# first round, one that ends inside a stage, and one element more
FEW_TILES = [(1, 64, 32, 129), (1, 65, 33, 136), (3, 90, 50, 321), (1, 200, 100, 210), (1, 512, 512, 24), (1, 500, 509, 67),
             (9, 250, 130, 17), (8, 1000, 61, 130), (1, 16, 256, 256), (1, 33, 47, 4099)]


@pytest.mark.parametrize("shape", FEW_TILES, ids=str)
def test_few_tiles(ctx, shape):
    h, m, n, k = shape
    rng = np.random.Generator(np.random.PCG64(m * 7 + k))
    A, B = cn(rng, (h, m, k)), cn(rng, (h, n, k))
    print(shape, flush=True)
    got = gemm(ctx, A, B)
    assert_gemm_close(got, exact(A, B), A, B, tol=2 * np.sqrt(k) * 2.0 ** -24 + 2.0 ** -24)
    A[0, m - 1, k - 1] = np.inf       # the last element of the last row's last stage
    B[0, n - 1, 0] = np.float32(2.0 ** -140)
    got2 = gemm(ctx, A, B)
    assert not np.any(np.isfinite(got2[0, m - 1, :-1].real))
    rows = np.ones((h, m), dtype=bool)
    rows[0, m - 1] = False
    assert np.all(np.abs(got2 - exact(np.where(np.isfinite(A), A, 0), B))[rows] <=
                  gemm_elem_bound(np.where(np.isfinite(A), A, 0), B)[rows])
