"""GPU: 4M GEMMs over float32's whole range, on the tiles and on the shapes for
few tiles.

A sum whose partial sums in order stay finite is finite, however the kernel
shares K out.  In complex64, scaling an operand by a power of two scales the
result, bit for bit, as long as nothing leaves float32's range, and one value
far below the others changes no other row's bits; values down to float32's
smallest keep every bit against a large partner.
"""
import numpy as np
import pytest

from tests.gpu_util import from_dev, to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2606_01852_amd import tnc  # noqa: E402

# by default: the shapes for few tiles (32 x 16, 32 x 32, 64 x 32 complex),
# then tiles; k ends inside a stage of 8 in some
FEW = [(1, 64, 32, 128), (10, 128, 128, 133), (20, 128, 128, 128)]
TILED = [(v, (3, 300, 161, 137)) for v in range(7)]
CALLS = [(-1, s) for s in FEW] + TILED


@pytest.fixture(scope="module")
def ctx():
    c = tnc.Context(0, arena_bytes=64 << 20)
    yield c
    c.close()


def cn(rng, shape):
    return (rng.standard_normal(shape + (2,), dtype=np.float32) * np.float32(np.sqrt(0.5))).view(np.complex64).reshape(shape)


def operands(shape):
    h, m, n, k = shape
    rng = np.random.Generator(np.random.PCG64(m * 17 + k))
    return cn(rng, (h, m, k)), cn(rng, (h, n, k))


def gemm(ctx, A, B, variant, prec=tnc.PREC_C64):
    (h, m, k), n = A.shape, B.shape[1]
    Ad, Bd = to_dev(torch, A), to_dev(torch, B)
    Cd = torch.full((h, m, n, 2), float("nan"), dtype=torch.float32, device="cuda")
    torch.cuda.synchronize()
    tnc.tnc_ctx_set_gemm_variant(ctx.handle, variant)
    try:
        tnc.tnc_batched_cgemm(ctx.handle, h, m, n, k, Ad.data_ptr(), m * k, Bd.data_ptr(), n * k, Cd.data_ptr(),
                              prec, tnc.GEMM_4M)
        ctx.sync()
    finally:
        tnc.tnc_ctx_set_gemm_variant(ctx.handle, -1)
    return from_dev(Cd).reshape(h, m, n, 2)


@pytest.mark.parametrize("prec", [tnc.PREC_C64, tnc.PREC_BF16X3], ids=["c64", "bf16x3"])
@pytest.mark.parametrize("variant, shape", CALLS, ids=str)
def test_partial_sums_stay_finite(ctx, variant, shape, prec):
    """+a +a . -a -a +a +a . +a -a -a over sixteen stages of eight k, a = 2^126:
    in order never above 3 a, but a sum over the stages 0, 8, 1, 9 alone is
    4 a, which no float32 holds."""
    h, m, n, _ = shape
    A, B = np.zeros((h, m, 128), np.complex64), np.ones((h, n, 128), np.complex64)
    for stage, sign in ((0, 1), (1, 1), (6, -1), (7, -1), (8, 1), (9, 1), (12, 1), (14, -1), (15, -1)):
        A[:, :, 8 * stage] = sign * 2.0 ** 63
    B *= np.float32(2.0 ** 63)
    print(variant, shape, flush=True)
    got = gemm(ctx, A, B, variant, prec)
    assert np.all(got[..., 0] == np.float32(2.0 ** 126)) and not np.any(got[..., 1])


@pytest.mark.parametrize("variant, shape", CALLS, ids=str)
@pytest.mark.parametrize("ea, eb", [(-100, 60), (60, -100), (45, 45), (-60, -20)])
def test_a_power_of_two_scales_the_bits(ctx, variant, shape, ea, eb):
    """Every operand value keeps its 24 bits above 2^-149 (values of CN(0, 1)
    below 2^-20 are set to zero), and so does every result."""
    A, B = operands(shape)
    for X in (A, B):
        f = X.view(np.float32)
        f[np.abs(f) < 2.0 ** -20] = 0
    print(variant, shape, ea, eb, flush=True)
    ref = gemm(ctx, A, B, variant)
    ref[np.abs(ref) < 2.0 ** -20] = 0   # below it a scaled result may round to a subnormal
    got = gemm(ctx, A * np.float32(2.0 ** ea), B * np.float32(2.0 ** eb), variant)
    got = got * np.float32(2.0 ** -(ea + eb))
    got[np.abs(got) < 2.0 ** -20] = 0
    np.testing.assert_array_equal(got, ref)


@pytest.mark.parametrize("variant, shape", CALLS, ids=str)
def test_a_tiny_value_leaves_other_rows_alone(ctx, variant, shape):
    """One value of the size of a product of two entries that should have been
    zero (6.1e-17 each), and one of full length near the smallest normal: the
    other rows' bits are those without them."""
    A, B = operands(shape)
    print(variant, shape, flush=True)
    ref = gemm(ctx, A, B, variant)
    A2 = A.copy()
    A2[0, 5, 3] = complex(np.float32(6.123234e-17) * np.float32(6.123234e-17), 1.3e-37)
    got = gemm(ctx, A2, B, variant)
    rows = np.ones(A.shape[:2], dtype=bool)
    rows[0, 5] = False
    np.testing.assert_array_equal(got[rows], ref[rows])


@pytest.mark.parametrize("variant, shape", CALLS, ids=str)
def test_small_values_keep_every_bit(ctx, variant, shape):
    """Values whose parts bf16 holds as subnormals or not at all, alone in
    their rows, against 2^100."""
    A, B = operands(shape)
    small = [2.0 ** -140, 2.0 ** -130, 2.0 ** -115 + 2.0 ** -130, 2.0 ** -149, float(np.float32(1.3e-37)),
             2.0 ** -126 - 2.0 ** -149, float(np.float32(3.7e-33))]
    l = A.shape[2] - 1
    for i, x in enumerate(small):
        A[0, 7 + i] = 0
        A[0, 7 + i, l] = np.float32(x)
    B[0, 9, l] = np.float32(2.0 ** 100)
    print(variant, shape, flush=True)
    got = gemm(ctx, A, B, variant)
    for i, x in enumerate(small):
        assert got[0, 7 + i, 9, 0] == np.float32(x * 2.0 ** 100) and got[0, 7 + i, 9, 1] == 0, x


@pytest.mark.parametrize("m", [128, 1024])
def test_small_values_in_a_fused_job(m):
    """The same through the server, where the steps of several requests share
    a launch: every request's result is bitwise its result alone."""
    ctx = tnc.Context(0, arena_bytes=1 << 30)
    rng = np.random.Generator(np.random.PCG64(m))
    nets, plans, k = [], [], 64
    for r in range(6):
        A, B = cn(rng, (m, k)), cn(rng, (m, k))
        A[7] = 0
        A[7, k - 1] = np.float32(2.0 ** -115 + 2.0 ** -130)
        A[8, 3] = np.inf if r == 2 else 1.3e-37
        B[9, k - 1] = np.float32(2.0 ** 100)
        nets.append(tnc.Network(ctx, [(0, 2), (1, 2)], np.array([m, m, k], dtype=np.int64), (0, 1), [A, B]))
        plans.append(tnc.Plan(nets[-1], [(0, 1)]))
    print(f"m {m}: variant {tnc.tnc_plan_get_step(plans[0].handle, 0).variant}", flush=True)
    alone = [p.contract() for p in plans]
    tnc.tnc_serve_start(ctx.handle, 1, 64)
    tnc.tnc_serve_set_fusion(ctx.handle, 8, tnc.FUSE_ALL)
    outs = [np.zeros(m * m, dtype=np.complex128) for _ in plans]
    ids = [tnc.tnc_submit(ctx.handle, p.handle, 0, 1, o) for p, o in zip(plans, outs)]
    for i in ids:
        tnc.tnc_wait(ctx.handle, i)
    fused = tnc.tnc_serve_get_stats(ctx.handle)[1]
    tnc.tnc_serve_stop(ctx.handle)
    assert fused >= 1
    for r, (o, a) in enumerate(zip(outs, alone)):
        np.testing.assert_array_equal(o.view(np.float64), np.asarray(a).reshape(-1).view(np.float64), err_msg=str(r))
        assert o.reshape(m, m)[7, 9] == 2.0 ** -15 + 2.0 ** -30
    for p, t in zip(plans, nets):
        p.close()
        t.close()
    ctx.close()
