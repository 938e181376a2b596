"""GPU: long dot products over shared operands, a block of outputs per
workgroup: rows and columns that do not fill the blocks, K that ends inside a
round of the threads, and blocks along a batch label that one operand does
not have (slices)."""
import numpy as np
import pytest

from tests.gpu_util import assert_close, assert_gemm_close, from_dev, split_elem_bound, gemm_elem_bound, to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2606_01852_amd import tnc  # noqa: E402


@pytest.fixture(scope="module")
def ctx():
    c = tnc.Context(0, arena_bytes=2 << 30)
    yield c
    c.close()


def cn(rng, shape):
    z = rng.standard_normal(tuple(shape) + (2,), dtype=np.float32) * np.float32(np.sqrt(0.5))
    return z.view(np.complex64).reshape(shape)


@pytest.mark.parametrize("prec", [tnc.PREC_C64, tnc.PREC_BF16X3], ids=["c64", "bf16x3"])
@pytest.mark.parametrize("shape", [(256, 8, 8, 2048), (700, 7, 7, 1000), (1000, 3, 8, 1500), (1100, 12, 3, 1025),
                                   (512, 4, 4, 4097), (2100, 2, 8, 1023), (515, 32, 2, 1111), (2300, 8, 2, 999)], ids=str)
def test_blocks_of_outputs(ctx, shape, prec):
    h, m, n, k = shape
    rng = np.random.Generator(np.random.PCG64(m * n + k))
    A, B = cn(rng, (h, m, k)), cn(rng, (h, n, k))
    Ad, Bd = to_dev(torch, A), to_dev(torch, B)
    Cd = torch.full((h, m, n, 2), float("nan"), dtype=torch.float32, device="cuda")
    torch.cuda.synchronize()
    print(shape, flush=True)
    tnc.tnc_batched_cgemm(ctx.handle, h, m, n, k, Ad.data_ptr(), m * k, Bd.data_ptr(), n * k, Cd.data_ptr(), prec,
                          tnc.GEMM_4M)
    ctx.sync()
    got = from_dev(Cd).view(np.complex64).reshape(h, m, n)
    ref = np.matmul(A.astype(np.complex128), B.astype(np.complex128).transpose(0, 2, 1))
    if prec == tnc.PREC_C64:
        # a thread's chain of k / 256 terms and a tree of 8 levels
        assert_gemm_close(got, ref, A, B, tol=2.0 ** -24 * (2 * np.sqrt(k / 256) + 10))
    else:
        assert np.all(np.abs(got - ref) <= split_elem_bound(A, B) + gemm_elem_bound(A, B))


@pytest.mark.parametrize("wide", ["n", "m"])
def test_blocks_along_a_sliced_label(ctx, wide):
    """sum over s1, s2 of A[s1, s2, k] B[s1, k, x] E[s2], A and B first (and the
    same with their order exchanged): s2 is a batch label that B lacks."""
    s1, s2, k, x = 0, 1, 2, 3
    ext = np.array([256, 8, 2048, 8])
    rng = np.random.Generator(np.random.PCG64(17))
    labels = [(s1, s2, k), (s1, k, x), (s2,)] if wide == "n" else [(s1, x, k), (s1, s2, k), (s2,)]
    leaves = [cn(rng, [ext[l] for l in lab]) for lab in labels]
    tn = tnc.Network(ctx, labels, ext, (x,), leaves)
    plan = tnc.Plan(tn, np.array([[0, 1], [3, 2]]), (s1, s2))
    assert plan.info.max_chunk == 2048
    step = tnc.tnc_plan_get_batch_step(plan.handle, 0)
    assert step.kernel == 2 and step.h == 2048 and step.split == 1
    print(wide, flush=True)
    got = plan.contract()
    P, Q, E = (a.astype(np.complex128) for a in leaves)
    if wide == "n":
        ref = np.tensordot(np.tensordot(P, E, axes=([1], [0])), Q, axes=([0, 1], [0, 1]))
    else:
        ref = np.tensordot(P, np.tensordot(Q, E, axes=([1], [0])), axes=([0, 2], [0, 1]))
    assert_close(got, ref)
    plan.close()
    tn.close()
