"""Which kernel and tile a planned step gets (host-only plans)."""
import numpy as np
import pytest

from paper_2606_01852_amd import tnc

MFMA, SMALL = 0, 1


@pytest.fixture(scope="module")
def ctx():
    c = tnc.Context(-1, arena_bytes=64 << 30)
    yield c
    c.close()


def step(ctx, h, m, n, k, prec, form):
    """The one step of a batch of h products [m, k] x [k, n]."""
    net = tnc.Network(ctx, [(0, 1, 3), (0, 2, 3)], np.array([h, m, n, k], dtype=np.int64), (0, 1, 2), None)
    plan = tnc.Plan(net, [(0, 1)], (), prec, form)
    s = tnc.tnc_plan_get_step(plan.handle, 0)
    plan.close()
    net.close()
    return s


@pytest.mark.parametrize("h, m, n, k", [(2, 2048, 2048, 512), (8, 1024, 1024, 256), (3, 2560, 1280, 300), (64, 500, 120, 777),
                                        (40, 256, 128, 2000), (9, 1500, 2048, 700), (64, 1024, 512, 64), (2, 4096, 8192, 64)])
def test_split_precision_keeps_two_sums_unless_it_had_one(ctx, h, m, n, k):
    """The 256 x 128 tile (3), whose products share one sum, only where 1024
    of it with little padding cover the step."""
    s = step(ctx, h, m, n, k, tnc.PREC_BF16X3, tnc.GEMM_4M)
    assert s.kernel == MFMA
    rows, cols = (s.n, s.m) if s.swapped else (s.m, s.n)
    tiles = s.h * -(-rows // 256) * -(-cols // 128)
    full = rows * cols * s.h / (tiles * 256 * 128)
    if s.variant == 3:
        assert tiles >= 1024 and full >= 0.875


@pytest.mark.parametrize("h, m, n, k", [(1, 16, 256, 256), (1, 60, 31, 512), (4, 16, 16, 1024), (1, 63, 31, 200)])
@pytest.mark.parametrize("prec, form, kernel", [(tnc.PREC_C64, tnc.GEMM_4M, MFMA), (tnc.PREC_C64, tnc.GEMM_3M, MFMA),
                                                (tnc.PREC_BF16X3, tnc.GEMM_4M, MFMA), (tnc.PREC_BF16X3, tnc.GEMM_3M, SMALL)],
                         ids=["c64_4M", "c64_3M", "bf16x3_4M", "bf16x3_3M"])
def test_few_outputs_and_a_long_k(ctx, h, m, n, k, prec, form, kernel):
    """On MFMA only where its kernels share K out; split precision's 3M tiles
    do not (and would round more than one thread per output does)."""
    assert step(ctx, h, m, n, k, prec, form).kernel == kernel


def chain(ctx, n_pairs, d, e, k, prec=tnc.PREC_C64, grouping=True):
    """Kernels of the first level of (A0 B0) (A1 B1) ...: n_pairs steps [d, k] x [k, e] or [e, k] x [k, d]."""
    ext, lab = [d if i % 2 == 0 else e for i in range(n_pairs + 1)], []
    for p in range(n_pairs):
        lab += [(p, n_pairs + 1 + p), (p + 1, n_pairs + 1 + p)]
        ext.append(k)
    pairs, ids, nxt = [(2 * p, 2 * p + 1) for p in range(n_pairs)], [2 * n_pairs + p for p in range(n_pairs)], 3 * n_pairs
    while len(ids) > 1:
        pairs += [(ids[i], ids[i + 1]) for i in range(0, len(ids) - 1, 2)]
        ids, nxt = list(range(nxt, nxt + len(ids) // 2)) + ids[len(ids) // 2 * 2:], nxt + len(ids) // 2
    net = tnc.Network(ctx, lab, np.array(ext, dtype=np.int64), (0, n_pairs), None)
    plan = tnc.Plan(net, pairs, (), prec, tnc.GEMM_4M)
    tnc.tnc_plan_set_grouping(plan.handle, grouping)
    kinds = [tnc.tnc_plan_get_step(plan.handle, s).kernel for s in range(n_pairs)]
    plan.close()
    net.close()
    return kinds


@pytest.mark.parametrize("d, e, k", [(16, 256, 256), (32, 32, 512), (16, 64, 256), (16, 1024, 128)])
@pytest.mark.parametrize("prec", [tnc.PREC_C64, tnc.PREC_BF16X3], ids=["c64", "bf16x3"])
def test_a_level_full_of_long_k_steps_shares_its_launch(ctx, d, e, k, prec):
    """A launch each only while that is less than the level's one launch of
    one thread per output, whatever the grouping."""
    for n_pairs in (1, 2, 8, 32):
        for grouping in (True, False):
            want = MFMA if 112 * n_pairs <= k else SMALL
            assert chain(ctx, n_pairs, d, e, k, prec, grouping) == [want] * n_pairs, (n_pairs, grouping)


TILES = [(128, 64), (256, 64), (128, 128), (256, 128), (64, 64), (128, 32), (64, 32)]


@pytest.mark.parametrize("h, m, n, k", [(4096, 32, 32, 128), (1738, 39, 31, 134), (579, 33, 51, 460), (134, 35, 193, 308),
                                        (7301, 18, 97, 46), (145, 34, 538, 916), (3777, 44, 63, 290), (2000, 64, 64, 64)])
def test_split_3m_does_not_pad_small_steps_to_large_tiles(ctx, h, m, n, k):
    """Batches of small steps on a tile that pads them no more than 64 x 64
    does (all of these ran longer on 128 x 64)."""
    s = step(ctx, h, m, n, k, tnc.PREC_BF16X3, tnc.GEMM_3M)
    assert s.kernel == MFMA
    rows, cols = (s.n, s.m) if s.swapped else (s.m, s.n)
    padded = [-(-rows // bm) * bm * -(-cols // bn) * bn for bm, bn in TILES]
    assert padded[s.variant] <= padded[4], (s.variant, s.swapped)


@pytest.mark.parametrize("h, m, n, k, near_best", [(639, 64, 18, 203, (6,)), (579, 33, 51, 460, (4,)), (78, 403, 157, 740, (0, 1)),
                                                   (13, 356, 1918, 1094, (0, 2))])
def test_split_4m_tile_is_near_the_best(ctx, h, m, n, k, near_best):
    """Ragged extents: the tiles that were measured within 7 % of the best."""
    s = step(ctx, h, m, n, k, tnc.PREC_BF16X3, tnc.GEMM_4M)
    assert not s.swapped and s.variant in near_best
