"""GPU: stand-alone permutations issued back to back, nothing waited for in
between: each call's tables are built on the device in the one area that the
context (or, allocation-free, the GPU) keeps.  Bit-exact with
numpy.transpose over extents that are no powers of two, digits above 64,
16-byte pairs and single elements, and a call whose tables outgrow the
area."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2606_01852_amd import tnc  # noqa: E402

CASES = [
    ((2,) * 16, (3, 12, 0, 7, 1, 13, 9, 2, 15, 11, 5, 4, 10, 14, 8, 6)),
    ((3,) * 9, (8, 2, 5, 0, 7, 1, 4, 6, 3)),
    ((5, 7, 11, 13, 3), (4, 1, 3, 0, 2)),
    ((64, 128, 96), (2, 0, 1)),
    ((100, 6, 90, 2), (1, 2, 0, 3)),          # the innermost pair stays: 16-byte pairs
    ((40, 10, 9, 2, 3), (1, 0, 2, 4, 3)),     # pairs of one run of 3 * 2, of different innermost modes
    ((9, 350, 33), (2, 1, 0)),                # 350 = 50 * 7, odd extents
    ((17, 8, 1, 24, 10), (3, 2, 0, 4, 1)),
    ((64, 48, 128), (1, 0, 2)),               # both runs in one mode: tiles that go on beyond it
    ((2,) * 18, (5, 0, 11, 3, 9, 1, 10, 4, 2, 8, 7, 6, 16, 13, 17, 12, 15, 14)),
    ((6,) * 7, (3, 0, 2, 1, 4, 6, 5)),        # runs of 36
    ((9, 10, 10, 10, 10, 10), (2, 0, 1, 3, 5, 4)),
    ((3, 70001, 2, 8), (1, 0, 3, 2)),         # more tiles than 16 bits count
    ((3, 4, 5), (2, 0, 1)),                   # plain gather
    ((1 << 17, 64, 64), (0, 2, 1)),           # 2 MiB of tables
]


@pytest.mark.parametrize("noalloc", [False, True], ids=["permute", "noalloc"])
def test_calls_in_a_row_keep_their_own_tables(noalloc):
    ctx = tnc.Context(0, stream=torch.cuda.current_stream().cuda_stream)
    call = tnc.tnc_permute_noalloc if noalloc else tnc.tnc_permute
    cases = CASES[:-1] if noalloc else CASES
    rng = np.random.Generator(np.random.PCG64(7))
    xs = [rng.integers(0, 1 << 62, size=ext) for ext, _ in cases]
    for rep in range(2):                      # 16-byte aligned operands, then ones that are not
        xd = [torch.empty(x.size + 1, dtype=torch.int64, device="cuda")[rep:rep + x.size] for x in xs]
        for d, x in zip(xd, xs):
            d.copy_(torch.from_numpy(x.reshape(-1)))
        yd = [torch.full((x.size + 1,), -1, dtype=torch.int64, device="cuda")[rep:rep + x.size] for x in xs]
        for i, (ext, perm) in enumerate(cases):
            print(f"{ext} {perm}", flush=True)
            call(ctx.handle, xd[i].data_ptr(), yd[i].data_ptr(), ext, perm)
        torch.cuda.synchronize()
        for i, (ext, perm) in enumerate(cases):
            assert np.array_equal(yd[i].cpu().numpy(), np.transpose(xs[i], perm).reshape(-1)), (rep, ext, perm)
    ctx.close()


def test_capture_takes_what_it_took():
    """Under capture a permutation that needs tiles is refused, and one whose
    tiles are only faster runs as a plain gather."""
    side = torch.cuda.Stream()
    ctx = tnc.Context(0, stream=side.cuda_stream)
    x = torch.arange(64 * 48 * 128, dtype=torch.int64, device="cuda")
    y = torch.zeros_like(x)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        tnc.tnc_permute(ctx.handle, x.data_ptr(), y.data_ptr(), (64, 48, 128), (1, 0, 2))
        with pytest.raises(tnc.TncError):
            tnc.tnc_permute(ctx.handle, x.data_ptr(), y.data_ptr(), (64, 48, 128), (2, 1, 0))
    ref = x.view(64, 48, 128).permute(1, 0, 2).reshape(-1)
    for rep in range(3):
        y.zero_()
        torch.cuda.synchronize()
        print("replay", rep, flush=True)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, ref)
    del g
    ctx.close()
