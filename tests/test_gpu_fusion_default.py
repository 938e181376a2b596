"""GPU: what the server fuses unasked (tnc_serve_set_fusion never called)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2606_01852_amd import tnc  # noqa: E402
from workloads.circuits import circuit_network, random_circuit  # noqa: E402
from workloads.paths import greedy_path, greedy_slice  # noqa: E402


def test_default_fuses_only_what_gains():
    """Queued behind a slow request on one slot: six 4x5 circuits of depth 10
    (2.2e7 FLOP per launch, 1.13 times the rate when fused) run as one job,
    six of depth 12 (1.4e8, 0.96) one by one; the binding's constant says so too."""
    ctx = tnc.Context(0, arena_bytes=8 << 30)
    held, items, below = [], [], []

    def plan(rows, cols, depth, seed, sliced):
        net = circuit_network(random_circuit(rows, cols, depth, seed=seed))
        path = greedy_path(net)
        tn = tnc.Network(ctx, net.labels, net.extents, net.open, net.c64().leaves)
        p = tnc.Plan(tn, path.pairs, greedy_slice(net, path.pairs, n_sliced=sliced))
        held.append((tn, p))
        return p, tnc.tnc_plan_get_info(p.handle)

    blocker, blocker_info = plan(6, 6, 10, 8100, 4)
    for depth in (10, 12):
        for seed in range(6):
            p, info = plan(4, 5, depth, 8500 + seed, 1)
            items.append((p, info.n_slices))
            below.append(info.flops_per_slice * info.n_slices < info.n_launches * tnc.FUSE_FLOPS_PER_LAUNCH)
    assert below == [True] * 6 + [False] * 6
    tnc.tnc_serve_start(ctx.handle, 1, 64)
    outs = [np.zeros(1, dtype=np.complex128) for _ in range(13)]
    ids = [tnc.tnc_submit(ctx.handle, blocker.handle, 0, blocker_info.n_slices, outs[12])]
    ids += [tnc.tnc_submit(ctx.handle, p.handle, 0, n, o) for (p, n), o in zip(items, outs)]
    for i in ids:
        tnc.tnc_wait(ctx.handle, i)
    stats = tnc.tnc_serve_get_stats(ctx.handle)
    tnc.tnc_serve_stop(ctx.handle)
    print(f"default fusion: {stats}", flush=True)
    assert stats == (1 + 1 + 6, 1, 6)
    for tn, p in held:
        p.close()
        tn.close()
    ctx.close()
