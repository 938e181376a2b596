"""GPU: steps, split-K epilogues, reductions and results of a fused serving
job go out once for all its requests.  Every result is bitwise the one the
request gets alone, where the job ends in a dot product, a dot product with
K cut, a reduction over 128 slices, and results too large to be fetched in one
copy."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2606_01852_amd import tnc  # noqa: E402
from tests.test_gpu_serving import _serve_each  # noqa: E402
from workloads.circuits import circuit_network, random_circuit  # noqa: E402
from workloads.paths import greedy_path, greedy_slice  # noqa: E402

DOT = 2
# rows, cols, depth, sliced labels, open qubits -> what the plan must hold
CASES = {
    "dot": ((4, 5, 8, 0, 0), lambda st, info: any(s.kernel == DOT for s in st)),
    "split_dot": ((4, 5, 10, 0, 4), lambda st, info: any(s.kernel == DOT and s.split > 1 for s in st)),
    "split_gemm": ((4, 5, 10, 0, 0), lambda st, info: any(s.kernel == 0 and s.split > 1 for s in st)),
    "slices": ((4, 5, 10, 7, 0), lambda st, info: info.max_chunk >= 64),
    "large_results": ((4, 4, 8, 0, 14), lambda st, info: info.n_result * 16 * 5 > 1 << 20),
}


@pytest.mark.parametrize("prec", [tnc.PREC_C64, tnc.PREC_BF16X3], ids=["c64", "bf16x3"])
@pytest.mark.parametrize("name", CASES)
@pytest.mark.parametrize("grouping", [True, False], ids=["levels", "steps"])
def test_fused_job_is_bitwise_alone(name, prec, grouping):
    (rows, cols, depth, n_sliced, n_open), holds = CASES[name]
    arena = torch.empty(2 << 30, dtype=torch.uint8, device="cuda")
    ctx = tnc.Context(0, arena_bytes=arena.numel(), arena_ptr=arena.data_ptr())
    items, handles = [], []
    for seed in range(5):
        net = circuit_network(random_circuit(rows, cols, depth, seed=9100 + seed), open_qubits=tuple(range(n_open)))
        path = greedy_path(net)
        sl = greedy_slice(net, path.pairs, n_sliced=n_sliced) if n_sliced else ()
        tn = tnc.Network(ctx, net.labels, net.extents, net.open, net.c64().leaves)
        p = tnc.Plan(tn, path.pairs, sl, prec)
        if not grouping:
            tnc.tnc_plan_set_grouping(p.handle, 0)
            p.info = tnc.tnc_plan_get_info(p.handle)
        handles.append((tn, p))
        items.append((p, 0, p.info.n_slices))
    if prec == tnc.PREC_C64:
        p = items[0][0]
        assert holds([tnc.tnc_plan_get_batch_step(p.handle, q) for q in range(p.info.n_steps)], p.info)
    print(name, flush=True)
    alone, st_alone = _serve_each(ctx, items, fuse=False)
    mix, st = _serve_each(ctx, items, fuse=True)
    assert st_alone[1] == 0 and st[1] == 1 and st[2] == 5
    for a, m in zip(alone, mix):
        assert np.any(a) and np.array_equal(a.view(np.uint64), m.view(np.uint64))
    for tn, p in handles:
        p.close()
        tn.close()
    ctx.close()
