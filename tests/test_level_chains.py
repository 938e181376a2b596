"""Levels with next to no work share a launch (a chain of levels, one
workgroup): fewer launches than levels on the host, and on the GPU bitwise
the step-by-step result, alone, replayed as a graph, and for several runs in
one fused job's launch."""
import numpy as np
import pytest

from paper_2606_01852_amd import tnc
from workloads import configs
from workloads.circuits import circuit_network, circuit_network_batched, random_circuit
from workloads.paths import greedy_path, greedy_slice


def networks():
    circ = configs.circuit12_circuit()
    bits = np.random.default_rng(3).integers(0, 2, size=(24, circ.n_qubits))
    wide = circuit_network(random_circuit(4, 5, 8, seed=11))
    return {"open": (circuit_network(circ, open_qubits=range(12)), 0),
            "batched": (circuit_network_batched(circ, bits), 0),   # batch dims inside a chain
            "sliced": (wide, 3)}                                   # chunks, and leaves read in place


def plan_of(ctx, net, n_sliced, prec=tnc.PREC_C64):
    path = greedy_path(net)
    sliced = greedy_slice(net, path.pairs, n_sliced=n_sliced) if n_sliced else ()
    tn = tnc.Network(ctx, net.labels, net.extents, net.open, net.c64().leaves)
    return tn, tnc.Plan(tn, path.pairs, sliced, prec)


@pytest.mark.parametrize("name", ["open", "batched", "sliced"])
def test_a_chain_saves_launches(name):
    net, n_sliced = networks()[name]
    ctx = tnc.Context(-1, arena_bytes=1 << 30)
    _, plan = plan_of(ctx, net, n_sliced)
    level = [0] * net.n_leaves
    for a, b in greedy_path(net).pairs:
        level.append(1 + max(level[a], level[b]))
    chunks = plan.info.n_slices // plan.info.max_chunk
    assert plan.info.n_launches < chunks * max(level), (plan.info.n_launches, max(level))


@pytest.mark.gpu
@pytest.mark.parametrize("prec", [tnc.PREC_C64, tnc.PREC_BF16X3], ids=["c64", "bf16x3"])
@pytest.mark.parametrize("name", ["open", "batched", "sliced"])
def test_chained_levels_are_bitwise_the_steps(name, prec):
    net, n_sliced = networks()[name]
    ctx = tnc.Context(0, arena_bytes=1 << 30)
    tn, plan = plan_of(ctx, net, n_sliced, prec)
    print(name, prec, flush=True)
    got = plan.contract()
    tnc.tnc_plan_set_graph(plan.handle, True)
    for _ in range(3):
        assert np.array_equal(plan.contract().view(np.uint64), got.view(np.uint64))
    tnc.tnc_plan_set_graph(plan.handle, False)
    tnc.tnc_plan_set_grouping(plan.handle, False)
    assert np.array_equal(plan.contract().view(np.uint64), got.view(np.uint64))
    # several runs of the structure in one job: one workgroup per run
    tnc.tnc_serve_start(ctx.handle, 1, 64)
    tnc.tnc_serve_set_fusion(ctx.handle, 8, tnc.FUSE_ALL)
    many = [plan_of(ctx, net, n_sliced, prec) for _ in range(6)]
    outs = [np.zeros(plan.info.n_result, dtype=np.complex128) for _ in many]
    ids = [tnc.tnc_submit(ctx.handle, p.handle, 0, p.info.n_slices, o) for (_, p), o in zip(many, outs)]
    for i in ids:
        tnc.tnc_wait(ctx.handle, i)
    for o in outs:
        assert np.array_equal(o.view(np.uint64), got.view(np.uint64))
    tnc.tnc_serve_stop(ctx.handle)
    for t, p in many + [(tn, plan)]:
        p.close()
        t.close()
    ctx.close()
