"""Stopping a server ends every worker, also those that slept because the
requests left were not admissible (host-only context: requests are admitted
and finish at once)."""
import subprocess
import sys

SCRIPT = """
import numpy as np
from paper_2606_01852_amd import tnc
from workloads.circuits import circuit_network, random_circuit
from workloads.paths import greedy_path

net = circuit_network(random_circuit(2, 3, 4, seed=1))
path = greedy_path(net)
ctx = tnc.Context(-1, arena_bytes=1 << 30)
tn = tnc.Network(ctx, net.labels, net.extents, net.open, net.c64().leaves)
plan = tnc.Plan(tn, path.pairs)
out = np.zeros(1, dtype=np.complex128)
for rep in range(60):
    tnc.tnc_serve_start(ctx.handle, 8, 1024)
    tnc.tnc_serve_set_heavy(ctx.handle, 1.0, 1)      # every request is heavy, one at a time
    for i in range(40):
        tnc.tnc_submit(ctx.handle, plan.handle, 0, 1, out)
    tnc.tnc_serve_stop(ctx.handle)
print("stopped")
"""


def test_stop_wakes_workers_that_wait_for_a_slot():
    r = subprocess.run([sys.executable, "-c", SCRIPT], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "stopped" in r.stdout, r.stderr[-2000:]
