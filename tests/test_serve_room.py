"""A fused job in an arena with room for its runs and its table only.

On a host-only context the server admits and queues as on a device but runs
nothing, so a few thousand requests queue up behind one slot in no time.
"""
import numpy as np

from paper_2606_01852_amd import tnc


def serve(arena_bytes, n):
    """(fused jobs, requests refused) of n requests of one structure, two to a job."""
    ctx = tnc.Context(-1, arena_bytes=arena_bytes)
    # 2^14 results: 256 KiB each
    net = tnc.Network(ctx, [(0, 2), (1, 2)], np.array([128, 128, 64], dtype=np.int64), (0, 1), None)
    try:
        plan = tnc.Plan(net, [(0, 1)])
    except tnc.TncError:
        return 0, n
    tnc.tnc_serve_start(ctx.handle, 1, 1 << 16)
    tnc.tnc_serve_set_fusion(ctx.handle, 2, tnc.FUSE_ALL)
    out, ids, refused = np.zeros(128 * 128, dtype=np.complex128), [], 0
    for _ in range(n):
        try:
            ids.append(tnc.tnc_submit(ctx.handle, plan.handle, 0, 1, out))
        except tnc.TncError:
            refused += 1
    for i in ids:
        try:
            tnc.tnc_wait(ctx.handle, i)
        except tnc.TncError:
            pass  # nothing runs here
    fused = tnc.tnc_serve_get_stats(ctx.handle)[1]
    tnc.tnc_serve_stop(ctx.handle)
    plan.close()
    net.close()
    ctx.close()
    return fused, refused


def test_no_room_for_packed_results():
    need = 1 << 14
    while serve(need, 1)[1]:
        need += 1 << 14
    assert need >= 1 << 18                                # a run holds its 256 KiB of results at least
    assert serve(2 * need + (1 << 16), 3000) != (0, 0)    # two runs and the table: no 512 KiB more
    assert serve(2 * need + (1 << 20), 3000) != (0, 0)    # the results side by side as well
    assert serve(need + (1 << 16), 300) == (0, 0)         # one run at a time
