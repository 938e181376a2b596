"""The work that users of the path executor have it do, as cases that can be timed and compared.

Kinds of case, each through the public binding (``paper_2606_01852_amd.tnc``):

  permute   one operand permutation (``tnc_permute``)
  gemm      one batched complex GEMM (``tnc_batched_cgemm``)
  pair      one pairwise contraction with permuted stored operands, as a plan
            (operand permutes, then the GEMM), result left on the device
  circuit   amplitudes of a grid circuit as a plan: a set of open qubits, a
            batch of bitstrings, or a range of slices of a sliced network
  grid      a 2D lattice with one site left open, as a plan
  serve     amplitude requests of circuits of one geometry through the server

Results are taken in complex64: the arithmetic is complex64 (FP64 only adds
the slices up).  One context, with one arena and one stream, serves every
plan of the process, as in a program that contracts one network after the
other; the server has a context of its own, because a serving context
refuses direct contractions.
"""
import functools
import math

import numpy as np
import torch

from paper_2606_01852_amd import tnc
from workloads.circuits import circuit_network, circuit_network_batched, random_circuit
from workloads.grids import grid_labels
from workloads.network import Network
from workloads.paths import greedy_path, greedy_slice, path_cost, path_tensors

ARENA = 32 << 30
SERVE_ARENA = 4 << 30
PRECS = {"c64": tnc.PREC_C64, "bf16x3": tnc.PREC_BF16X3}
FORMS = {"4M": tnc.GEMM_4M, "3M": tnc.GEMM_3M}


# ---------------------------------------------------------------- the cases
def listed():
    return [
        # a leaf of a lattice or circuit slice put in GEMM order: the smallest call there is
        {"name": "permute_small", "kind": "permute", "ext": 4, "rank": 9, "order": 3},
        # the operand of a large pairwise step (2^27 complex64, 1 GiB) put in GEMM order
        {"name": "permute_large", "kind": "permute", "ext": 2, "rank": 27, "order": 5},
        # a step of a network with extents that are no powers of two
        {"name": "gemm_ragged", "kind": "gemm", "h": 6, "m": 1000, "n": 500, "k": 777, "prec": "c64", "form": "4M"},
        # the same call in the three-product form, a batch of mid-sized steps
        {"name": "gemm_batch_3M", "kind": "gemm", "h": 16, "m": 1024, "n": 512, "k": 768, "prec": "c64", "form": "3M"},
        # 64 independent contractions of 20 by 18 modes, 10 shared (the benchmark's second leg)
        {"name": "pair_batch", "kind": "pair", "ext": 2, "nm": 10, "nk": 10, "nn": 8, "batch": 64, "prec": "c64", "form": "4M", "order": 1},
        # the benchmark's large pairwise contraction, one mode shorter in each of M, K and N
        {"name": "pair_large", "kind": "pair", "ext": 2, "nm": 15, "nk": 13, "nn": 13, "batch": 1, "prec": "c64", "form": "4M", "order": 2},
        # large steps in split precision, in both complex forms
        {"name": "pair_bf16x3", "kind": "pair", "ext": 2, "nm": 14, "nk": 13, "nn": 13, "batch": 1, "prec": "bf16x3", "form": "4M", "order": 3},
        {"name": "pair_bf16x3_3M", "kind": "pair", "ext": 2, "nm": 14, "nk": 13, "nn": 13, "batch": 1, "prec": "bf16x3", "form": "3M", "order": 4},
        # all 4096 amplitudes of a 12-qubit circuit: latency of a whole small network, replayed as a graph
        {"name": "circuit_amps", "kind": "circuit", "rows": 3, "cols": 4, "depth": 8, "open": 12, "rowsb": 0, "sliced": 0, "count": 1, "prec": "c64", "form": "4M", "graph": True},
        # a closed-but-one-site 8x8 lattice of bond 4: few steps with work, many without
        {"name": "grid8", "kind": "grid", "rows": 8, "cols": 8, "bond": 4, "prec": "c64", "form": "4M", "graph": True},
        # 256 slices of a 40-qubit circuit with 16 sliced labels, as one batch: a rank's share of a large contraction
        {"name": "circuit_slices", "kind": "circuit", "rows": 5, "cols": 8, "depth": 12, "open": 3, "rowsb": 0, "sliced": 16, "count": 256, "prec": "c64", "form": "4M", "graph": False},
        # amplitude requests of 32 circuits of one geometry, queued at once: the server's launch-bound load
        {"name": "serve", "kind": "serve", "rows": 4, "cols": 5, "depth": 10, "requests": 32, "prec": "c64", "form": "4M"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["permute", "gemm", "gemm", "pair", "pair", "circuit", "circuit", "grid", "serve"])
    prec = rng.choice(["c64", "c64", "bf16x3"])
    form = rng.choice(["4M", "4M", "3M"])
    order = rng.randrange(1 << 16)
    if kind == "permute":
        ext = rng.choice([2, 2, 3, 4, 5, 6, 8, 10])
        size = rng.uniform(12, 27)
        return {"kind": kind, "ext": ext, "rank": max(3, int(size / math.log2(ext))), "order": order}
    if kind == "gemm":
        m, n, k = _log(rng, 24, 2500), _log(rng, 24, 2500), _log(rng, 24, 2500)
        h = _log(rng, 1, 256)
        while h > 1 and h * (m * k + n * k + m * n) > 1 << 27:
            h //= 2
        return {"kind": kind, "h": h, "m": m, "n": n, "k": k, "prec": prec, "form": form}
    if kind == "pair":
        ext = rng.choice([2, 2, 2, 3])
        lo, hi = (7, 13) if ext == 2 else (4, 8)
        nm, nk, nn = rng.randint(lo, hi + 1), rng.randint(lo, hi), rng.randint(lo, hi)
        batch = _log(rng, 1, 96)
        while batch > 1 and batch * ext ** (nm + max(nk, nn)) > 1 << 27:
            batch //= 2
        return {"kind": kind, "ext": ext, "nm": nm, "nk": nk, "nn": nn, "batch": batch, "prec": prec, "form": form, "order": order}
    if kind == "grid":
        return {"kind": kind, "rows": rng.randint(4, 8), "cols": rng.randint(4, 8), "bond": rng.choice([2, 3, 4]), "prec": prec,
                "form": form, "graph": rng.random() < 0.7}
    if kind == "serve":
        return {"kind": kind, "rows": rng.randint(3, 4), "cols": rng.randint(4, 5), "depth": rng.randint(6, 10),
                "requests": _log(rng, 8, 64), "prec": "c64", "form": form}
    while True:
        sliced = rng.choice([0, 0, 4, 6, 8])
        open_, rowsb = (0, _log(rng, 12, 96)) if not sliced and rng.random() < 0.4 else (rng.randint(4, 10), 0)
        c = {"kind": kind, "rows": rng.randint(3, 5), "cols": rng.randint(4, 6), "depth": rng.randint(6, 12), "open": open_, "rowsb": rowsb,
             "sliced": sliced, "count": 1, "prec": prec, "form": form, "graph": rng.random() < 0.5}
        net, pairs, sl = _circuit_structure(c["rows"], c["cols"], c["depth"], c["open"], c["rowsb"], c["sliced"])
        big, ops = path_cost(net, pairs, sl)
        c["count"] = rng.choice([2 ** sliced, max(1, 3 * 2 ** sliced // 4)])
        if big <= 1 << 23 and 8 * ops * c["count"] < 2e12 and big * c["count"] <= 1 << 28:
            return c


# ---------------------------------------------------------------- networks
@functools.lru_cache(maxsize=None)
def _circuit_structure(rows, cols, depth, n_open, rowsb, n_sliced):
    """(network with some gates, path, sliced labels): the structure does not depend on the gates."""
    net = _circuit(rows, cols, depth, n_open, rowsb, 0)
    pairs = greedy_path(net).pairs
    return net, pairs, greedy_slice(net, pairs, n_sliced=n_sliced) if n_sliced else ()


def _circuit(rows, cols, depth, n_open, rowsb, seed):
    circ = random_circuit(rows, cols, depth, seed=seed)
    if rowsb:
        bits = np.random.default_rng(seed).integers(0, 2, size=(rowsb, rows * cols))
        return circuit_network_batched(circ, bits)
    return circuit_network(circ, open_qubits=range(n_open))


def _grid(rows, cols, bond, seed):
    """Lattice with entries CN(0, 1) / sqrt(numel) times 2^floor(degree/2) (as the benchmark's), one site with an open mode."""
    labels, n_lab = grid_labels(rows, cols)
    labels = [tuple(lab) for lab in labels]
    labels[0] = labels[0] + (n_lab,)
    extents = np.full(n_lab + 1, bond, dtype=np.int64)
    extents[n_lab] = 16
    rng = np.random.default_rng(seed)
    leaves = []
    for lab in labels:
        shape = tuple(int(extents[l]) for l in lab)
        z = (rng.standard_normal(shape) + 1j * rng.standard_normal(shape)) / math.sqrt(2.0)
        leaves.append(z / math.sqrt(z.size) * 2.0 ** (len(lab) // 2))
    return Network(leaves, labels, extents, (n_lab,))


@functools.lru_cache(maxsize=None)
def _grid_path(rows, cols, bond):
    return greedy_path(_grid(rows, cols, bond, 0)).pairs


def _pair_labels(c):
    """(labels of A, of B, of the result, extents): stored orders are a random permutation, fixed by ``order``."""
    nm, nk, nn = c["nm"], c["nk"], c["nn"]
    rng = np.random.default_rng(c["order"])
    M, K, N = range(nm), range(nm, nm + nk), range(nm + nk, nm + nk + nn)
    a = tuple(int(x) for x in rng.permutation([*M, *K]))
    b = tuple(int(x) for x in rng.permutation([*N, *K]))
    out = (*M, *N)
    ext = [c["ext"]] * (nm + nk + nn)
    if c["batch"] > 1:
        z = len(ext)
        ext.append(c["batch"])
        a, b, out = (z, *a), (z, *b), (z, *out)
    return a, b, out, ext


def _network(c, seed):
    """(network, path, sliced labels) of a circuit or grid case."""
    if c["kind"] == "grid":
        return _grid(c["rows"], c["cols"], c["bond"], seed).c64(), _grid_path(c["rows"], c["cols"], c["bond"]), ()
    shape = (c["rows"], c["cols"], c["depth"], c["open"], c["rowsb"])
    _, pairs, sliced = _circuit_structure(*shape, c["sliced"])
    return _circuit(*shape, seed).c64(), pairs, sliced


def _serve_networks(c, seed):
    shape = (c["rows"], c["cols"], c["depth"], 0, 0)
    pairs = _circuit_structure(*shape, 0)[1]
    return [_circuit(*shape, seed * 1000 + i).c64() for i in range(c["requests"])], pairs


def _cn(shape, seed):
    """CN(0, 1) entries on the GPU."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    x = torch.randn((*shape, 2), generator=g, device="cuda", dtype=torch.float32)
    return torch.view_as_complex(x.mul_(math.sqrt(0.5)))


# ---------------------------------------------------------------- contexts
@functools.lru_cache(maxsize=None)
def _context():
    arena = torch.empty(ARENA, dtype=torch.uint8, device="cuda")
    return tnc.Context(0, arena_bytes=ARENA, arena_ptr=arena.data_ptr()), arena


@functools.lru_cache(maxsize=None)
def _server():
    arena = torch.empty(SERVE_ARENA, dtype=torch.uint8, device="cuda")
    ctx = tnc.Context(0, arena_bytes=SERVE_ARENA, arena_ptr=arena.data_ptr())
    tnc.tnc_serve_start(ctx.handle, 8, 1024)
    return ctx, arena


def prepare(case, seed):
    c, kind = case, case["kind"]
    if kind == "serve":
        ctx = _server()[0]
        nets, pairs = _serve_networks(c, seed)
        held = [tnc.Network(ctx, n.labels, n.extents, n.open, n.leaves) for n in nets]
        plans = [tnc.Plan(n, pairs, (), PRECS[c["prec"]], FORMS[c["form"]]) for n in held]
        return {"case": c, "ctx": ctx, "nets": held, "plans": plans,
                "out": [np.zeros(1, dtype=np.complex128) for _ in plans]}
    ctx = _context()[0]
    if kind == "permute":
        perm = [int(x) for x in np.random.default_rng(c["order"]).permutation(c["rank"])]
        x = _cn((c["ext"],) * c["rank"], seed)
        return {"case": c, "ctx": ctx, "x": x, "out": torch.empty_like(x), "ext": [c["ext"]] * c["rank"], "perm": perm}
    if kind == "gemm":
        h, m, n, k = c["h"], c["m"], c["n"], c["k"]
        return {"case": c, "ctx": ctx, "a": _cn((h, m, k), 2 * seed), "b": _cn((h, n, k), 2 * seed + 1),
                "out": torch.empty((h, m, n), dtype=torch.complex64, device="cuda")}
    if kind == "pair":
        a, b, out, ext = _pair_labels(c)
        shapes = [tuple(ext[l] for l in lab) for lab in (a, b)]
        net = tnc.Network(ctx, [a, b], ext, out, [np.zeros(s, dtype=np.complex64) for s in shapes])
        for t in (0, 1):  # the operands are made where they are used: a previous computation's results
            x = _cn(shapes[t], 2 * seed + t)
            torch.cuda.synchronize()
            tnc.tnc_net_set_tensor_device(net.handle, t, x.data_ptr())
            ctx.sync()
        plan = tnc.Plan(net, [(0, 1)], (), PRECS[c["prec"]], FORMS[c["form"]])
        return {"case": c, "ctx": ctx, "net": net, "plan": plan, "count": 1,
                "out": torch.empty([ext[l] for l in out], dtype=torch.complex64, device="cuda")}
    net64, pairs, sliced = _network(c, seed)
    net = tnc.Network(ctx, net64.labels, net64.extents, net64.open, net64.leaves)
    plan = tnc.Plan(net, pairs, sliced, PRECS[c["prec"]], FORMS[c["form"]])
    tnc.tnc_plan_set_graph(plan.handle, c["graph"])
    shape = [int(net64.extents[l]) for l in net64.open]
    return {"case": c, "ctx": ctx, "net": net, "plan": plan, "count": c.get("count", 1),
            "out": torch.empty(shape, dtype=torch.complex64, device="cuda")}


def run(state):
    s, kind = state, state["case"]["kind"]
    if kind == "permute":
        tnc.tnc_permute(s["ctx"].handle, s["x"].data_ptr(), s["out"].data_ptr(), s["ext"], s["perm"])
        return s["out"]
    if kind == "gemm":
        c = s["case"]
        h, m, n, k = c["h"], c["m"], c["n"], c["k"]
        tnc.tnc_batched_cgemm(s["ctx"].handle, h, m, n, k, s["a"].data_ptr(), m * k, s["b"].data_ptr(), n * k,
                              s["out"].data_ptr(), PRECS[c["prec"]], FORMS[c["form"]])
        return s["out"]
    if kind == "serve":
        ctx = s["ctx"].handle
        ids = [tnc.tnc_submit(ctx, p.handle, 0, 1, o) for p, o in zip(s["plans"], s["out"])]
        for i in ids:
            tnc.tnc_wait(ctx, i)
        return np.concatenate(s["out"]).astype(np.complex64)
    tnc.tnc_contract_async(s["plan"].handle, 0, s["count"], s["out"].data_ptr(), tnc.OUT_C64)
    return s["out"]


# ---------------------------------------------------------------- what a pass cannot do without
def _slice_flops(net, pairs, sliced, count):
    """8 operations per complex multiply-add of every step, once for every value that the sliced labels below it take
    in slices [0, count)."""
    _, ops = path_tensors(net, pairs, sliced)
    under = [frozenset(l for l in lab if l in set(sliced)) for lab in net.labels]
    total = 0
    for (a, b), o in zip(pairs, ops):
        under.append(under[a] | under[b])
        seen = 1
        rest = count
        for l in reversed(sliced):  # the last label turns fastest
            e = int(net.extents[l])
            if l in under[-1]:
                seen *= min(e, rest)
            rest = -(-rest // e)
        total += 8 * o * seen
    return total


def work(case):
    c, kind = case, case["kind"]
    if kind == "permute":
        return {"bytes": 16 * c["ext"] ** c["rank"], "flops": 0}
    if kind == "gemm":
        h, m, n, k = c["h"], c["m"], c["n"], c["k"]
        return {"bytes": 8 * h * (m * k + n * k + m * n), "flops": 8 * h * m * n * k}
    if kind == "pair":
        m, n, k = (c["ext"] ** c[x] for x in ("nm", "nn", "nk"))
        return {"bytes": 8 * c["batch"] * (m * k + n * k + m * n), "flops": 8 * c["batch"] * m * n * k}
    if kind == "serve":
        net, pairs, _ = _circuit_structure(c["rows"], c["cols"], c["depth"], 0, 0, 0)
        leaves = sum(x.size for x in net.leaves)
        return {"bytes": c["requests"] * (8 * leaves + 16), "flops": c["requests"] * 8 * path_cost(net, pairs)[1]}
    net, pairs, sliced = _network(c, 0)
    n_out = int(np.prod([net.extents[l] for l in net.open]))
    return {"bytes": 8 * (sum(x.size for x in net.leaves) + n_out),
            "flops": _slice_flops(net, pairs, sliced, c.get("count", 1))}


# ---------------------------------------------------------------- the same in 64 bits, with torch alone
def _transposed(x, order):
    """x.permute(order), contiguous; by an index per element above the dozen modes that torch copies by strides."""
    if x.dim() <= 12:
        return x.permute(order).contiguous()
    shape = [x.shape[j] for j in order]
    at = torch.zeros(1, dtype=torch.int64, device=x.device)
    for j in order:
        step = torch.arange(x.shape[j], device=x.device) * x.stride(j)
        at = (at[:, None] + step[None, :]).reshape(-1)
    return x.reshape(-1)[at].reshape(shape)


def _product(xa, la, xb, lb, keep, ext):
    """Contraction of two tensors over the shared labels that are not kept; kept shared labels are batch labels."""
    shared = [l for l in la if l in lb]
    batch = [l for l in shared if l in keep]
    summed = [l for l in shared if l not in keep]
    ra = [l for l in la if l not in shared]
    rb = [l for l in lb if l not in shared]
    size = lambda ls: int(np.prod([ext[l] for l in ls], dtype=np.int64))  # noqa: E731
    pa = _transposed(xa, [la.index(l) for l in batch + ra + summed]).reshape(size(batch), size(ra), size(summed))
    pb = _transposed(xb, [lb.index(l) for l in batch + summed + rb]).reshape(size(batch), size(summed), size(rb))
    out = torch.matmul(pa, pb)
    labels = batch + ra + rb
    return out.reshape([ext[l] for l in labels]), labels


def _contract64(net, pairs, sliced=(), count=1):
    """Sum over slices [0, count), up to 64 at a time behind one more batch label."""
    ext = {l: int(e) for l, e in enumerate(net.extents)}
    z = len(ext)
    batch = {l for l in net.open if sum(l in lab for lab in net.labels) > 1}
    leaves = [torch.from_numpy(np.asarray(x, dtype=np.complex64)).cuda().to(torch.complex128) for x in net.leaves]
    total = 0
    for s0 in range(0, count, 64):
        s = torch.arange(s0, min(count, s0 + 64), device="cuda")
        ext[z] = len(s)
        digit = {}
        for l in reversed(sliced):
            digit[l] = s % ext[l]
            s = s // ext[l]
        tens = []
        for x, lab in zip(leaves, net.labels):
            fixed = [l for l in lab if l in digit]
            left = [l for l in lab if l not in digit]
            if fixed:
                x = _transposed(x, [lab.index(l) for l in fixed + left])[tuple(digit[l] for l in fixed)]
                left = [z] + left
            tens.append((x, left))
        keep = batch | {z}
        for a, b in pairs:
            (xa, la), (xb, lb) = tens[a], tens[b]
            tens[a] = tens[b] = None
            tens.append(_product(xa, la, xb, lb, keep, ext))
        x, lab = tens[-1]
        if z in lab:
            x = x.sum(lab.index(z))
            lab = [l for l in lab if l != z]
        else:
            x = x * ext[z]
        total = total + _transposed(x, [lab.index(l) for l in net.open])
    return total


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind == "permute":
        perm = [int(x) for x in np.random.default_rng(c["order"]).permutation(c["rank"])]
        return _transposed(_cn((c["ext"],) * c["rank"], seed), perm).to(torch.complex128)
    if kind == "gemm":
        a = _cn((c["h"], c["m"], c["k"]), 2 * seed).to(torch.complex128)
        b = _cn((c["h"], c["n"], c["k"]), 2 * seed + 1).to(torch.complex128)
        return torch.matmul(a, b.transpose(1, 2).contiguous())
    if kind == "pair":
        a, b, out, ext = _pair_labels(c)
        xa, xb = (_cn([ext[l] for l in lab], 2 * seed + t).to(torch.complex128) for t, lab in enumerate((a, b)))
        x, lab = _product(xa, list(a), xb, list(b), set(out), dict(enumerate(ext)))
        return x if lab == list(out) else _transposed(x, [lab.index(l) for l in out])
    if kind == "serve":
        nets, pairs = _serve_networks(c, seed)
        return torch.stack([_contract64(n, pairs).reshape(()) for n in nets])
    net, pairs, sliced = _network(c, seed)
    return _contract64(net, pairs, sliced, c.get("count", 1))
