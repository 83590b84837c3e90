"""The edge kernels' windows at the sizes where they can go wrong: tables of one
entry (64 edges in one tile), rows of 2, 52, 63 and 93 entries (rows and edges
that start inside a tile, more rows than a tile has lanes' worth of), single
tiles and the longest windows; the single table, the sweep and the link
classes, entry by entry against the oracle."""
import random

import pytest

from paper_2301_04285_amd import workloads as W
from test_gpu_parity import (T, _topology_check, backward_check, full_check, say,  # noqa: F401
                             sweep_check)

pytestmark = pytest.mark.gpu


def _chain(n_ops, axes, seed):
    """Element-wise operators over `axes` axes of 256 or more, in a chain with a
    few second edges; matmuls now and then, so that rows and columns differ."""
    r = random.Random(seed)
    g = W.Graph()
    names, lens = tuple("abcd"[:axes]), (256, 512, 1024, 256)[:axes]
    prev = None
    for k in range(n_ops):
        if axes == 2 and prev is not None and r.random() < 0.3:
            op = g.add(W.matmul(f"mm{k}", lens[0], lens[1], lens[1], 2))
        else:
            op = g.add(W.elementwise(f"e{k}", "e", names, lens, 1, r.choice((1, 2, 3))))
        if prev is not None:
            g.connect(prev, op, 0)
        prev = op
    return g


@pytest.mark.parametrize("devices,axes,ops", [
    (1, 2, 150),    # one strategy each: tables of one entry
    (2, 2, 40),     # rows of 2 and 3 entries
    (8, 4, 6),      # 52
    (32, 3, 6),     # 63
    (64, 3, 5),     # 93
    (256, 3, 4),    # 171
])
@pytest.mark.parametrize("long_windows", [False, True])
def test_windows_at_their_edges(T, devices, axes, ops, long_windows):  # noqa: F811
    g = _chain(ops, axes, devices + axes)
    per_node = max(1, devices // 4)
    cl = W.Cluster(devices // per_node, per_node, 600 * W.GB, 100 * W.GB)
    name = f"chain of {ops} x {axes} axes on {devices}, long windows {long_windows}"
    say(f"[gpu] {name}")
    prev = T.taps_set_long_segments_min(0 if long_windows else 1 << 40)
    try:
        full_check(T, g, cl, name)
        sweep_check(T, g, [cl, W.Cluster(cl.nodes, per_node, 600 * W.GB, 25 * W.GB)], name)
        domains = sorted({per_node, max(1, devices // 2), devices})
        _topology_check(T, g, cl, W.Topology(tuple(domains),
                                             (600 * W.GB, 100 * W.GB, 25 * W.GB)[:len(domains)]),
                        name)
    finally:
        T.taps_set_long_segments_min(prev)


@pytest.mark.parametrize("pattern", [
    "n" * 9, "n" * 10,                 # 8 tables of one entry in a window, and 9: the first crowded one
    "n" * 65, "n" * 66, "n" * 131,     # a whole tile of them, one more, a whole tile after those
    "w" + "n" * 70 + "www" + "n" * 20 + "w" + "n" * 150 + "ww",   # crowded windows between others
    "wn" * 60,                         # tables of 21 entries: three to a tile, 48 to a long window
])
@pytest.mark.parametrize("long_windows", [False, True])
def test_windows_of_many_tables(T, pattern, long_windows):  # noqa: F811
    """Operators of one strategy (n) and of 21 (w) in a chain."""
    g, prev = W.Graph(), None
    for k, kind in enumerate(pattern):
        op = g.add(W.Op(f"{kind}{k}", "e", ("a", "b", "c"), (256, 256, 256),
                        (True,) + (kind == "w",) * 2, 2, ins=((0, 1, 2),), ws=(), out=(0, 1, 2)))
        if prev is not None:
            g.connect(prev, op, 0)
        prev = op
    cl = W.Cluster(4, 2, 600 * W.GB, 100 * W.GB)
    name = f"chain {pattern}, long windows {long_windows}"
    say(f"[gpu] {name}")
    before = T.taps_set_long_segments_min(0 if long_windows else 1 << 40)
    try:
        full_check(T, g, cl, name)
        backward_check(T, g, cl, name)
        wide = W.Cluster(4, 2, 600 * W.GB + 1, 100 * W.GB + 3)
        for points in ([cl, W.Cluster(4, 2, 600 * W.GB, 25 * W.GB)], [wide, cl]):
            sweep_check(T, g, points, name)
        full_check(T, g, wide, name + ", 128-bit keys")
        for domains in ((8,), (2, 8), (2, 4, 8), (1, 2, 4, 8)):
            _topology_check(T, g, cl, W.Topology(domains, (600 * W.GB, 100 * W.GB, 50 * W.GB,
                                                           25 * W.GB)[:len(domains)]), name)
    finally:
        T.taps_set_long_segments_min(before)


@pytest.mark.parametrize("devices,axes,ops", [
    (1, 2, 40),     # tables of one entry
    (2, 3, 12),     # 9
    (8, 4, 7),      # 2704: a chunk and a part of one
    (32, 3, 9),     # 3969
    (64, 3, 15),    # 8649, into more tables than one task writes
])
@pytest.mark.parametrize("shift", [0, 1])
def test_shared_tables_are_copied_whole(T, devices, axes, ops, shift):  # noqa: F811
    """Copies start and end on the lines of each destination: every entry, and none behind
    the last, into arrays that start on a line or `shift` entries after one."""
    import torch
    r = W.Graph()
    prev = None
    for k in range(ops):   # one kind of operator: all tables but one are copies
        op = r.add(W.elementwise(f"e{k}", "e", tuple("abcd"[:axes]), (256,) * axes, 1, 2))
        if prev is not None:
            r.connect(prev, op, 0)
        prev = op
    cl = W.Cluster(1, devices, 600 * W.GB, 100 * W.GB)
    say(f"[gpu] {ops} shared tables on {devices}, {axes} axes, shift {shift}")
    want = T.taps_build_tables(r, cl)
    n = int(want.edge_offsets[-1])
    wide = {k: v.view(torch.int32 if k == "meta" else torch.int64)
            for k, v in T.alloc_table(n + shift + 40).items()}
    for v in wide.values():
        v.fill_(-7)
    edge = {k: v[shift:shift + n].view(want.edge[k].dtype) for k, v in wide.items()}
    out = T.Tables(want.op_offsets, torch.empty_like(want.strategies),
                   T.alloc_table(len(want.strategies)), want.edge_offsets, edge)
    got = T.taps_build_tables(r, cl, out=out, shared=True)
    for k, v in wide.items():
        assert torch.equal(got.edge[k].view(v.dtype), want.edge[k].view(v.dtype)), k
        assert bool((v[:shift] == -7).all()) and bool((v[shift + n:] == -7).all()), k


@pytest.mark.parametrize("devices", [4, 16, 256])
def test_strategies_that_leave_levels_unused(T, devices):  # noqa: F811
    """Degrees that multiply to less than the devices: the tensors are replicated along the
    levels left, as when an axis that no edge tensor has holds the outermost of them.  Every
    entry whose runs end where the other side has a boundary (the rest has no reference)."""
    import numpy as np
    import torch
    g = W.Graph()
    a, b = g.add(W.matmul("a", 256, 256, 256, 2)), g.add(W.matmul("b", 256, 256, 256, 2))
    g.connect(a, b, 0)
    n, per_node = devices.bit_length() - 1, max(2, devices // 8)
    cl = W.Cluster(devices // per_node, per_node, 600 * W.GB, 100 * W.GB)
    say(f"[gpu] unused levels on {devices}")
    offs, full = T.taps_enumerate_strategies(g, cl)
    deg, pos = T.strategies_to_numpy(full)
    ends, cuts = [], []
    for s in range(len(full)):
        free = 1 if s < offs[1] else 2   # a's inner axis, b's output columns
        order = sorted((int(pos[s, x]), int(deg[s, x]), x) for x in range(3) if deg[s, x])
        starts = [sum(w for _, w, _ in order[:k]) for k in range(1, len(order))]
        if order and order[-1][2] == free:   # outermost: left out of the partial strategy
            deg[s, free], pos[s, free] = 0, -1
            starts = starts[:-1]
        ends.append(sum(int(deg[s, x]) for x in range(3)))
        cuts.append(set(starts) | {0, n})
    partial = torch.from_numpy(np.concatenate([deg, pos.view(np.uint8)], 1)).to(full.device)
    na = int(offs[1])
    clean = np.array([[ends[i] in cuts[j] and ends[j] in cuts[i]
                       for j in range(na, len(full))] for i in range(na)])
    left = np.array([[min(ends[i], ends[j]) < n for j in range(na, len(full))] for i in range(na)])
    assert int((clean & left).sum()) > 2
    topo = W.Topology((per_node, devices // 2, devices), (600 * W.GB, 100 * W.GB, 25 * W.GB))
    points = [cl, W.Cluster(cl.nodes, per_node, 600 * W.GB, 25 * W.GB)]
    for what, call, keep in (
            ("edges", lambda s: T.taps_edge_costs(g, cl, s, offs)[1], clean),
            ("backward", lambda s: T.taps_edge_costs(g, cl, s, offs, backward=True)[1], clean.T),
            ("sweep", lambda s: T.taps_edge_costs_sweep(g, points, s, offs)[1][1], clean),
            ("classes", lambda s: T.taps_edge_costs_topology(g, topo, s, offs)[1], clean)):
        want, got = call(full), call(partial)
        mask = torch.from_numpy(keep.ravel().copy()).to(full.device)
        for k, v in want.items():
            signed = torch.int32 if k == "meta" else torch.int64
            assert torch.equal(got[k].view(signed)[mask], v.view(signed)[mask]), (what, k)


@pytest.mark.parametrize("shift", [1, 6])
def test_strategies_at_any_address(T, shift):  # noqa: F811
    """A strategy is 16 bytes and its array may start on any of them."""
    import torch
    g, cl = W.mlp2(), W.Cluster(2, 2, 600 * W.GB, 100 * W.GB)
    say(f"[gpu] strategies {shift} bytes after an aligned address")
    want = T.taps_build_tables(g, cl)
    n = len(want.strategies)
    wide = torch.full((16 * n + 16,), 0xEE, dtype=torch.uint8, device="cuda")
    out = T.Tables(want.op_offsets, wide[shift:shift + 16 * n].view(n, 16),
                   T.alloc_table(n), want.edge_offsets, T.alloc_table(int(want.edge_offsets[-1])))
    got = T.taps_build_tables(g, cl, out=out)
    assert torch.equal(got.strategies, want.strategies)
    assert bool((wide[:shift] == 0xEE).all()) and bool((wide[shift + 16 * n:] == 0xEE).all())
    _, again = T.taps_edge_costs(g, cl, got.strategies, want.op_offsets)
    node = T.taps_node_costs(g, cl, got.strategies, want.op_offsets)
    for k in want.edge:
        signed = torch.int32 if k == "meta" else torch.int64
        for a, b in ((got.edge[k], want.edge[k]), (again[k], want.edge[k]), (node[k], want.node[k])):
            assert torch.equal(a.view(signed), b.view(signed)), k
