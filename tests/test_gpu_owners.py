"""The strategy kernels that find each strategy's operator per wavefront: operators of one
strategy (64 to a wavefront), of a few and of many, up to more operators than one step of
the search covers; node records against the build's and memory against its definition."""
import random

import pytest

from paper_2301_04285_amd import workloads as W
from test_gpu_parity import T, say  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_ops", [1, 2, 63, 64, 65, 129, 4096, 4097])
@pytest.mark.parametrize("devices", [1, 2, 16])
def test_operators_of_any_number(T, n_ops, devices):  # noqa: F811
    import torch
    r = random.Random(n_ops + devices)
    g = W.Graph()
    for k in range(n_ops):
        lens = tuple(16 * r.randrange(1, 99) for _ in range(r.choice((1, 2, 3))))
        if len(lens) == 2 and r.random() < 0.5:
            g.add(W.matmul(f"m{k}", 16 * r.randrange(1, 99), lens[0], lens[1], 2))
        else:
            g.add(W.elementwise(f"e{k}", "e", "abc"[:len(lens)], lens, 1, r.choice((1, 2, 4))))
    cl = W.Cluster(max(1, devices // 4), min(4, devices), 600 * W.GB, 100 * W.GB)
    say(f"[gpu] {n_ops} operators on {devices}")
    want = T.taps_build_tables(g, cl)
    node = T.taps_node_costs(g, cl, want.strategies, want.op_offsets)
    for k, v in node.items():
        signed = torch.int32 if k == "meta" else torch.int64
        assert torch.equal(v.view(signed), want.node[k].view(signed)), k
    topo = W.Topology((cl.devices_per_node, devices), (600 * W.GB, 100 * W.GB))
    classes = T.taps_node_costs_topology(g, topo, want.strategies, want.op_offsets)
    for k in ("vol", "intra", "inter"):
        assert torch.equal(classes[k].view(torch.int64), want.node[k].view(torch.int64)), k
    memory = T.taps_memory_costs(g, want.strategies, want.op_offsets).cpu().tolist()
    deg, pos = T.strategies_to_numpy(want.strategies)
    for k, op in enumerate(g.ops):
        for s in range(int(want.op_offsets[k]), int(want.op_offsets[k + 1])):
            total = 0
            for tensor in [op.out] + list(op.ws):
                size = op.dtype_bytes
                for a in tensor:
                    size *= op.axis_len[a] >> (int(deg[s, a]) if pos[s, a] >= 0 else 0)
                total += size
            assert memory[s] == total, (k, s)
