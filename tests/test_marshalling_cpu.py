"""Arguments and results of the Python calls: arrays of any kind, whole and partial tables."""
from types import SimpleNamespace

import numpy as np
import pytest
import torch

from paper_2301_04285_amd import taps as T
from paper_2301_04285_amd import workloads as W


def _offsets(kind, offs):
    if kind == "read-only":
        offs = offs.copy()
        offs.flags.writeable = False
    elif kind == "strided":
        offs = np.repeat(offs, 2)[::2]
    elif kind == "list":
        offs = [int(x) for x in offs]
    elif kind == "int64":
        offs = offs.astype(np.int64)
    return offs


@pytest.mark.parametrize("kind", ["writable", "read-only", "strided", "list", "int64"])
def test_offsets_of_any_kind(kind):
    g = W.mlp2()
    c = W.Cluster(2, 2, 300, 30)
    offs, eoffs = T.taps_build_tables(g, c, size_only=True)
    got, none = T.taps_edge_costs(g, c, None, _offsets(kind, offs), size_only=True,
                                  stream=SimpleNamespace(cuda_stream=0))
    assert none is None and np.array_equal(got, eoffs)


def test_no_operators_and_no_edges():
    g = T.pack_graph(W.Graph([], []))
    offs, eoffs = T.taps_build_tables(g, W.Cluster(2, 2, 300, 30), size_only=True)
    assert offs.tolist() == [0] and eoffs.tolist() == [0]


@pytest.mark.parametrize("n", [0, 1, 6, 7])
def test_results_are_the_first_entries(n):
    tab = T.alloc_table(7, device="cpu")
    got = T._first_of(tab, n)
    assert list(got) == list(tab)
    for k, v in got.items():
        assert v.shape == (n,) and v.dtype == tab[k].dtype
        assert n == 0 or v.data_ptr() == tab[k].data_ptr()
    s = torch.zeros((7, T.STRATEGY_BYTES), dtype=torch.uint8)
    assert T._first(s, n).shape == (n, T.STRATEGY_BYTES)
    assert T._capacity({**tab, "t": torch.empty(n)}) == n
