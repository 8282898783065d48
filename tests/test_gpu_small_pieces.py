"""The small-graph engine where its passes divide the work: more pieces than
threads (a path or a star deleted whole), none (a delete without tree edges,
an insert inside one component: the forest stays as it is), graphs of 1 and 2
vertices and of a whole number of rounds, batches read in place on the device,
alone and beside a large graph.  Bit-exact with the oracle after every call,
and the call's figures the same however the graphs are scheduled."""
from __future__ import annotations

import numpy as np
import pytest

import gen
from test_gpu_multi import MultiPair, _case

pytestmark = pytest.mark.gpu


class DevicePair(MultiPair):
    """MultiPair with every input in device memory."""

    def __init__(self, graphs, **kw):
        import torch
        from paper_2607_20211_amd import drsf

        class Forest(drsf.MultiForest):
            def __init__(self, off, row, col, par, **k):
                dev = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (row, col, par)]
                super().__init__(off, *dev, inputs_on_device=True, **k)

            def apply_multi(self, edges, b_off, op):
                e = torch.from_numpy(np.ascontiguousarray(edges, np.int32)).cuda()
                torch.cuda.synchronize()
                return super().apply_multi(e, b_off, op)

            def parent(self):
                return _host(super().parent())

            def label(self):
                return _host(super().label())

        def _host(a):
            return a.cpu().numpy() if hasattr(a, "cpu") else a

        keep, drsf.MultiForest = drsf.MultiForest, Forest
        try:
            super().__init__(graphs, **kw)
        finally:
            drsf.MultiForest = keep


def _pairs(keys):
    return np.stack([keys >> np.uint64(32), keys & np.uint64(0xffffffff)], 1).astype(np.int32)


def _graphs(big):
    def path(n):
        return np.array([(i << 32) | (i + 1) for i in range(n - 1)], np.uint64)
    gs = [gen.make_graph("path", 1500, path(1500)),
          gen.make_graph("star", 1100, np.array([i for i in range(1, 1100)], np.uint64)),
          gen.make_graph("one", 1, np.zeros(0, np.uint64)),
          gen.make_graph("two", 2, np.array([1], np.uint64)),
          gen.make_graph("dense", 512, gen.gnm(512, 3000, 5)),
          gen.make_graph("empty", 1024, np.zeros(0, np.uint64))]
    if big:
        gs.append(gen.make_graph("big", 9000, gen.gnm(9000, 30000, 6)))
    return gs


@pytest.mark.parametrize("kind", [MultiPair, DevicePair])
@pytest.mark.parametrize("big", [False, True])
@pytest.mark.parametrize("threads", [256, 512, 1024])
def test_pieces_beyond_and_below_the_workgroup(kind, big, threads):
    _case(f"small pieces {kind.__name__} big {big} threads {threads}")
    graphs = _graphs(big)
    G = len(graphs)
    pair = kind(graphs, max_batch=1 << 14, small_graph_vertices=2048, small_threads=threads)
    none = np.zeros((0, 2), np.int32)
    whole = [_pairs(g.keys) for g in graphs]
    dense = pair.state[4]
    tree = np.minimum(dense[2], np.arange(512)).astype(np.uint64) << np.uint64(32) | \
        np.maximum(dense[2], np.arange(512)).astype(np.uint64)
    off_tree = _pairs(np.setdiff1d(dense[1], tree)[:200])
    last = [whole[6][:700]] if big else []
    # everything goes but the dense graph's tree and the large graph's rest
    pair.step([whole[0], whole[1], none, whole[3], off_tree, none] + last, np.ones(G, np.int8), "delete")
    # back, the off-tree edges inside the dense graph's component; a path where nothing was
    ins = [whole[0], whole[1], none, whole[3], off_tree, whole[0][:1023]] + last
    pair.step(ins, np.zeros(G, np.int8), "insert")
    # half of each, both ops in one call
    ops = np.array([1, 0, 0, 1, 1, 1] + [1] * big, np.int8)
    pair.step([whole[0][::2], none, none, whole[3], whole[4][:900], whole[0][:1023:3]] + last, ops, "mixed")
    pair.gpu.close()


@pytest.mark.parametrize("count", [1, 2, 257])
def test_runs_of_many_graphs(count):
    """Every entry finds its graph: one graph, empty runs at both ends and in a
    row, no small-graph engine and with it."""
    _case(f"runs of {count} graphs")
    ns = [40 + 7 * (i % 50) for i in range(count)]
    graphs = [gen.make_graph(f"g{i}", n, gen.gnm(n, 3 * n, i)) for i, n in enumerate(ns)]
    for T in (0, 150):
        pair = MultiPair(graphs, max_batch=1 << 15, small_graph_vertices=T)
        for skip in (1, 3):
            size = [0 if i % skip else 20 for i in range(count)]
            size[0], size[-1] = (0, 0) if count > 2 else (size[0], size[-1])
            cut = [_pairs(st[1])[:k] for st, k in zip(pair.state, size)]
            pair.step(cut, np.ones(count, np.int8), "delete")
            pair.step(cut, np.zeros(count, np.int8), "insert")
        pair.gpu.close()
