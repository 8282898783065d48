"""Hooking and orphan bookkeeping where their tiles, tables and words end:
many pieces per workgroup (the LDS table of minima fills and is written out
early), long chains of hooks (shortened while they are followed), one piece
that every edge touches, vertex counts around the orphan bitmap's words and
the vertex blocks.  Bit-exact with the oracle after every batch."""
from __future__ import annotations

import numpy as np
import pytest

import gen
import oracle
from test_gpu_parity import Pair, _case, _lib

pytestmark = pytest.mark.gpu


def _run(g, batches, **kw):
    pair = Pair(g, max_batch=max(len(b) for b, _ in batches), **kw)
    for i, (b, op) in enumerate(batches):
        pair.step(np.ascontiguousarray(b, np.int32), op, f"{g.name} batch {i}")
    pair.gpu.close()


@pytest.mark.parametrize("n", [2, 63, 64, 65, 255, 256, 257, 4095, 16385])
@pytest.mark.parametrize("sweep_mode", [0, 1])
def test_vertex_counts_around_words_and_blocks(n, sweep_mode):
    drsf = _lib()
    _case(f"n = {n}, sweep mode {sweep_mode}")
    # a ring with chords: every cut leaves a run of consecutive ids behind
    ring = [(i, (i + 1) % n) for i in range(n if n > 2 else 1)]
    chords = [(i, (i * 7 + 3) % n) for i in range(0, n, 5)] if n > 9 else []
    keys = np.unique(gen.keys_of_edges(np.array([e for e in ring + chords if e[0] != e[1]], np.int32)))
    g = gen.make_graph(f"ring{n}", n, keys)
    rng = np.random.default_rng(n)
    cut = rng.choice(keys, max(1, len(keys) // 3), replace=False)
    pairs = np.stack([cut >> np.uint64(32), cut & np.uint64(0xffffffff)], 1).astype(np.int32)
    _run(g, [(pairs, drsf.DRSF_DELETE), (pairs, drsf.DRSF_INSERT), (pairs[::2], drsf.DRSF_DELETE)],
         sweep_mode=sweep_mode)


@pytest.mark.parametrize("sweep_mode", [0, 1])
@pytest.mark.parametrize("rows,cols,cuts", [(200, 211, 6000), (5, 9001, 9000), (301, 300, 45000)])
def test_many_pieces_and_long_hook_chains(rows, cols, cuts, sweep_mode):
    drsf = _lib()
    _case(f"grid {rows} x {cols}, {cuts} tree edges cut, sweep mode {sweep_mode}")
    g = gen.make_graph("grid", rows * cols, gen.grid(rows, cols, 0, gen.seed(84, rows, gen.P_GRAPH)))
    dl = gen.delete_batches(g.n, g.keys, g.parent, 1, cuts, cuts, gen.seed(84, rows, gen.P_DELETE))[0]
    _run(g, [(dl, drsf.DRSF_DELETE), (dl, drsf.DRSF_INSERT)], sweep_mode=sweep_mode)


@pytest.mark.parametrize("leaves", [700, 5000])
def test_one_piece_that_every_edge_touches(leaves):
    """Inserts and deletes of a star's rays: all edges meet the centre's piece."""
    drsf = _lib()
    _case(f"star of {leaves} rays")
    n = leaves + 1
    rays = np.stack([np.full(leaves, n - 1), np.arange(leaves)], 1).astype(np.int32)
    g = gen.make_graph("star", n, np.zeros(0, np.uint64))
    _run(g, [(rays, drsf.DRSF_INSERT), (rays[::2], drsf.DRSF_DELETE), (rays[::2], drsf.DRSF_INSERT),
             (rays, drsf.DRSF_DELETE)])


@pytest.mark.parametrize("k,bits", [(300, (2, 0, 0)), (16384, (2, 2, 0))])
@pytest.mark.parametrize("launch_mode", [2, 1])
def test_super_trees_searched_then_oriented_as_they_grow(k, bits, launch_mode):
    """A chain of k two-vertex pieces joined by edges whose keys follow the
    ruler sequence, inserted three times: a context's first deep super-tree is
    finished by the host (search and tour), the next is oriented while it
    grows, which on the long chain meets a walk past its bound, so the host
    finishes it too and the third queues the tour."""
    drsf = _lib()
    _case(f"ruler chain of {k} pieces, launch mode {launch_mode}")
    weight = [((j + 1) & -(j + 1)).bit_length() for j in range(k)]
    order = sorted(range(k), key=lambda j: (weight[j], j))
    u = np.empty(k + 1, np.int64)
    u[np.array(order)] = np.arange(k)
    u[k] = 2 * k + 1
    v = np.arange(k, 2 * k + 1, dtype=np.int64)
    keys = np.sort(gen.keys_of_edges(np.stack([u, v], 1)))
    g = gen.make_graph("ruler", 2 * k + 2, keys)
    pair = Pair(g, max_batch=k, launch_mode=launch_mode)
    ins = np.stack([u[:k], v[1:k + 1]], axis=1).astype(np.int32)
    for i, want in enumerate(bits):
        st, _ = pair.step(ins, drsf.DRSF_INSERT, f"insert {i}")
        assert st["host_finished"] & 2 == want, (i, st)
        pair.step(ins, drsf.DRSF_DELETE, f"delete {i}")
    pair.gpu.close()
