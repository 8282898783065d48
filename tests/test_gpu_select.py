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


@pytest.mark.parametrize("rows,cols,cuts", [(2, 40001, 32767), (2, 40001, 32768), (1, 65537, 65536)])
def test_chains_shortened_by_their_own_pieces(rows, cols, cuts):
    """Batches around the one from which a pass after the first hooks shortens
    their chains; in a path every hook fails to find an edge."""
    drsf = _lib()
    _case(f"grid {rows} x {cols}, {cuts} tree edges cut")
    g = gen.make_graph("grid", rows * cols, gen.grid(rows, cols, 0, gen.seed(85, rows, gen.P_GRAPH)))
    dl = gen.delete_batches(g.n, g.keys, g.parent, 1, cuts, cuts, gen.seed(85, rows, gen.P_DELETE))[0]
    _run(g, [(dl, drsf.DRSF_DELETE), (dl, drsf.DRSF_INSERT), (dl[::2], drsf.DRSF_DELETE)])


@pytest.mark.parametrize("b", [131071, 131072, 140001])
def test_batches_around_the_wide_workgroups(b):
    """Few edges per vertex, so that most entries cut or join trees."""
    drsf = _lib()
    _case(f"G(300000, 400000), batches of {b}")
    g = gen.make_graph("gnm", 300000, gen.gnm(300000, 400000, gen.seed(86, 1, gen.P_GRAPH)))
    cut = np.random.default_rng(b).choice(g.keys, b, replace=False)
    pairs = np.stack([cut >> np.uint64(32), cut & np.uint64(0xffffffff)], 1).astype(np.int32)
    _run(g, [(pairs, drsf.DRSF_DELETE), (pairs, drsf.DRSF_INSERT), (pairs[::-1], drsf.DRSF_DELETE)])


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


@pytest.mark.parametrize("k", [300, 16384])
@pytest.mark.parametrize("launch_mode", [2, 1])
def test_shallow_super_trees_first_then_deep_ones(k, launch_mode):
    """A star's rays, for which the search suffices (a later update then does
    without it), then the ruler chain above, its walks short or past their
    bound, and both again."""
    drsf = _lib()
    _case(f"rays, then a ruler chain of {k} pieces, launch mode {launch_mode}")
    weight = [((j + 1) & -(j + 1)).bit_length() for j in range(k)]
    order = sorted(range(k), key=lambda j: (weight[j], j))
    u = np.empty(k + 1, np.int64)
    u[np.array(order)] = np.arange(k)
    u[k] = 2 * k + 1
    v = np.arange(k, 2 * k + 1, dtype=np.int64)
    rays, c = 5000, 2 * k + 2
    g = gen.make_graph("rays and ruler", 2 * k + 3 + rays, np.sort(gen.keys_of_edges(np.stack([u, v], 1))))
    star = np.stack([np.full(rays, c), np.arange(c + 1, c + 1 + rays)], 1).astype(np.int32)
    chain = np.stack([u[:k], v[1:k + 1]], axis=1).astype(np.int32)
    both = np.concatenate([star, chain])
    _run(g, [(star, drsf.DRSF_INSERT), (star, drsf.DRSF_DELETE), (star, drsf.DRSF_INSERT), (chain, drsf.DRSF_INSERT),
             (both, drsf.DRSF_DELETE), (both, drsf.DRSF_INSERT), (both[::2], drsf.DRSF_DELETE)],
         launch_mode=launch_mode)


@pytest.mark.parametrize("queued", [False, True])
@pytest.mark.parametrize("launch_mode", [2, 1])
def test_the_tour_is_queued_for_a_while(launch_mode, queued):
    """The long ruler chain above, until the tour is queued; after sixteen
    updates of the kind super-trees grow oriented again, so that the next long
    walk is the host's once more, and shallow ones need neither."""
    drsf = _lib()
    k = 16384
    _case(f"ruler chain of {k} pieces and rays, launch mode {launch_mode}, queued {queued}")
    weight = [((j + 1) & -(j + 1)).bit_length() for j in range(k)]
    order = sorted(range(k), key=lambda j: (weight[j], j))
    u = np.empty(k + 1, np.int64)
    u[np.array(order)] = np.arange(k)
    u[k] = 2 * k + 1
    v = np.arange(k, 2 * k + 1, dtype=np.int64)
    c = 2 * k + 2
    g = gen.make_graph("tour for a while", 2 * k + 43, np.sort(gen.keys_of_edges(np.stack([u, v], 1))))
    star = np.stack([np.full(40, c), np.arange(c + 1, c + 41)], 1).astype(np.int32)
    chain = np.stack([u[:k], v[1:k + 1]], axis=1).astype(np.int32)
    pair = Pair(g, max_batch=k, launch_mode=launch_mode, device=queued)

    def there_and_back(batch, what):
        if not queued:
            st, _ = pair.step(batch, drsf.DRSF_INSERT, what)
            pair.step(batch, drsf.DRSF_DELETE, what)
            return st["host_finished"] & 2
        import torch
        with torch.cuda.stream(pair.stream):
            e = torch.from_numpy(batch).to(pair.dev)
        for op in (drsf.DRSF_INSERT, drsf.DRSF_DELETE):
            pair.gpu.apply_async(e, op)
        st = pair.gpu.wait()
        pair.gpu.wait()
        for op in (oracle.INSERT, oracle.DELETE):
            r = oracle.apply(pair.n, pair.keys, pair.parent, batch, op, label=pair.label)
            pair.keys, pair.parent, pair.label = r.keys, r.parent, r.label
        pair.check_equal(what)
        return st["host_finished"] & 2

    assert [there_and_back(chain, f"chain {i}") for i in range(3)] == [2, 2, 0]
    assert [there_and_back(star, f"rays {i}") for i in range(16)] == [0] * 16
    assert [there_and_back(chain, f"chain again {i}") for i in range(3)] == [2, 0, 0]
    assert [there_and_back(star, f"rays again {i}") for i in range(29)] == [0] * 29
    assert [there_and_back(chain, f"chain at last {i}") for i in range(3)] == [0, 2, 0]
    pair.gpu.close()


@pytest.mark.parametrize("device", [True, False])
@pytest.mark.parametrize("b", [1, 2, 511, 512, 513, 4096, 4097, 8193])
def test_batches_around_the_one_workgroup_bounds(b, device):
    drsf = _lib()
    _case(f"batches of {b}, device {device}")
    n = 20011
    g = gen.make_graph("gnm", n, gen.gnm(n, 30000, gen.seed(85, 0, gen.P_GRAPH)))
    ins = gen.insert_batches(n, g.keys, 2, b, gen.seed(85, b, gen.P_INSERT))
    dl = gen.delete_batches(n, g.keys, g.parent, 1, b, (b + 1) // 2, gen.seed(85, b, gen.P_DELETE))[0]
    pair = Pair(g, device=device, max_batch=max(b, 16))
    for i, (e, op) in enumerate([(ins[0], 0), (dl, 1), (ins[1], 0), (dl, 0), (ins[0], 1)]):
        pair.step(e, (drsf.DRSF_INSERT, drsf.DRSF_DELETE)[op], f"batch {i}")
    bad = np.concatenate([ins[0], ins[1][:1]]) if b > 1 else np.array([[3, 3]], np.int32)  # ins[1] is there
    if len(bad) <= max(b, 16):
        with pytest.raises(drsf.DrsfError):
            if device:
                import torch
                with torch.cuda.stream(pair.stream):
                    bad = torch.from_numpy(np.ascontiguousarray(bad)).to(pair.dev)
            pair.gpu.apply(bad, drsf.DRSF_INSERT)
        pair.check_equal("rejected")
    pair.gpu.close()


def test_one_workgroup_rounds_meet_a_long_list():
    """Pieces that pair up in round 0 (their smallest vertices are joined) and
    keep 60,000 edges between them: the list after the first selection is too
    long for one workgroup, the host finishes the update, and later ones make
    more full-grid selections first."""
    drsf = _lib()
    k, size = 800, 10
    n = k * size
    # piece p: its smallest vertex p, then k + 9 p ... k + 9 p + 8, a path
    verts = [[p] + list(range(k + (size - 1) * p, k + (size - 1) * (p + 1))) for p in range(k)]
    parent = np.arange(n, dtype=np.int32)
    edges = []
    for p, vs in enumerate(verts):
        for a, c in zip(vs, vs[1:]):
            edges.append((a, c))
            parent[c] = a
        if p:
            edges.append((verts[p - 1][-1], vs[0]))  # the edges that go
            parent[vs[0]] = verts[p - 1][-1]
    chain = np.array([(verts[p - 1][-1], verts[p][0]) for p in range(1, k)], np.int32)
    edges += [(2 * j, 2 * j + 1) for j in range(k // 2)]
    rng = np.random.default_rng(86)
    r = rng.integers(k, n, (60000, 2))
    keys = np.unique(gen.keys_of_edges(np.concatenate([np.array(edges), r[r[:, 0] != r[:, 1]]])))
    row_ptr, col = gen.keys_to_csr(n, keys)
    _case(f"long list: {k} pieces, {len(keys)} edges")
    pair = Pair(gen.Graph("pairs", n, keys, row_ptr, col, parent), max_batch=1024)
    done = []
    for i in range(6):
        st, _ = pair.step(chain, drsf.DRSF_DELETE, f"delete {i}")
        done.append(st["host_finished"] & 1)
        # back to the chain: a fresh context would start there too
        pair.step(chain, drsf.DRSF_INSERT, f"insert {i}")
        if i == 0:
            assert done[0] == 1, st
            chain = np.stack([np.arange(n), pair.parent], 1)[pair.parent != np.arange(n)][: len(chain)].astype(np.int32)
    assert done[-1] == 0, done
    pair.gpu.close()
