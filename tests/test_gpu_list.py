"""The inserted-edge list under edges that come and go: deleted base entries
revived in place, list positions and index slots used again, the list kept or
merged at its merge points.  Bit-exact with the oracle after every batch, and
the orphan figures as the merge points define them (each vertex's edges as of
the last one)."""
from __future__ import annotations

import numpy as np
import pytest

import gen
import oracle
from test_gpu_parity import Pair, _case, _lib, _roots

pytestmark = pytest.mark.gpu


def _degrees(n, keys):
    k = np.asarray(keys, np.uint64)
    return (np.bincount((k >> np.uint64(32)).astype(np.int64), minlength=n)
            + np.bincount((k & np.uint64(0xffffffff)).astype(np.int64), minlength=n))


def _pairs(keys):
    k = np.asarray(keys, np.uint64)
    return np.stack([k & np.uint64(0xffffffff), k >> np.uint64(32)], 1).astype(np.int32)


# new: random non-edges a step (they expire one step later); back: edges of
# the graph (they come back one step later).  The list of 1500 keeps at most
# 187 live entries at a merge point, so 60 new edges are kept and 400 merged;
# its index of 4096 slots is cleared of deleted keys after 2048 uses.
@pytest.mark.parametrize("validate", [True, False])
@pytest.mark.parametrize("device", [True, False])
@pytest.mark.parametrize("new,back,steps", [(60, 240, 60), (400, 50, 12), (0, 300, 12), (300, 0, 16)])
def test_edges_that_come_and_go(new, back, steps, device, validate):
    drsf = _lib()
    n, dcap = 3001, 1500
    g = gen.make_graph("flap", n, gen.gnm(n, 5003, gen.seed(81, new, gen.P_GRAPH)))
    _case(f"edges that come and go: {new} new, {back} back, device {device}, validate {validate}")
    pair = Pair(g, device=device, max_batch=512, delta_capacity=dcap, validate_batches=validate)
    fresh = gen.insert_batches(n, g.keys, steps, new, gen.seed(81, new, gen.P_INSERT)) if new else \
        np.zeros((steps, 0, 2), np.int32)
    rng = np.random.default_rng(81 + new)
    down = [rng.choice(g.keys, back, replace=False) for _ in range(steps)]
    gone = np.zeros(0, np.uint64)  # base edges that are down now
    deg, since = _degrees(n, g.keys), 0
    for k in range(steps):
        ins = np.concatenate([fresh[k], _pairs(gone)])
        if validate and k % 5 == 3:  # a rejected batch leaves list and figures alone
            bad = np.concatenate([ins, ins[:1]])
            if since + len(bad) > dcap:
                deg, since = _degrees(n, pair.keys), 0
            with pytest.raises(drsf.DrsfError):
                if device:
                    import torch
                    with torch.cuda.stream(pair.stream):
                        eb = torch.from_numpy(bad).to(pair.dev)
                    pair.gpu.apply(eb, drsf.DRSF_INSERT)
                else:
                    pair.gpu.apply(bad, drsf.DRSF_INSERT)
        if len(ins):
            if since + len(ins) > dcap:
                deg, since = _degrees(n, pair.keys), 0
            since += len(ins)
            pair.step(ins, drsf.DRSF_INSERT, f"insert {k}")
        dl = np.concatenate([fresh[k - 1] if k else fresh[0][:0], _pairs(down[k])])
        cut = pair.parent.copy()
        u, v = dl[:, 0], dl[:, 1]
        cut[u[cut[u] == v]] = u[cut[u] == v]
        cut[v[cut[v] == u]] = v[cut[v] == u]
        orphans = _roots(cut) != pair.label
        st, _ = pair.step(dl, drsf.DRSF_DELETE, f"delete {k}")
        assert st["num_orphans"] == orphans.sum() and st["orphan_slots"] == deg[orphans].sum(), (k, st)
        gone = down[k]
        if k % 4 == 0:
            assert np.array_equal(pair.gpu.edges(), pair.keys)
    pair.gpu.close()


def test_mixed_ops_share_the_list():
    """Several graphs per call: some delete from the list (positions freed)
    while others insert into it (positions taken), through merge points."""
    drsf = _lib()
    _case("mixed ops on the inserted-edge list")
    ns = [700, 90, 1501, 400]
    graphs = [gen.make_graph(f"g{i}", n, gen.gnm(n, 2 * n, gen.seed(82, i, gen.P_GRAPH))) for i, n in enumerate(ns)]
    mg = gen.multi_graph(graphs)
    per = [40, 7, 90, 23]
    f = drsf.MultiForest(mg.n_off, mg.row_ptr, mg.col, mg.parent, max_batch=256, delta_capacity=600)
    state = []
    for g in graphs:
        r = oracle.apply(g.n, g.keys, g.parent, np.zeros((0, 2), np.int32), oracle.DELETE)
        state.append([g.keys, r.parent, r.label])
    fresh = [gen.insert_batches(n, g.keys, 20, p, gen.seed(82, i, gen.P_INSERT))
             for i, (n, g, p) in enumerate(zip(ns, graphs, per))]
    for call in range(30):
        ops, batches = [], []
        for i in range(len(ns)):
            t = call + i  # graphs out of step: two calls of inserts, then two of deletes
            k = 2 * (t // 4) % 20
            op = drsf.DRSF_INSERT if t % 4 < 2 else drsf.DRSF_DELETE
            b = fresh[i][k + t % 2]
            live = np.isin(gen.keys_of_edges(b), state[i][0])
            b = b[~live] if op == drsf.DRSF_INSERT else b[live]
            ops.append(op)
            batches.append(b)
        b_off = np.concatenate([[0], np.cumsum([len(b) for b in batches])]).astype(np.int64)
        edges = np.concatenate([b + o for b, o in zip(batches, mg.n_off)]).astype(np.int32)
        assert (f.apply_multi(edges, b_off, np.array(ops, np.int8)) == 0).all()
        p, lab = f.parent(), f.label()
        for i, g in enumerate(graphs):
            r = oracle.apply(g.n, state[i][0], state[i][1], batches[i],
                             oracle.INSERT if ops[i] == drsf.DRSF_INSERT else oracle.DELETE, label=state[i][2])
            state[i] = [r.keys, r.parent, r.label]
            o = int(mg.n_off[i])
            assert np.array_equal(p[o:o + g.n] - o, r.parent), (call, i)
            assert np.array_equal(lab[o:o + g.n] - o, r.label), (call, i)
        want = np.sort(np.concatenate([gen.shift_keys(s[0], int(o)) for s, o in zip(state, mg.n_off)]))
        assert np.array_equal(f.edges(), want), call
    f.close()


def test_snapshot_keeps_the_list():
    """A snapshot taken with free and taken list positions, restored after
    further updates of the same merge period."""
    drsf = _lib()
    _case("snapshot of the inserted-edge list")
    n = 2000
    g = gen.make_graph("snap", n, gen.gnm(n, 4000, gen.seed(83, 0, gen.P_GRAPH)))
    fresh = gen.insert_batches(n, g.keys, 6, 100, gen.seed(83, 0, gen.P_INSERT))
    pair = Pair(g, max_batch=256, delta_capacity=2000)
    for b, op in ((fresh[0], 0), (fresh[1], 0), (fresh[0], 1), (_pairs(g.keys[:50]), 1)):
        pair.step(b, op, "before")
    snap = pair.gpu.snapshot()
    was = pair.keys, pair.parent, pair.label
    for _ in range(2):
        for b, op in ((fresh[2], 0), (_pairs(g.keys[:50]), 0), (fresh[1], 1), (fresh[3], 0), (fresh[2], 1)):
            pair.step(b, op, "after")
        pair.gpu.restore(snap)
        pair.keys, pair.parent, pair.label = was
        pair.check_equal("restored")
        assert np.array_equal(pair.gpu.edges(), pair.keys)
    drsf.drsf_snapshot_free(snap)
    pair.gpu.close()


# of 1500 inserted edges `stay` live on (the list keeps at most 187 at a merge point)
@pytest.mark.parametrize("stay", [0, 1, 150])
@pytest.mark.parametrize("launch_mode", [1, 2])
def test_a_burst_that_went_away_leaves_a_short_list(stay, launch_mode):
    """A list filled by edges that are deleted again is as short as its live
    entries after the merge point, and they are found and deleted as before."""
    drsf = _lib()
    _case(f"a burst of inserted edges that goes away: {stay} stay, launch mode {launch_mode}")
    n, dcap = 3001, 1500
    g = gen.make_graph("burst", n, gen.gnm(n, 5003, gen.seed(85, 0, gen.P_GRAPH)))
    pair = Pair(g, max_batch=500, delta_capacity=dcap, launch_mode=launch_mode)
    fresh = gen.insert_batches(n, g.keys, 7, 500, gen.seed(85, 0, gen.P_INSERT))
    burst = np.concatenate(fresh[:3])

    def figures():
        return drsf.drsf_store_figures(pair.gpu.ctx)

    for b in fresh[:3]:
        pair.step(b, drsf.DRSF_INSERT, "burst")
    for k in range(stay, dcap, 500):
        pair.step(burst[k:k + 500], drsf.DRSF_DELETE, "burst goes")
    assert figures() == {"base": len(g.keys), "deleted": 0, "list": dcap, "free": dcap - stay}
    for k in range(2):  # the second round takes and frees positions of the short list
        pair.step(fresh[3 + k][:100], drsf.DRSF_INSERT, "after the merge point")
        assert figures() == {"base": len(g.keys), "deleted": 0, "list": stay + 100, "free": 0}
        assert np.array_equal(pair.gpu.edges(), pair.keys)
        pair.step(fresh[3 + k][:100], drsf.DRSF_DELETE, "again")
        assert figures()["free"] == 100
    if stay:
        pair.step(burst[:stay], drsf.DRSF_DELETE, "the rest of the burst")
    assert np.array_equal(pair.gpu.edges(), g.keys)
    pair.gpu.close()


@pytest.mark.parametrize("gone", [625, 626, 2501])  # of 5003: an eighth, just over it, half
def test_deleted_base_entries_are_dropped(gone):
    """A merge point drops the base store's deleted entries once more than an
    eighth of them are, also where the list's own entries would stay."""
    drsf = _lib()
    _case(f"deleted base entries at a merge point: {gone} of 5003")
    n, dcap = 3001, 1500
    g = gen.make_graph("shrunk", n, gen.gnm(n, 5003, gen.seed(86, 0, gen.P_GRAPH)))
    pair = Pair(g, max_batch=2501, delta_capacity=dcap)
    fresh = gen.insert_batches(n, g.keys, 4, 500, gen.seed(86, 0, gen.P_INSERT))
    down = np.random.default_rng(86).choice(g.keys, gone, replace=False)
    pair.step(_pairs(down), drsf.DRSF_DELETE, "shrink")
    for b in fresh[:3]:
        pair.step(b, drsf.DRSF_INSERT, "short-lived")
        pair.step(b, drsf.DRSF_DELETE, "short-lived")
    was = drsf.drsf_store_figures(pair.gpu.ctx)
    assert was == {"base": 5003, "deleted": gone, "list": 500, "free": 500}
    pair.step(fresh[3][:10], drsf.DRSF_INSERT, "merge point")
    kept = 8 * gone <= 5003
    assert drsf.drsf_store_figures(pair.gpu.ctx) == {
        "base": 5003 if kept else 5003 - gone, "deleted": gone if kept else 0, "list": 10, "free": 0}
    assert np.array_equal(pair.gpu.edges(), pair.keys)
    pair.step(_pairs(down[:300]), drsf.DRSF_INSERT, "some come back")
    assert np.array_equal(pair.gpu.edges(), pair.keys)
    pair.gpu.close()
