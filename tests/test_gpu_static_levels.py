"""The static rebuild where its kernels divide the work: rows of 32 and 33
slots (one workgroup's levels), 64 and 65 (a lane's part of a bottom-up row),
1024 and 1025 (a hub's row), frontiers of 511 to 513, more levels than one
launch does, columns that two XCDs' blocks both link, rows in any order, and
rows skipped inside the sampled component.  Whole numbers: compared exactly."""
import numpy as np
import pytest

import gen
from test_gpu_static import _run
from test_zz_no_alloc import _both

pytestmark = pytest.mark.gpu


def _keys(u, v):
    u, v = np.asarray(u, np.uint64), np.asarray(v, np.uint64)
    keep = u != v
    lo, hi = np.minimum(u, v)[keep], np.maximum(u, v)[keep]
    return np.unique((lo << np.uint64(32)) | hi)


def _graph(name, n, u, v, rng=None):
    """Optionally with vertices renamed and every row's slots shuffled."""
    u, v = np.asarray(u), np.asarray(v)
    if rng is not None:
        p = rng.permutation(n)
        u, v = p[u], p[v]
    g = gen.make_graph(name, n, _keys(u, v))
    if rng is not None:
        row = np.repeat(np.arange(n), np.diff(g.row_ptr))
        g.col[:] = g.col[np.lexsort((rng.random(g.col.size), row))]
    return g


@pytest.mark.parametrize("shuffled", [False, True])
@pytest.mark.parametrize("d", [31, 32, 33, 64, 65, 1023, 1024, 1025, 5000])
def test_rows_at_the_edges_of_the_walks(d, shuffled):
    # three hubs in a chain, d - 1 leaves each and a tail
    n = 3 + 3 * d + 40
    u = [0, 1] + [h for h in range(3) for _ in range(d)] + list(range(n - 41, n - 1))
    v = [1, 2] + list(range(3, 3 + 3 * d)) + list(range(n - 40, n))
    _run(_graph("hubs", n, u, v, np.random.default_rng(d) if shuffled else None), f"hubs {d} {shuffled}")


@pytest.mark.parametrize("k", [511, 512, 513, 2100])
def test_frontiers_at_the_edge_of_one_workgroup(k):
    # k legs of five vertices from a root
    legs = np.arange(k * 5).reshape(k, 5) + 1
    u = np.concatenate([np.zeros(k, np.int64), legs[:, :-1].ravel()])
    v = np.concatenate([legs[:, 0], legs[:, 1:].ravel()])
    assert _run(_graph("spider", k * 5 + 1, u, v), f"spider {k}") == 6
    _run(_graph("spider", k * 5 + 1, u, v, np.random.default_rng(k)), f"spider {k} shuffled")


@pytest.mark.parametrize("n", [4096, 4097, 4098, 8200])
def test_more_levels_than_one_launch(n):
    i = np.arange(n - 1)
    assert _run(_graph("path", n, i, i + 1), f"path {n}") == n


def test_columns_linked_by_two_blocks():
    rows, cols = 96, 2048
    g = gen.make_graph("grid", rows * cols, gen.grid(rows, cols, 900, gen.seed(16, 5, gen.P_GRAPH)))
    for k in range(3):
        _run(g, f"grid {rows} x {cols}, call {k}")


@pytest.mark.parametrize("m", [200, 6000, 9000, 40000])
def test_outside_the_sampled_component(m):
    n = 12011
    rng = np.random.default_rng(m)
    u, v = rng.integers(0, n, m), rng.integers(0, n, m)
    _both(_graph("random", n, u, v, rng), f"random {m}")
    # two equal halves: whichever is sampled, the other walks its rows
    half = n // 2
    _both(_graph("halves", n, u % half + (v % 2) * half, v % half + (v % 2) * half, rng), f"halves {m}")
