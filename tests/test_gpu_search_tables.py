"""The search's three token tables at their limits, exact against the oracle.

A start state with a loop (column 0), an arc into each of n states (column 1),
which have an arc to the next of them (column 2) and one back (column 3), but
every third only an epsilon arc to the next state: a dead end without emitting
arcs until its closure.  A frame lets only one column's arcs into the beam, so
that a token set holds one, two or n survivors.  n lies on both sides of what
the small table's copy of a set holds (2496), of the states the small table
takes (6144) and of those the big one takes (12800); the frames walk from one
table to the next and back.  The rows' widths are no multiple of a fetch.
"""
import numpy as np
import pytest

from paper_1808_00687_amd import workloads as W
import parity
from test_gpu_parity import both, dec, to_dev, torch_mod  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("max_active", [0, 2000])
@pytest.mark.parametrize("n,cols", [(2495, 4), (2496, 67), (2497, 1025), (6143, 7), (6144, 4099), (6145, 9),
                                    (12799, 5), (12800, 6), (12801, 1023)])
def test_search_table_edges(dec, torch_mod, oracle_mod, n, cols, max_active):  # noqa: F811
    rng = np.random.default_rng(n)
    ids = np.arange(1, n + 1)
    dead = ids[(ids % 3 == 0) & (ids < n)]
    live = np.setdiff1d(ids, dead)
    zero = np.zeros(n, np.int64)
    src = np.concatenate([[0], zero, live, live, dead])
    dst = np.concatenate([[0], ids, live % n + 1, live * 0, dead + 1])
    col = np.concatenate([[0], zero + 1, live * 0 + 2, live * 0 + 3, dead * 0 + 4])
    order = np.argsort(src, kind="stable")
    src, dst, col = src[order].astype(np.int32), dst[order].astype(np.int32), col[order]
    # the columns of the four kinds of emitting arc; label 0 is epsilon
    at = np.array([0, 1, cols - 2, cols - 1])
    il = np.where(col < 4, np.append(at + 1, 0)[col], 0)
    # whole-number weights: ties, decided by the lowest arc
    g = W.Graph(n + 1, src, dst, il.astype(np.int32), np.zeros(src.size, np.int32),
                rng.integers(0, 4, size=src.size).astype(np.float32))
    kind = np.array([0, 1, 2, 2, 3, 0, 1, 3, 0, 1])
    ll = np.full((kind.size, cols), -1000.0, np.float32)
    ll[np.arange(kind.size), at[kind]] = rng.integers(-3, 4, size=kind.size)
    ro = oracle_mod.decode(g, ll, 50.0, max_active, 4.0)
    gh = dec.load_graph(g)
    rg = dec.wfst_decode(gh, to_dev(torch_mod, ll), beam=50.0, max_active=max_active, lattice_beam=4.0,
                         record_tokens=True, capacity_hint=n + 8)
    parity.assert_same(ro, rg, lattice=True, tag="%d states, %d columns, max_active %d" % (n, cols, max_active))
    gh.free()


def gated_graph(n, cols, seed):
    """The graph of the module's first paragraph without the dead ends, and the frames' rows."""
    rng = np.random.default_rng(seed)
    ids = np.arange(1, n + 1)
    src = np.concatenate([[0], ids * 0, ids, ids])
    dst = np.concatenate([[0], ids, ids % n + 1, ids * 0])
    col = np.concatenate([[0], ids * 0 + 1, ids * 0 + 2, ids * 0 + 3])
    order = np.argsort(src, kind="stable")
    src, dst, col = src[order].astype(np.int32), dst[order].astype(np.int32), col[order]
    at = np.array([0, 1, cols - 2, cols - 1])
    g = W.Graph(n + 1, src, dst, (at[col] + 1).astype(np.int32), np.zeros(src.size, np.int32),
                rng.integers(0, 4, size=src.size).astype(np.float32))
    kind = np.array([0, 1, 2, 2, 3, 0, 1, 3, 0, 1, 2])
    ll = np.full((kind.size, cols), -1000.0, np.float32)
    ll[np.arange(kind.size), at[kind]] = rng.integers(-3, 4, size=kind.size)
    return g, ll


@pytest.mark.parametrize("permute", [0, 1])
@pytest.mark.parametrize("n,cols", [(12159, 6144), (12160, 6145), (12161, 6144), (17000, 5)])
def test_device_table_set_edges(dec, torch_mod, oracle_mod, n, cols, permute):  # noqa: F811
    # beside the device-memory table (the LDS ones take 100 states here) the
    # LDS copy of a set holds 12,160 tokens, the row 6144 columns
    g, ll = gated_graph(n, cols, n)
    with dec.debug_opts(lds_fill=100, permute=permute):
        ro, rg = both(dec, torch_mod, oracle_mod, g, ll, beam=50.0, lattice_beam=4.0)
    parity.assert_same(ro, rg, lattice=True, tag="%d states, %d columns" % (n, cols))


def test_device_table_without_frames(dec, torch_mod, oracle_mod):  # noqa: F811
    # the start state's closure alone overflows the LDS tables, and there is no row
    g = W.random_small_graph(77, 400, mean_deg=4.0, eps_frac=0.9, num_labels=5)
    ll = W.random_small_loglikes(77, 0, 5)
    with dec.debug_opts(lds_fill=1):
        ro, rg = both(dec, torch_mod, oracle_mod, g, ll, lattice_beam=4.0)
    assert ro.tokens > 1
    parity.assert_same(ro, rg, lattice=True, tag="no frames")


@pytest.mark.parametrize("permute", [0, 1])
@pytest.mark.parametrize("n,deg", [(10000, 8.0), (11500, 8.0)])
def test_device_table_chunks(dec, torch_mod, oracle_mod, n, deg, permute):  # noqa: F811
    # sets of fewer and of more than the 65,536 arcs whose chunks are described
    # beside the device-memory table
    g = W.random_small_graph(n, n, mean_deg=deg, eps_frac=0.2, num_labels=5, weights="int")
    assert ((g.ilabel > 0).sum() > 65536) == (n == 11500)
    ll = W.random_small_loglikes(n, 10, 5, kind="int")
    with dec.debug_opts(lds_fill=100, permute=permute):
        ro, rg = both(dec, torch_mod, oracle_mod, g, ll, lattice_beam=3.0)
    assert ro.tokens > 4 * 9000
    parity.assert_same(ro, rg, lattice=True, tag="%d states" % n)


@pytest.mark.parametrize("permute,queue", [(0, 0), (1, 0), (0, 3)])
@pytest.mark.parametrize("n,deg", [(7000, 3.0), (9500, 5.0), (12700, 4.0), (16000, 4.0)])
def test_tables_on_random_graphs(dec, torch_mod, oracle_mod, n, deg, permute, queue):  # noqa: F811
    # With an infinite beam every reachable state is a token: more than the
    # small table takes, fewer than the big one (or more: 16,000), and at 9,500
    # states and up more than the 32,768 arcs whose chunks are described.  The
    # narrower beam walks between the tables.
    for seed, kind in ((n, "int"), (n + 1, "exp")):
        g = W.random_small_graph(seed, n, mean_deg=deg, eps_frac=0.2, num_labels=5, weights=kind, final=kind == "int")
        ll = W.random_small_loglikes(seed, 14, 5, kind={"int": "int", "exp": "gauss"}[kind])
        for beam in (float("inf"), 7.0):
            with dec.debug_opts(permute=permute, queue_cap=queue):
                ro, rg = both(dec, torch_mod, oracle_mod, g, ll, beam=beam, lattice_beam=3.0)
            parity.assert_same(ro, rg, lattice=True, tag="%d states, beam %g, %s weights" % (n, beam, kind))
