"""Back-pointers and lattice records at the edges of the record pass's tables.

A start state with a loop (column 0), an arc into each of n states (column 1),
which have an arc to the next of them (column 2) and one back (column 3); a
frame lets only one column's arcs into the beam, so that a token set holds
exactly one or n survivors.  n lies on both sides of the small table's limit
(3072 survivors) and at the middle one's (6144), the log-likelihood
rows on both sides of the 4096 columns kept in LDS, and the sets of the
utterance on both sides of the 2048 up to which one launch takes all and of a
multiple of eight, the shares a launch divides them into.  Exact against the
oracle.
"""
import numpy as np
import pytest

from paper_1808_00687_amd import workloads as W
import parity
from test_gpu_parity import both, dec, torch_mod  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,cols,frames", [(3071, 4096, 2047), (3072, 4097, 2048), (3073, 4096, 2055),
                                           (6144, 5, 2056), (700, 5, 8), (70, 4096, 7)])
def test_record_table_edges(dec, torch_mod, oracle_mod, n, cols, frames):  # noqa: F811
    rng = np.random.default_rng(n)
    ids = np.arange(1, n + 1)
    zero = np.zeros(n, np.int64)
    src = np.concatenate([[0], zero, ids, ids])
    dst = np.concatenate([[0], ids, np.roll(ids, 1), zero])
    col = np.concatenate([[0], zero + 1, zero + 2, zero + 3])
    order = np.argsort(src, kind="stable")
    src, dst, col = src[order].astype(np.int32), dst[order].astype(np.int32), col[order]
    # the columns of the four kinds of arc: the row's first and last ones
    at = np.array([0, 1, cols - 2, cols - 1])
    # whole-number weights: ties, decided by the lowest arc
    g = W.Graph(n + 1, src, dst, (at[col] + 1).astype(np.int32), np.zeros(src.size, np.int32),
                rng.integers(0, 4, size=src.size).astype(np.float32))
    kind = np.zeros(frames, np.int64)
    for t in (0, frames // 2, frames - 3):
        kind[t:t + 3] = (1, 2, 3)
    kind[-1] = 2
    ll = np.full((frames, cols), -1000.0, np.float32)
    ll[np.arange(frames), at[kind]] = rng.integers(-3, 4, size=frames)
    ro, rg = both(dec, torch_mod, oracle_mod, g, ll, beam=50.0, lattice_beam=4.0)
    parity.assert_same(ro, rg, lattice=True, tag="%d survivors, %d columns, %d frames" % (n, cols, frames))


@pytest.mark.parametrize("n,cols,frames", [(3072, 4096, 2048), (3071, 4095, 2056), (6145, 4096, 2048)])
def test_record_table_edges_two_launches(dec, torch_mod, oracle_mod, n, cols, frames):  # noqa: F811
    # more than 2048 sets: the small table at its limit with the row in LDS,
    # and a set beyond the middle table's limit
    test_record_table_edges(dec, torch_mod, oracle_mod, n, cols, frames)
