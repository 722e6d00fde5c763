"""States without emitting arcs, which own a placeholder record on the device.

A placeholder reaches nothing, so it may take no room: no lattice record slot
of a fixed workspace and no slot of a token table.  Exact against
wfst_decode and the oracle.
"""
import numpy as np
import pytest

from paper_1808_00687_amd import workloads as W
import parity
from test_gpu_parity import both, dec, to_dev, torch_mod  # noqa: F401
from test_zz_no_alloc import _same

pytestmark = pytest.mark.gpu


def test_fixed_workspace_capacity(dec, torch_mod):  # noqa: F811
    # 60 states with two emitting arcs each on average, a third of them
    # without any.  56,000 frames of up to 60 tokens need 152 bytes a token
    # (32 of the survivor arrays, 5 emitting and one epsilon record slot of 20)
    # and 92 a frame: 516 of the fixed workspace's 536.9 million bytes.  One
    # more slot a token (20 * 60 * 56,000 = 67 million) would not fit.
    n, frames = 60, 56_000
    rng = np.random.default_rng(60)
    live = np.flatnonzero(np.arange(n) % 3 < 2)
    src = np.sort(np.concatenate([live, rng.choice(live, 2 * n - live.size)])).astype(np.int32)
    dst = rng.integers(0, n, size=src.size).astype(np.int32)
    g = W.Graph(n, src, dst, rng.integers(1, 5, size=src.size).astype(np.int32), np.zeros(src.size, np.int32),
                rng.integers(0, 4, size=src.size).astype(np.float32))
    x = to_dev(torch_mod, W.random_small_loglikes(60, frames, 4, kind="int"))
    gh = dec.load_graph(g)
    got = dec.wfst_decode_noalloc(gh, x, 6.0, 0, 2.0, path_cap=1 << 17, lattice_cap=1 << 22, kept_cap=frames)
    assert got.rc == 0, got.rc
    _same(dec.wfst_decode(gh, x, 6.0, 0, 2.0), got, "%d frames" % frames)
    gh.free()


def test_table_slots(dec, torch_mod, oracle_mod):  # noqa: F811
    # With an infinite beam every candidate is within the early-drop bound.
    # Frame 1 reaches n dead ends and one live state, frame 2 from that one n
    # states more: each n fits the largest token table a graph of this size
    # gets (24,576 states), the two of them do not.
    n = 14_000
    ids = np.arange(n)
    live = 1 + n
    src = np.concatenate([np.zeros(n + 1), np.full(n, live), live + 1 + ids]).astype(np.int32)
    dst = np.concatenate([1 + ids, [live], live + 1 + ids, live + 1 + ids]).astype(np.int32)
    rng = np.random.default_rng(14)
    g = W.Graph(2 * n + 2, src, dst, rng.integers(1, 4, size=src.size).astype(np.int32), np.zeros(src.size, np.int32),
                rng.integers(0, 4, size=src.size).astype(np.float32))
    ll = W.random_small_loglikes(14, 3, 3, kind="int")
    inf = float("inf")
    ro, rg = both(dec, torch_mod, oracle_mod, g, ll, beam=inf, lattice_beam=inf)
    assert ro.tokens == 1 + (n + 1) + n + n
    parity.assert_same(ro, rg, lattice=True, tag="%d dead ends" % n)
