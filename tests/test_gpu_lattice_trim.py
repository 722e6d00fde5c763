"""The chunk pruning before the lattice backward pass, exact against the oracle.

Utterances on both sides of the 512 frames from which it runs and of multiples
of its chunks' 32 sets; LDS limits that leave some sets of a chunk, or all,
whole; and a batch large enough for the smaller table.  About 250 states, most
of them reached every frame, with epsilon arcs and ties.
"""
import numpy as np
import pytest

from paper_1808_00687_amd import workloads as W
import parity
from test_gpu_parity import both, dec, to_dev, torch_mod  # noqa: F401
from test_gpu_search_tables import gated_graph

pytestmark = pytest.mark.gpu


def case(seed, frames):
    g = W.random_small_graph(3000 + seed, 250, mean_deg=3.0, eps_frac=0.25, num_labels=5,
                             weights=["int", "exp"][seed % 2], final=seed % 3 == 0)
    return g, W.random_small_loglikes(3000 + seed, frames, 5, kind=["int", "gauss"][seed % 2])


@pytest.mark.parametrize("frames,cap,beam", [(511, 0, 9.0), (512, 0, 9.0), (513, 0, float("inf")), (543, 0, 7.0),
                                             (545, 100, 7.0), (520, 60, 5.0), (512, 1, 9.0)])
def test_trimmed_lattice(dec, torch_mod, oracle_mod, frames, cap, beam):  # noqa: F811
    for seed in (frames, frames + 1):
        g, ll = case(seed, frames)
        with dec.debug_opts(lattice_lds=cap):
            ro, rg = both(dec, torch_mod, oracle_mod, g, ll, beam=beam, lattice_beam=4.0)
        parity.assert_same(ro, rg, lattice=True, tag="%d frames, cap %d, seed %d" % (frames, cap, seed))


def test_trimmed_lattice_batch(dec, torch_mod, oracle_mod):  # noqa: F811
    g, ll = case(1, 540)
    lls = [to_dev(torch_mod, ll[: 505 + u % 36]) for u in range(180)]
    gh = dec.load_graph(g)
    res = dec.wfst_decode_batch(gh, lls, 9.0, 0, 4.0, record_tokens=True)
    for u in range(0, 36, 5):
        ro = oracle_mod.decode(g, ll[: 505 + u], 9.0, 0, 4.0)
        for r in (res[u], res[u + 144]):
            parity.assert_same(ro, r, lattice=True, tag="batch %d" % u)
    gh.free()


def decode_copies(dec, torch_mod, g, ll, copies, **o):  # noqa: F811
    """The utterance `copies` times in one call: one of them gets the kernel of 1,024 threads and 8192
    survivors (up to 512 blocks of 32 sets), 31 of more than 512 frames the one of half that."""
    gh = dec.load_graph(g)
    x = to_dev(torch_mod, ll)
    res = dec.wfst_decode_batch(gh, [x] * copies, record_tokens=True, **o)
    gh.free()
    return res[0], res[-1]


@pytest.mark.parametrize("copies,n,ne,nx,beam", [
    (1, 600, 2047, 2049, 1.0), (1, 600, 2048, 2048, 3.0), (1, 600, 2049, 2047, 1.0), (1, 900, 6200, 4200, 3.0),
    (31, 400, 1023, 1025, 1.0), (31, 400, 1024, 1024, 3.0), (31, 400, 1025, 1023, 1.0), (31, 500, 3100, 2100, 3.0)])
def test_trim_in_several_rounds(dec, torch_mod, oracle_mod, copies, n, ne, nx, beam):  # noqa: F811
    # A round takes two records a thread.  Every state has a loop and an arc
    # from the start state, so with an infinite beam every set but the first
    # holds all states and as many raw records as the graph has arcs.
    rng = np.random.default_rng(ne + nx)
    ids = np.arange(n)
    low = rng.integers(0, n - 1, size=nx)
    src = np.concatenate([ids, np.zeros(n - 1, np.int64), rng.integers(0, n, size=ne - 2 * n + 1), low])
    dst = np.concatenate([ids, ids[1:], rng.integers(0, n, size=ne - 2 * n + 1),
                          low + 1 + (rng.random(nx) * (n - 1 - low)).astype(np.int64)])
    il = np.concatenate([rng.integers(1, 6, size=ne), np.zeros(nx, np.int64)])
    order = np.argsort(src, kind="stable")
    g = W.Graph(n, src[order].astype(np.int32), dst[order].astype(np.int32), il[order].astype(np.int32),
                np.zeros(ne + nx, np.int32), rng.integers(0, 4, size=ne + nx).astype(np.float32))
    frames = 530
    ll = W.random_small_loglikes(ne + nx, frames, 5, kind="int")
    inf = float("inf")
    ro = oracle_mod.decode(g, ll, inf, 0, beam)
    assert ro.lat_raw >= (frames - 1) * (ne + nx)
    for r in decode_copies(dec, torch_mod, g, ll, copies, beam=inf, max_active=0, lattice_beam=beam):
        parity.assert_same(ro, r, lattice=True, tag="%d x %d + %d records" % (copies, ne, nx))


@pytest.mark.parametrize("copies,n", [(1, 8191), (1, 8192), (1, 8193), (31, 4095), (31, 4096), (31, 4097)])
def test_trim_survivor_limit(dec, torch_mod, oracle_mod, copies, n):  # noqa: F811
    # sets of n survivors among sets of one, across the border of a chunk of
    # 32 sets and inside one; a set beyond the kernel's arrays is left whole
    g, ll0 = gated_graph(n, 4, n)
    one, seq = ll0[:1], ll0[[1, 2, 3, 7]]
    parts = [one] * 29 + [seq] + [one] * 12 + [seq] + [one] * 100 + [seq]
    ll = np.concatenate(parts + [one] * (530 - sum(len(x) for x in parts)))
    ro = oracle_mod.decode(g, ll, 50.0, 0, 4.0)
    assert ro.lat_raw > 64 * 531 and np.diff(ro.tok_off).max() == n
    for r in decode_copies(dec, torch_mod, g, ll, copies, beam=50.0, max_active=0, lattice_beam=4.0):
        parity.assert_same(ro, r, lattice=True, tag="%d x %d survivors" % (copies, n))
