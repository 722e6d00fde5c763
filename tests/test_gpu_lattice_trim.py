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
