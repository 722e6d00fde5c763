"""The decodes whose speed is measured: which calls, on which graphs, with which inputs.

A case names a graph family with its size, the utterances of one call, and the
call's options.  The families and their default sizes are the ones of
``paper_1808_00687_amd/workloads.py`` (synthetic stand-ins for a small
grammar, a medium graph and an LVCSR graph with a hybrid acoustic model, and
for CTC and HMM topologies with blank-like units):

* ``tiny``: 1 + Poisson(3) arcs per state, 15% epsilon, labels read N(0, 2) logits;
* ``medium``: 5 arcs per state, 12% epsilon, N(0, 3) logits, output labels on 30% of the arcs;
* ``lvcsr``: 2.5 arcs per state, 20% epsilon, N(0, 3) logits, output labels on 10% of the arcs;
* ``ctc``: a blank self-loop on every state and 2 more arcs per state, 15% of those epsilon;
  the blank dominates 85% of the frames;
* ``hmm``: as ``ctc``, each self-loop on one of 8 blank-like units, drawn per state; one of
  those units, drawn per frame, dominates 85% of the frames.

A graph belongs to its case and is loaded once per process, as a program that
serves decodes keeps its graph; the log-likelihoods come from the seed.
Decoding is exact (results do not depend on the order of the work), so every
output has to be the same bit for bit.
"""
import collections
import math

import numpy as np
import torch

from paper_1808_00687_amd import wfstdec, workloads

BLANK_UNITS = 8       # blank-like units of the hmm family (columns 0 .. 7)
BOOST = 8.0           # logit added to a dominating blank unit
P_BLANK = 0.85        # share of frames it dominates
VOCABULARY = 50       # output labels of the medium family
GRAPHS_KEPT = 8       # graphs that stay loaded in one process
LATTICE_ARCS = {"tiny": 400, "medium": 64, "lvcsr": 16, "ctc": 16, "hmm": 64}   # room per frame for kept arcs

# arcs per state (rank law, mean), epsilon share, mean weight, logit deviation, share of arcs with an output label
FAMILIES = {
    "tiny": (4.0, 0.15, 1.5, 2.0, 0.0),
    "medium": (5.0, 0.12, 2.0, 3.0, 0.3),
    "lvcsr": (2.5, 0.20, 2.5, 3.0, 0.1),
    "ctc": (2.0, 0.15, 2.0, 1.0, 0.0),
    "hmm": (2.0, 0.15, 2.0, 1.0, 0.0),
}

DEFAULTS = {
    "call": "decode",         # wfst_decode, "batch" (wfst_decode_batch) or "noalloc" (wfst_decode_noalloc)
    "utterances": 1,
    "max_active": 0,
    "lattice_beam": -1.0,     # no lattice
    "threshold": 2.0,         # frame-synchronous
    "stride": 1,
    "words": False,           # word-level lattice
    "incremental": False,     # lattice pruned beside the search
    "host": False,            # log-likelihoods in host memory
}


def listed():
    """The calls of the repository's benchmark configurations and of the options that serving uses."""
    lv = {"family": "lvcsr", "states": 10_000_000, "labels": 6000, "beam": 15.0, "max_active": 10000}
    md = {"family": "medium", "states": 200_000, "labels": 2000, "beam": 13.0, "max_active": 7000}
    ct = {"family": "ctc", "states": 5_000_000, "labels": 80, "beam": 14.0, "max_active": 8000, "lattice_beam": 8.0}
    hm = dict(ct, family="hmm")
    return [
        # a short command against a small grammar, one best path: the latency of a call
        {"name": "command", "family": "tiny", "states": 2000, "labels": 64, "t_min": 50, "t_max": 50, "beam": 12.0},
        # an utterance on a medium graph with wide beams: thousands of tokens per frame
        {"name": "medium-lattice", **md, "t_min": 500, "t_max": 500, "lattice_beam": 8.0},
        # the same graph for second-pass rescoring: every word sequence of the lattice
        {"name": "medium-words", **md, "t_min": 120, "t_max": 120, "lattice_beam": 6.0, "words": True},
        # one utterance of 10 s on the LVCSR graph (interactive use)
        {"name": "lvcsr-one", **lv, "t_min": 1000, "t_max": 1000, "lattice_beam": 8.0},
        # offline transcription: the batch of the benchmark, and one that fills the chip
        {"name": "lvcsr-64", "call": "batch", **lv, "utterances": 64, "t_min": 300, "t_max": 1500, "lattice_beam": 8.0},
        {"name": "lvcsr-256", "call": "batch", **lv, "utterances": 256, "t_min": 300, "t_max": 1500,
         "lattice_beam": 8.0},
        # a few ragged short utterances, best paths only (live captions of several speakers)
        {"name": "lvcsr-11-best", "call": "batch", **lv, "utterances": 11, "t_min": 37, "t_max": 423},
        # lattices with a bounded workspace
        {"name": "lvcsr-24-incremental", "call": "batch", **lv, "utterances": 24, "t_min": 300, "t_max": 700,
         "lattice_beam": 8.0, "incremental": True},
        # a CTC model: one long utterance label-synchronously, and a ragged batch frame by frame
        {"name": "ctc-lsd", **ct, "t_min": 2000, "t_max": 2000, "threshold": 0.95},
        {"name": "ctc-23-fsd", "call": "batch", **ct, "utterances": 23, "t_min": 300, "t_max": 1500},
        # the HMM topology, log-likelihoods from a host-side model; and at a third of the frame rate in a
        # program that may not allocate
        {"name": "hmm-lsd", **hm, "t_min": 2000, "t_max": 2000, "threshold": 0.95, "host": True},
        {"name": "hmm-stride3-noalloc", "call": "noalloc", **hm, "t_min": 701, "t_max": 701, "threshold": 0.95,
         "stride": 3},
    ]


def _spread(rng, lo, hi):
    """A whole number of [lo, hi], spread over its logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    family = rng.choice(["tiny", "medium", "lvcsr", "lvcsr", "ctc", "hmm"])
    c = {"family": family, "call": rng.choice(["decode", "batch", "batch"])}
    if family == "tiny":
        c.update(states=_spread(rng, 300, 20_000), labels=_spread(rng, 24, 300), beam=rng.uniform(8.0, 12.0),
                 t_max=_spread(rng, 10, 400), max_active=rng.choice([0, 300, 1000]),
                 lattice_beam=rng.choice([-1.0, 4.0, 8.0]))
        most = 24
    elif family == "medium":
        c.update(states=_spread(rng, 30_000, 400_000), labels=_spread(rng, 300, 4000), beam=rng.uniform(10.0, 13.0),
                 t_max=_spread(rng, 40, 500), max_active=rng.choice([2000, 5000, 7000]),
                 lattice_beam=rng.choice([-1.0, 6.0, 8.0]))
        most = 24
    elif family == "lvcsr":
        c.update(states=_spread(rng, 500_000, 10_000_000), labels=_spread(rng, 1500, 9000),
                 beam=rng.uniform(13.0, 15.0), t_max=_spread(rng, 80, 1500), max_active=rng.choice([2000, 7000, 10000]),
                 lattice_beam=rng.choice([-1.0, 6.0, 8.0]))
        most = 160
        c["incremental"] = c["lattice_beam"] >= 0 and rng.random() < 0.15
    else:
        c.update(states=_spread(rng, 200_000, 5_000_000), labels=_spread(rng, 40, 300), beam=rng.uniform(10.0, 14.0),
                 t_max=_spread(rng, 150, 2000), max_active=rng.choice([2000, 8000]),
                 lattice_beam=rng.choice([-1.0, 6.0, 8.0]), threshold=rng.choice([0.95, 0.95, 2.0]))
        most = 24
        if family == "hmm":
            c["stride"] = rng.choice([1, 1, 2, 3])
        if c["call"] == "decode":
            c["host"] = rng.random() < 0.3
            if not c["host"] and rng.random() < 0.3:
                c.update(call="noalloc", t_max=min(c["t_max"], 900))
    c["utterances"] = _spread(rng, 2, most) if c["call"] == "batch" else 1
    c["t_min"] = c["t_max"] // rng.choice([1, 2, 5]) if c["utterances"] > 1 else c["t_max"]
    return c


def _options(case):
    return {**DEFAULTS, **case}


# ---- graphs ----

def _degrees(family, n, rng):
    mean = FAMILIES[family][0]
    if family == "tiny":
        return 1 + rng.poisson(mean - 1.0, size=n)
    return workloads.rank_law_degrees(n, int(mean * n), 1.2, 200, rng)


def _graph(case):
    """The case's arcs, sorted by source, the same at every call."""
    c = _options(case)
    family, n, labels = c["family"], c["states"], c["labels"]
    _, eps, mean_w, _, out = FAMILIES[family]
    rng = np.random.default_rng([1808, 687, sorted(FAMILIES).index(family), n, labels])
    deg = _degrees(family, n, rng)
    loops = {"ctc": 1, "hmm": BLANK_UNITS}.get(family, 0)
    a = workloads.arcs_from_degrees(n, deg, eps, labels, mean_w, rng, first_label=loops + 1)
    if loops:
        # a self-loop on a blank unit in front of each state's other arcs
        first = np.zeros(n, np.int64)
        np.cumsum(deg[:-1] + 1, out=first[1:])
        other = np.ones(n + a["src"].size, bool)
        other[first] = False
        own = dict(src=np.arange(n, dtype=np.int32), dst=np.arange(n, dtype=np.int32),
                   ilabel=rng.integers(1, loops + 1, size=n, dtype=np.int32),
                   weight=rng.exponential(mean_w, size=n).astype(np.float32))
        both = {}
        for k, v in a.items():
            both[k] = np.empty(other.size, v.dtype)
            both[k][first] = own[k]
            both[k][other] = v
        a = both
    ol = np.zeros(a["src"].size, np.int32)
    if out:
        has = rng.random(ol.size) < out
        ol[has] = rng.integers(1, VOCABULARY, size=int(has.sum()))
    return workloads.Graph(n, a["src"], a["dst"], a["ilabel"], ol, a["weight"])


_loaded = collections.OrderedDict()


def _handle(case):
    key = (case["family"], case["states"], case["labels"])
    if key not in _loaded:
        _loaded[key] = wfstdec.load_graph(_graph(case))
        while len(_loaded) > GRAPHS_KEPT:
            _loaded.popitem(last=False)
    _loaded.move_to_end(key)
    return _loaded[key]


# ---- inputs ----

def _loglikes(case, seed):
    """One [T x labels] tensor of log-likelihoods per utterance, on the GPU."""
    c = _options(case)
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed))
    lens = workloads.batch_lengths(c["utterances"], c["t_min"], c["t_max"])
    sigma = FAMILIES[c["family"]][3]
    units = {"ctc": 1, "hmm": BLANK_UNITS}.get(c["family"], 0)
    out = []
    for t in (int(x) for x in lens):
        z = torch.randn(t, c["labels"], generator=gen, device=dev) * sigma
        if units:
            boost = (torch.rand(t, generator=gen, device=dev) < P_BLANK) * BOOST
            unit = torch.randint(0, units, (t,), generator=gen, device=dev)
            z[torch.arange(t, device=dev), unit] += boost
        out.append(torch.log_softmax(z, dim=1))
    return out


def prepare(case, seed):
    c = _options(case)
    lls = _loglikes(case, seed)
    if c["host"]:
        lls = [x.cpu().numpy() for x in lls]
    args = dict(beam=c["beam"], max_active=c["max_active"], lattice_beam=c["lattice_beam"],
                blank_threshold=c["threshold"], frame_stride=c["stride"])
    if c["family"] == "hmm":
        args["blank_ids"] = tuple(range(BLANK_UNITS))
    state = {"call": c["call"], "graph": _handle(c), "loglikes": lls, "args": args}
    if c["call"] == "noalloc":
        def device(*n):
            return torch.zeros(*n, dtype=torch.int32, device="cuda:0")
        # path arcs, path frames, lattice records and decoded frames: owned and kept by the program
        args["outputs"] = (device(16384), device(16384), device(1 << 18, 4), device(4096))
        return state
    args.update(word_lattice=c["words"], incremental_lattice=c["incremental"])
    # the arrays the program gathers the utterances' results in, one utterance after another
    frames = sum(x.shape[0] for x in lls)
    size = {"kept": frames, "path_arcs": 4 * frames + 64, "path_frames": 4 * frames + 64}
    if c["lattice_beam"] >= 0:
        size.update({k: LATTICE_ARCS[c["family"]] * (frames + 1) for k in _LATTICE})
    if c["words"]:
        size.update(words=1 << 20, words_n=1 << 16, word_costs=1 << 16)
    state["out"] = {k: np.zeros(n, np.float32 if k.endswith(("cost", "extra", "costs")) else np.int32)
                    for k, n in size.items()}
    state["used"] = dict.fromkeys(size, 0)
    return state


# ---- one pass ----

_LATTICE = ("lat_frame", "lat_arc", "lat_cost", "lat_extra")
_COUNTS = ("tokens", "arcs_expanded", "eps_arcs", "lattice_raw", "lattice_kept")


def _gather(state, name, parts):
    """The parts one after another at the front of the program's array, zeros behind them."""
    to, n = state["out"][name], 0
    for x in parts:
        to[n:n + len(x)] = x
        n += len(x)
    to[n:state["used"][name]] = 0
    state["used"][name] = n


def run(state):
    args = state["args"]
    if state["call"] == "noalloc":
        r = wfstdec.wfst_decode_noalloc(state["graph"], state["loglikes"][0], **args)
        return {"rc": r.rc, "cost": r.cost, "final_state": r.final_state, "tokens": r.tokens,
                "arcs_expanded": r.arcs_expanded, "num_decoded": r.num_decoded, "path_len": r.path_len,
                "lattice_n": r.lattice_n, "kept": r.kept, "path_arcs": r.path_arcs, "path_frames": r.path_frames,
                "lattice": r.lattice}
    if state["call"] == "decode":
        res = [wfstdec.wfst_decode(state["graph"], state["loglikes"][0], **args)]
    else:
        res = wfstdec.wfst_decode_batch(state["graph"], state["loglikes"], **args)
    ok = [r for r in res if r.status == wfstdec.WFST_OK]
    for k in state["out"]:
        if not k.startswith("word"):
            _gather(state, k, [getattr(r, k) for r in ok])
    if args["word_lattice"]:
        words = res[0].words or []
        _gather(state, "words", [seq for seq, _ in words])
        _gather(state, "words_n", [[len(seq) for seq, _ in words]])
        _gather(state, "word_costs", [[c for _, c in words]])
    out = {"status": np.array([r.status for r in res]), "cost": np.array([r.cost for r in res], np.float32),
           "final_state": np.array([r.final_state for r in res]),
           "counts": np.array([[r.stats[k] for k in _COUNTS] + [r.num_decoded] +
                               ([r.path_arcs.size] if r.status == wfstdec.WFST_OK else [0]) for r in res])}
    out.update(state["out"])
    return out


# ---- what a pass cannot do without ----

# Tokens, emitting arcs and epsilon arcs per decoded frame that the decodes of
# the listed cases report (beams as listed; a narrower beam keeps fewer: about a factor e per 3 units).
_PER_FRAME = {"tiny": (1285, 4160, 775), "medium": (4300, 19000, 2600), "lvcsr": (1190, 2380, 595),
              "ctc": (3, 5.6, 0.6), "hmm": (140, 360, 40)}
_BEAM = {"tiny": 12.0, "medium": 13.0, "lvcsr": 15.0, "ctc": 14.0, "hmm": 14.0}


def work(case):
    c = _options(case)
    lens = workloads.batch_lengths(c["utterances"], c["t_min"], c["t_max"]).astype(float)
    frames = float(lens.sum()) / c["stride"]
    if c["threshold"] <= 1.0:
        frames *= 0.5      # of the dominated frames, about three in five pass the threshold
    scale = math.exp(min(0.0, (c["beam"] - _BEAM[c["family"]]) / 3.0))
    tok, arcs, eps = (scale * x for x in _PER_FRAME[c["family"]])
    # per token its state, cost and two row offsets; per emitting arc its
    # destination, label, weight, log-likelihood and the token it may lower;
    # per epsilon arc its destination, weight and token; 16 bytes per
    # path or lattice arc (about two per frame)
    b = frames * (16 * tok + 24 * arcs + 16 * eps + 16 * 2)
    return {"bytes": b, "flops": frames * (2 * arcs + eps)}


def tolerance(case):
    return "exact"


# ---- the best path's cost in 64 bits ----

def _relax(cost, src_cost, row, dst, weight, states, score=None):
    """Lower cost[] over the arcs of `states` (rows of a CSR table); returns the arcs' destinations that went down."""
    lo, hi = row[states], row[states + 1]
    n = hi - lo
    if not int(n.sum()):
        return np.zeros(0, np.int64)
    at = np.repeat(lo - np.concatenate([[0], np.cumsum(n)[:-1]]), n) + np.arange(int(n.sum()))
    c = np.repeat(src_cost, n) + weight[at]
    if score is not None:
        c = c - score(at)
    d = dst[at]
    low = c < cost[d]
    np.minimum.at(cost, d[low], c[low])
    return np.unique(d[low])


def exact(case, seed):
    """Beam search in float64: the cost of the best path (one utterance a call; a batch would take minutes)."""
    c = _options(case)
    if c["utterances"] > 1:
        return None
    g = _graph(case)
    n = g.num_states
    emit = g.ilabel > 0
    rows = {}
    for kind, pick in (("emit", emit), ("eps", ~emit)):
        row = np.zeros(n + 1, np.int64)
        np.cumsum(np.bincount(g.src[pick], minlength=n), out=row[1:])
        rows[kind] = (row, g.dst[pick].astype(np.int64), g.weight[pick].astype(np.float64))
    col = g.ilabel[emit].astype(np.int64) - 1
    ll = _loglikes(case, seed)[0].cpu().numpy()
    blank = {"ctc": [0], "hmm": list(range(BLANK_UNITS))}.get(c["family"], [0])
    frames = np.arange(0, ll.shape[0], c["stride"])
    if c["threshold"] <= 1.0:
        thr = np.float32(math.log(c["threshold"]))
        frames = frames[~(ll[frames][:, blank] > thr).any(axis=1)]
    cost = np.full(n, np.inf)
    old = np.array([0])
    old_cost = np.zeros(1)
    for j in range(-1, frames.size):
        if j < 0:
            cost[0] = 0.0
            seen = old
        else:
            x = ll[frames[j]].astype(np.float64)
            seen = _relax(cost, old_cost, *rows["emit"], old, score=lambda at: x[col[at]])
        found, fresh = [seen], seen
        while fresh.size:
            fresh = _relax(cost, cost[fresh], *rows["eps"], fresh)
            found.append(fresh)
        seen = np.unique(np.concatenate(found))
        v = cost[seen]
        cost[seen] = np.inf
        keep = v <= v.min() + c["beam"]
        if 0 < c["max_active"] < int(keep.sum()):
            keep &= v <= np.partition(v, c["max_active"] - 1)[c["max_active"] - 1]
        old, old_cost = seen[keep], v[keep]
    best = float(old_cost.min())
    return {"cost": best if c["call"] == "noalloc" else np.array([best])}
