"""The work that users of the graph builder have it do, as timed cases.

Every case is one pass through a public entry point of paper_2202_06929_amd.frnn on
inputs with the distributions of the repository's own events (events.py): clusters
that stand for tracks over a uniform background.  The kinds:

  build     frnn.build_into: one event into the loop's own buffers, the edge count
            waited for; the call of a plain event loop
  step      frnn.AsyncBatch over one event or a batch: workspace and outputs kept,
            nothing waited for; one step of a pipeline between two GPU stages
  served    frnn.build_events_async: a few events in tensors of their own, what the
            server launches for the requests that arrived together
  label     frnn.components: track labels of a graph, allocated and waited for
  label_step  frnn.components_async: the same into kept buffers

listed() names the cases; draw() gives more of the same ranges; see each entry for
what it stands for.  All results are whole numbers (edges, ranges, labels), so no
case has a 64-bit reference: exact() returns None.
"""

import dataclasses
import math

import numpy as np
import torch

from paper_2202_06929_amd import events, frnn

DEVICE = "cuda:0"


def _event(n, d, r, K, size_lo, size_hi, spread, noise, **more):
    """One event's shape.  `spread` is the root mean square distance of two points of
    a cluster in units of r (0.8 in the repository's single event)."""
    return {"n": n, "d": d, "r": r, "K": K, "size_lo": size_lo, "size_hi": size_hi, "spread": spread,
            "noise": noise, **more}


def listed():
    return [
        # A small event: 2,000 hits, where launches and the host path are the time.
        {"name": "tiny_2k", "kind": "build", **_event(2_000, 8, 0.1, 64, 8, 15, 0.8, 0.10)},
        # An ordinary event of a ragged size in a ten-coordinate embedding (rows padded
        # to twelve floats and never 16-byte aligned).
        {"name": "ragged_47k_d10", "kind": "build", **_event(47_311, 10, 0.1, 256, 5, 18, 0.8, 0.15)},
        # The benchmark's size: 120,000 hits in 8 coordinates, steps back to back.
        {"name": "single_120k", "kind": "step", **_event(120_000, 8, 0.1, 256, 5, 18, 0.8, 0.15), "events": 1},
        # The nearest 8 within the radius (a graph of bounded degree) on the same event.
        {"name": "nearest8_120k", "kind": "step", **_event(120_000, 8, 0.1, 8, 5, 18, 0.8, 0.15), "events": 1},
        # The large event of the test suite: 300,000 hits in 12 coordinates.
        {"name": "high_300k_d12", "kind": "step", **_event(300_000, 12, 0.12, 512, 6, 20, 1.2, 0.20), "events": 1},
        # A wide embedding: 32 coordinates.
        {"name": "wide_60k_d32", "kind": "build", **_event(60_000, 32, 0.1, 256, 5, 18, 0.8, 0.15)},
        # A batch for a training or re-processing job: 64 events of 20k to 150k hits.
        {"name": "batch_64", "kind": "step", **_event(20_000, 8, 0.1, 256, 5, 18, 0.8, 0.15), "n_hi": 150_000,
         "events": 64},
        # What the server launches at once: six requests of 10k to 300k hits.
        {"name": "served_6", "kind": "served", **_event(10_000, 8, 0.1, 256, 5, 18, 0.8, 0.15), "n_hi": 300_000,
         "events": 6},
        # A loose embedding or a wide radius: some 45 neighbours per hit, as early in a
        # metric-learning training or when the graph is to miss no true edge.
        {"name": "dense_60k", "kind": "build", **_event(60_000, 8, 0.1, 256, 20, 80, 0.8, 0.15), "per_point": 64},
        # The same with crowded neighbourhoods and the cap binding: the nearest 32.
        {"name": "dense_nearest32_20k", "kind": "build", **_event(20_000, 8, 0.1, 32, 40, 150, 0.8, 0.15),
         "per_point": 32},
        # Track labels of the single event's graph, every edge kept, in the pipeline.
        {"name": "label_120k", "kind": "label_step", **_event(120_000, 8, 0.1, 256, 5, 18, 0.8, 0.15)},
        # Track labels of a large event's graph with the edge filter's scores cut at 0.5.
        {"name": "label_scored_300k", "kind": "label", **_event(300_000, 8, 0.1, 256, 5, 18, 0.8, 0.15),
         "threshold": 0.5},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges; rng is a random.Random."""
    what = rng.choice(("build", "build", "step", "nearest", "wide", "batch", "batch", "served", "dense", "dense",
                       "dense_nearest", "label", "label_step"))
    noise = round(rng.uniform(0.05, 0.25), 3)
    spread = round(rng.uniform(0.7, 1.1), 3)
    lo, hi = rng.choice(((5, 18), (6, 20), (8, 15)))
    K = rng.choice((64, 256, 512))
    if what == "build":
        d = rng.choice((3, 5, 6, 7, 8, 8, 10, 12))
        return {"kind": "build", **_event(_log_int(rng, 1_000, 200_000), d, 0.03 if d < 5 else 0.1, K, lo, hi, spread,
                                          noise)}
    if what == "step":
        return {"kind": "step", **_event(_log_int(rng, 10_000, 300_000), rng.choice((6, 8, 8, 12)), 0.1, K, lo, hi,
                                         spread, noise), "events": 1}
    if what == "nearest":
        return {"kind": "step", **_event(_log_int(rng, 5_000, 200_000), 8, 0.1, rng.randint(4, 15), lo, hi, spread,
                                         noise), "events": 1}
    if what == "wide":
        return {"kind": "build", **_event(_log_int(rng, 2_000, 60_000), rng.choice((16, 20, 24, 32)), 0.1, K, lo, hi,
                                          spread, noise)}
    if what in ("batch", "served"):
        count = _log_int(rng, 2, 64) if what == "batch" else rng.randint(2, 8)
        top = 150_000 if what == "batch" else 300_000
        least = _log_int(rng, 2_000, 40_000)
        most = min(top, least * rng.randint(2, 8))
        return {"kind": "step" if what == "batch" else "served",
                **_event(least, 8, 0.1, K, lo, hi, spread, noise), "n_hi": most, "events": count}
    if what == "dense":
        size = rng.randint(20, 80)
        return {"kind": "build", **_event(_log_int(rng, 3_000, 50_000), rng.choice((6, 8, 12)), 0.1, 256, size // 2,
                                          size, spread, noise), "per_point": 80}
    if what == "dense_nearest":
        size = rng.randint(30, 150)
        K = rng.choice((8, 16, 24, 32, 48))
        return {"kind": "build", **_event(_log_int(rng, 3_000, 20_000), 8, 0.1, K, size // 2, size, spread, noise),
                "per_point": 48}
    case = {"kind": what, **_event(_log_int(rng, 5_000, 300_000), 8, 0.1, K, lo, hi, spread, noise)}
    if rng.random() < 0.5:
        case["threshold"] = round(rng.uniform(0.3, 0.7), 3)
    return case


def _sizes(case):
    """Hits of each event of the case (part of its shape: the same for every seed)."""
    if case.get("events", 1) == 1:
        return [case["n"]]
    rng = np.random.Generator(np.random.PCG64(99))
    lo, hi = case["n"], case["n_hi"]
    if case["kind"] == "served":  # requests: log-uniform
        return [int(round(v)) for v in np.exp(rng.uniform(math.log(lo), math.log(hi), size=case["events"]))]
    return [int(v) for v in rng.integers(lo, hi + 1, size=case["events"])]


def _generate(case, n, seed):
    """(points float32 [n, d], cluster of each point) as the repository draws its events."""
    lo, hi, d = case["size_lo"], case["size_hi"], case["d"]
    quota = n - int(round(case["noise"] * n))
    clusters = max(1, -(-quota // hi), min(quota // lo, round(quota / (0.5 * (lo + hi)))))
    spec = events.EventSpec(n=n, d=d, n_clusters=clusters, size_lo=min(lo, quota // clusters), size_hi=hi,
                            sigma=case["spread"] * case["r"] / math.sqrt(2 * d), noise_frac=case["noise"],
                            r=case["r"], K=case["K"], seed=seed)
    return events.generate(spec)


@dataclasses.dataclass
class State:
    case: dict
    points: object = None       # the event's (or the batch's) points
    parts: object = None        # served: one tensor per request
    step: object = None         # the kept call
    workspace: object = None
    src: object = None
    dst: object = None
    ranges: object = None       # edge ranges and status
    scores: object = None
    labels: object = None
    result: object = None


def prepare(case, seed):
    sizes = _sizes(case)
    drawn = [_generate(case, n, seed * 1009 + 31 * e) for e, n in enumerate(sizes)]
    st = State(case)
    K, r, d = case["K"], case["r"], case["d"]
    offsets = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    rows = int(offsets[-1])
    if case["kind"] in ("build", "step", "served"):
        st.workspace = torch.empty(frnn.batch_workspace_bytes(offsets, d), dtype=torch.uint8, device=DEVICE)
        # Room for 16 edges per hit, as frnn.build's default, or more for a denser graph;
        # entries past the edges are never written.
        capacity = case.get("per_point", 16) * rows
        st.src = torch.zeros(capacity, dtype=torch.int64, device=DEVICE)
        st.dst = torch.zeros(capacity, dtype=torch.int64, device=DEVICE)
        st.ranges = torch.zeros(len(sizes) + 2, dtype=torch.int64, device=DEVICE)
    if case["kind"] == "build":
        st.points = torch.from_numpy(drawn[0][0]).to(DEVICE)
    elif case["kind"] == "step":
        st.points = torch.from_numpy(np.concatenate([X for X, _ in drawn])).to(DEVICE)
        st.step = frnn.AsyncBatch(st.points, offsets, r, K, st.workspace, st.src, st.dst)
    elif case["kind"] == "served":
        st.parts = [torch.from_numpy(X).to(DEVICE) for X, _ in drawn]
    else:  # a graph to label
        edges = frnn.build(torch.from_numpy(drawn[0][0]).to(DEVICE), r, K)
        st.src, st.dst = edges[0].clone(), edges[1].clone()
        if "threshold" in case:
            # Filter scores: most edges inside a cluster high, most others low.
            track = torch.from_numpy(drawn[0][1]).to(DEVICE)
            gen = torch.Generator(device=DEVICE)
            gen.manual_seed(seed)
            u = torch.rand(st.src.numel(), generator=gen, device=DEVICE)
            true = (track[st.src] == track[st.dst]) & (track[st.src] >= 0)
            st.scores = torch.where(true, 1.0 - 0.6 * u * u, 0.7 * u).contiguous()
        if case["kind"] == "label_step":
            st.workspace = torch.empty(frnn.components_workspace_bytes(rows), dtype=torch.uint8, device=DEVICE)
            st.labels = torch.empty(rows, dtype=torch.int64, device=DEVICE)
            st.result = torch.zeros(2, dtype=torch.int64, device=DEVICE)
    return st


def run(state):
    case = state.case
    kind = case["kind"]
    if kind == "build":
        status, count = frnn.build_into(state.points, case["r"], case["K"], state.workspace, state.src, state.dst)
        if status != frnn.FRNN_OK:
            raise frnn.FrnnError(status, frnn.status_string(status))
        return state.src, state.dst, count
    if kind == "step":
        status = state.step(state.ranges)
        if status != frnn.FRNN_OK:
            raise frnn.FrnnError(status, frnn.status_string(status))
        return state.src, state.dst, state.ranges
    if kind == "served":
        status = frnn.build_events_async(state.parts, case["r"], case["K"], state.workspace, state.src, state.dst,
                                         state.ranges)
        if status != frnn.FRNN_OK:
            raise frnn.FrnnError(status, frnn.status_string(status))
        return state.src, state.dst, state.ranges
    threshold = case.get("threshold", 0.0)
    if kind == "label":
        return frnn.components(state.src, state.dst, case["n"], state.scores, threshold)
    status = frnn.components_async(state.src, state.dst, case["n"], state.workspace, state.labels, state.result,
                                   state.scores, threshold)
    if status != frnn.FRNN_OK:
        raise frnn.FrnnError(status, frnn.status_string(status))
    return state.labels, state.result


def _chi2_cdf(x, k):
    """P(chi-square with k degrees of freedom < x), by the series of the lower gamma function."""
    a, h = 0.5 * k, 0.5 * x
    term = total = 1.0 / a
    for i in range(1, 500):
        term *= h / (a + i)
        total += term
    return min(1.0, total * math.exp(a * math.log(h) - h - math.lgamma(a)))


def _expected_edges(case, n):
    """Expected edges of an event: pairs of one cluster closer than r, at most K per hit."""
    lo, hi = case["size_lo"], case["size_hi"]
    mean = 0.5 * (lo + hi)
    var = ((hi - lo + 1) ** 2 - 1) / 12.0
    others = mean + var / mean - 1.0  # other points of a point's cluster
    near = others * _chi2_cdf(case["d"] / case["spread"] ** 2, case["d"])
    return n * (1.0 - case["noise"]) * min(near, case["K"])


def work(case):
    """Points read once and edges written once (or edges read and labels written);
    one distance per edge."""
    count = case.get("events", 1)
    n = case["n"]
    if count > 1:
        lo, hi = case["n"], case["n_hi"]
        n = 0.5 * (lo + hi) if case["kind"] == "step" or hi == lo else (hi - lo) / math.log(hi / lo)
    rows, edges = count * n, count * _expected_edges(case, n)
    if case["kind"] in ("label", "label_step"):
        return {"bytes": edges * (20 if "threshold" in case else 16) + 8 * rows, "flops": 0}
    return {"bytes": 4 * rows * case["d"] + 16 * edges, "flops": edges * (3 * case["d"] + 1)}


def exact(case, seed):
    """Edges, ranges and labels are whole numbers: compared as they are."""
    return None
