"""The labeling's min-neighbour pass on edge lists in and out of order.

Where targets ascend within every source (the graph builder's lists), a source's
smallest kept target is its first; elsewhere a segmented minimum finds it.  Runs of one
source of 1 to 300 edges cross the 64-edge groups and the 256-edge share of a wave, with
scores that leave out a run's first, middle or all edges, ascending, descending and
shuffled.  Labels against the CPU oracle.
"""

import numpy as np
import pytest
import torch

from oracle import components as cc_oracle
from paper_2202_06929_amd import frnn

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("order", ["ascending", "descending", "shuffled", "one_swap"])
@pytest.mark.parametrize("scored", [False, True])
@pytest.mark.parametrize("lengths", [(1, 2, 3), (63, 64, 65), (7, 255, 256, 257, 300)])
def test_runs_in_every_order(order, scored, lengths):
    n = 4000
    rng = np.random.Generator(np.random.PCG64(len(order) + sum(lengths)))
    src, dst = [], []
    for k, v in enumerate(np.sort(rng.choice(n, size=60, replace=False))):
        m = lengths[k % len(lengths)]
        t = np.sort(rng.choice(np.arange(max(0, v - 400), min(n, v + 400)), size=m, replace=False))
        if order == "descending":
            t = t[::-1]
        elif order == "shuffled":
            t = rng.permutation(t)
        elif order == "one_swap" and m > 1:
            t[[0, 1]] = t[[1, 0]]
        src.append(np.full(m, v))
        dst.append(t)
    src, dst = np.concatenate(src).astype(np.int64), np.concatenate(dst).astype(np.int64)
    scores = rng.uniform(0, 1, size=src.size).astype(np.float32) if scored else None
    print(f"{order} scored={scored} lengths={lengths} edges={src.size}", flush=True)
    to = lambda x: None if x is None else torch.from_numpy(np.ascontiguousarray(x)).to(DEV)  # noqa: E731
    got, count = frnn.components(to(src), to(dst), n, to(scores), 0.7)
    want = cc_oracle.labels(src, dst, n, scores, 0.7)
    assert np.array_equal(got.cpu().numpy(), want)
    assert count == len(np.unique(want))
