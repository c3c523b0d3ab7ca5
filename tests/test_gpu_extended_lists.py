"""Lists of 17 to 32 neighbours: kept by the search beside its 16-entry lists.

Clumps put lists at both edges of that range; a batch of queries with more such hits
than it keeps, and an input with more such lists than there are blocks for, send them to
the collection in the placement pass instead.  Caps in the range select again.  Edges
against the CPU oracle, and the count of lists of more than 16.
"""

import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2202_06929_amd import events, frnn

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def check(X, K, sizes=None):
    print(f"n={len(X)} d={X.shape[1]} K={K}", flush=True)
    got, st = frnn.build(torch.from_numpy(X).to(DEV), 0.1, K, return_stats=True)
    want = oracle.frnn_grid(X, 0.1, K)
    got = got.cpu().numpy()
    assert got.shape == want.shape and np.array_equal(got, want)
    if sizes is not None:
        assert st["overflow_queries"] == sum(m for m in sizes if m - 1 > 16)


@pytest.mark.parametrize("d", [3, 8, 16, 48, 64])
@pytest.mark.parametrize("K", [4096, 33, 32, 31, 17, 16])
def test_lists_at_the_edges(d, K):
    sizes = [16, 17, 18, 19, 25, 32, 33, 34, 35] * 2
    check(events.tight_clumps(sizes, d, 0.1, seed=d, noise=400), K, sizes)


@pytest.mark.parametrize("size", [18, 24, 33])
def test_more_lists_than_a_batch_or_the_extension_holds(size):
    # Every query has such a list: 8 n bytes of extension hold one for an eighth of them,
    # and a batch of queries in one cell spills more than it keeps.
    sizes = [size] * 3000
    check(events.tight_clumps(sizes, 8, 0.1, seed=size), 256, sizes)


def test_spread_in_an_ordinary_event_and_a_batch():
    evs = [events.generate(events.EventSpec(n=n, d=8, n_clusters=max(1, n // 13), size_lo=5, size_hi=22, sigma=0.02,
                                            noise_frac=0.1, r=0.1, K=256, seed=n))[0] for n in (900, 20_000, 7_000)]
    offsets = np.concatenate([[0], np.cumsum([len(x) for x in evs])]).astype(np.int64)
    edges, eo, st = frnn.build_batch(torch.from_numpy(np.concatenate(evs)).to(DEV), offsets, 0.1, 256,
                                     return_stats=True)
    edges = edges.cpu().numpy()
    assert st["overflow_queries"] > 500
    for e, X in enumerate(evs):
        assert np.array_equal(edges[:, eo[e]:eo[e + 1]], oracle.frnn_grid(X, 0.1, 256)), e
