"""The search's batches of queries: cells at the edges of a batch, pairs of cells, events.

A wave takes its queries in batches of at most 32 (16 when K is below the list size)
that end between cells, builds the runs of two cells at once when a cell has at most 32
of them (49 with three axes and cells of a third of r), and never crosses an event.
Clumps put cells of 15, 16, 17, 31, 32, 33, 63, 64 and 65 queries side by side, alone and
as small events of a batch, for every run count, against the CPU oracle.
"""

import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2202_06929_amd import events, frnn

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
SIZES = [1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 2]
CONFIGS = [None, frnn.Config(axes=3), frnn.Config(axes=3, cell_div=2), frnn.Config(axes=3, cell_div=3)]


@pytest.mark.parametrize("K", [256, 16, 15, 4])
@pytest.mark.parametrize("config", CONFIGS, ids=["axes4", "axes3", "div2", "div3"])
def test_cells_at_the_edges_of_a_batch(config, K):
    X = events.tight_clumps(SIZES, 8, 0.1, seed=K, noise=40)
    evs = [X] + [events.tight_clumps([m], 8, 0.1, seed=m) for m in SIZES] + [X[:50]]
    offsets = np.concatenate([[0], np.cumsum([len(e) for e in evs])]).astype(np.int64)
    print(f"{len(evs)} events, {offsets[-1]} rows, K={K}, config={config}", flush=True)
    edges, eo = frnn.build_batch(torch.from_numpy(np.concatenate(evs)).to(DEV), offsets, 0.1, K, config)
    edges = edges.cpu().numpy()
    for e, P in enumerate(evs):
        assert np.array_equal(edges[:, eo[e]:eo[e + 1]], oracle.frnn_grid(P, 0.1, K)), e


@pytest.mark.parametrize("d", [4, 12, 16, 24, 32, 48, 64])
def test_every_row_width(d):
    for K in (256, 8):
        X = events.tight_clumps(SIZES * 3, d, 0.1, seed=d, noise=100)
        print(f"n={len(X)} d={d} K={K}", flush=True)
        got = frnn.build(torch.from_numpy(X).to(DEV), 0.1, K).cpu().numpy()
        assert np.array_equal(got, oracle.frnn_grid(X, 0.1, K))
