"""Batches whose largest event is far above the mean are binned in a one-dimensional grid:
every event's edges must be those of the event alone by the oracle (whole numbers)."""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2202_06929_amd import frnn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [[40_000] + [1] * 20, [0] * 9 + [5_000] + [0] * 9, [50, 0, 70_001] + [51] * 40,
                                   [1] * 60 + [9_217, 1_024, 1_025, 0], [530_000] + [3] * 30])
def test_edges_of_every_event(sizes):
    rng = np.random.Generator(np.random.PCG64(len(sizes)))
    offsets = np.concatenate([[0], np.cumsum(sizes)])
    assert max(sizes) * len(sizes) > 8 * offsets[-1]
    X = rng.uniform(-1, 1, size=(offsets[-1], 4)).astype(np.float32)
    edges, eo = frnn.build_batch(torch.from_numpy(X).cuda(), offsets, 0.05, 64)
    edges = edges.cpu().numpy()
    for e in range(len(sizes)):
        got = edges[:, eo[e]:eo[e + 1]]
        if sizes[e] == 0:
            assert got.shape[1] == 0
            continue
        s, t = oracle.frnn_grid(X[offsets[e]:offsets[e + 1]], 0.05, 64)[:2]
        assert np.array_equal(got[0], s) and np.array_equal(got[1], t), e
