"""Lists too long for a wave of the placement pass: sizes around the chunks of their sort
and around what is kept in LDS, below the cap and cut by it, against the oracle (whole
numbers: the edges must be the same)."""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2202_06929_amd import frnn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hits,K", [(512, 4096), (513, 4096), (1024, 4096), (1025, 4096), (2047, 4096), (2049, 4096),
                                    (4095, 4096), (4096, 4096), (4097, 4096), (2048, 2048), (2049, 2048),
                                    (1100, 600), (2100, 600), (4200, 1), (600, 512), (600, 513)])
@pytest.mark.parametrize("d", [8, 16])
def test_one_clump(hits, K, d):
    rng = np.random.Generator(np.random.PCG64(hits + K))
    clump = rng.normal(0, 0.002, size=(hits + 1, d))
    X = np.concatenate([clump, rng.uniform(1, 2, size=(300, d))]).astype(np.float32)
    rng.shuffle(X)
    got = frnn.build(torch.from_numpy(X).cuda(), 0.1, K).cpu().numpy()
    s, t = oracle.frnn_grid(X, 0.1, K)[:2]
    assert np.array_equal(got[0], s) and np.array_equal(got[1], t)
