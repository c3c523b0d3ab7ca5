"""Long lists at the edges of the placement pass's own collection.

A wave collects a list of up to 512 hits (in 1, 2, 4 or 8 registers per lane)
and a workgroup a larger one; with the cap binding, the nearest K are selected bit by
bit, ties in D by id.  Clump sizes put lists at both sides of each of those widths;
copies of one point make every distance of a list equal.  Edges against the CPU
oracle, byte for byte.  The event sizes of the last test lie around the 16,384 rows
whose kept counts one workgroup sums.
"""

import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2202_06929_amd import events, frnn

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
SIZES = [18, 65, 66, 129, 130, 257, 258, 513, 514, 1025, 1026]


def check(X, r, K):
    print(f"n={len(X)} d={X.shape[1]} K={K}", flush=True)
    got = frnn.build(torch.from_numpy(X).to(DEV), r, K)
    torch.cuda.synchronize()
    want = oracle.frnn_grid(X, r, K)
    got = got.cpu().numpy()
    assert got.shape == want.shape, (got.shape, want.shape)
    assert np.array_equal(got, want)


@pytest.mark.parametrize("d,K", [(8, 4096), (8, 1024), (8, 257), (8, 128), (8, 64), (8, 17), (8, 1), (3, 65), (64, 256)])
def test_lists_at_each_collection_width(d, K):
    check(events.tight_clumps(SIZES, d, 0.1, seed=17 + d, noise=200), 0.1, K)


@pytest.mark.parametrize("copies,K", [(40, 20), (200, 64), (1025, 1000), (1100, 70)])
def test_equal_distances_are_kept_by_id(copies, K):
    rng = np.random.Generator(np.random.PCG64(copies))
    base = rng.uniform(-1, 1, size=(1, 8))
    X = np.concatenate([np.repeat(base, copies, axis=0), base + rng.normal(0, 0.01, size=(30, 8)),
                        rng.uniform(-1, 1, size=(100, 8))])
    check(X[rng.permutation(len(X))].astype(np.float32), 0.1, K)


@pytest.mark.parametrize("n", [16_383, 16_384, 16_385, 32_769])
def test_rows_around_a_group_of_tiles(n):
    sizes = [20, 40] * (n // 100)
    check(events.tight_clumps(sizes, 5, 0.1, seed=n, noise=n - sum(sizes)), 0.1, 25)
