"""Binning of events whose points crowd into few tiles.

A tile of 4,096 points and more (8,192 in calls beyond 2^19 rows) gets workgroups beside its
own, one for every 2,048 of them (or more, where the event's tiles leave few blocks over);
its points are counted by the shares of 1,024 rows that hold enough of them.  Events with
narrow binned axes beside an outlier put all their points into one tile, one cell or a few:
sizes lie around the first count, at whole and broken parts and with shares of 2,048 rows;
batches mix them with empty, small and spread events, in both grids.  Edges against the CPU
oracle, byte for byte (it bins the leading coordinates, which are spread).  The rows' stage
of a crowded event is timed against a spread one's.
"""

import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2202_06929_amd import frnn

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def crowded(n, d, thin, far, seed, width=1e-3):
    """n points within `width` of 0 along the last `thin` coordinates, one of them at `far`."""
    rng = np.random.Generator(np.random.PCG64(seed))
    X = rng.uniform(-1, 1, size=(n, d))
    X[:, d - thin:] *= width
    if n:
        X[rng.integers(n), d - thin:] = far
    return X.astype(np.float32)


def check(X, r, K, **config):
    print(f"n={len(X)} d={X.shape[1]} r={r} K={K} {config}", flush=True)
    got = frnn.build(torch.from_numpy(X).to(DEV), r, K, frnn.Config(**config) if config else None).cpu().numpy()
    want = oracle.frnn_grid(X, r, K)
    assert got.shape == want.shape and np.array_equal(got, want)


@pytest.mark.parametrize("n", [4095, 4096, 4097, 4608, 6143, 8192, 20_001, 65_536])
@pytest.mark.parametrize("d,thin", [(3, 2), (3, 3), (5, 2), (8, 4), (12, 3), (20, 4)])
def test_all_points_in_few_tiles(n, d, thin):
    r = {3: 0.004, 5: 0.06, 8: 0.25, 12: 0.6, 20: 1.2}[d]
    if d >= 12 and n > 30_000:
        pytest.skip("the oracle tests every pair there")
    if thin == d:  # a line, and the far point along all three axes
        X = crowded(n, d, thin, 3.0, n + d)
        X[:, 0] = np.random.Generator(np.random.PCG64(1)).permutation(n) * np.float32(1e-5)
        check(X, 5e-5, 64)
    else:
        check(crowded(n, d, thin, 20 * r, n + d), r, 64)


@pytest.mark.parametrize("config", [dict(axes=3), dict(axes=3, cell_div=2), dict(dims=(2, 5, 0, 7))])
def test_other_grids(config):
    X = crowded(30_000, 8, 3, 4.0, 7)
    X[:, 0] *= 0.01
    check(X, 0.2, 12, **config)


@pytest.mark.parametrize("n", [20_000, 60_000])
def test_few_blocks_over(n):
    # Cells that divide into nearly as many tiles as there are blocks, all points in one row of them.
    r = np.float32(0.01)
    c = r * np.float32(1.0009765625)
    rng = np.random.Generator(np.random.PCG64(n))
    X = rng.uniform(0, 1e-5, size=(n, 3))
    wide = 100 if n == 20_000 else 170  # 100 x 98 and 170 x 172 cells: 77 of 78 and 229 of 234 tiles
    high = {100: 98, 170: 172}[wide]
    X[:, 0] = rng.uniform(0, (wide - 0.5) * c, size=n)
    X[:2, 0] = 0, (wide - 0.5) * c
    X[5, 1] = (high - 0.5) * c
    X = X.astype(np.float32)
    _, stats = frnn.build(torch.from_numpy(X).to(DEV), float(r), 64, return_stats=True)
    assert stats["grid"][:3] == [wide, high, 1], stats["grid"]
    check(X, float(r), 64)


def test_shares_of_2048_rows():
    check(crowded(600_001, 3, 1, 0.3, 3, width=1e-5), 0.0008, 64)


@pytest.mark.parametrize("others", [[30_000, 0, 5, 1024], [3] * 40, [0, 9000, 9000]])
def test_batches(others):
    evs = [crowded(m, 6, 3, 2.0, m) for m in others[:2]] + [crowded(40_000, 6, 3, 4.0, 1)]
    rng = np.random.Generator(np.random.PCG64(2))
    evs += [rng.uniform(-1, 1, size=(m, 6)).astype(np.float32) for m in others[2:]] + [crowded(10_000, 6, 4, 2.0, 4)]
    offsets = np.concatenate([[0], np.cumsum([len(X) for X in evs])]).astype(np.int64)
    print(f"batch {[len(X) for X in evs]}", flush=True)
    edges, eo = frnn.build_batch(torch.from_numpy(np.concatenate(evs)).to(DEV), offsets, 0.1, 64)
    edges = edges.cpu().numpy()
    for e, X in enumerate(evs):
        assert np.array_equal(edges[:, eo[e]:eo[e + 1]], oracle.frnn_grid(X, 0.1, 64)), e


def test_one_workspace_for_events_in_turn():
    n, d, r, K = 30_000, 8, 0.25, 64
    rng = np.random.Generator(np.random.PCG64(4))
    evs = [crowded(n, d, 4, 5.0, 1), rng.uniform(-1, 1, size=(n, d)).astype(np.float32), crowded(n, d, 3, 5.0, 2),
           crowded(n - 9_000, d, 4, 5.0, 3), crowded(n, d, 4, 5.0, 1)]
    ws = torch.full((frnn.workspace_bytes(n, d),), 0xA5, dtype=torch.uint8, device=DEV)
    out = torch.empty((2, K * n), dtype=torch.int64, device=DEV)
    for k, X in enumerate(evs):
        print(f"event {k}: n={len(X)}", flush=True)
        st, E = frnn.build_into(torch.from_numpy(X).to(DEV), r, K, ws, out[0], out[1])
        assert st == frnn.FRNN_OK
        assert np.array_equal(out[:, :E].cpu().numpy(), oracle.frnn_grid(X, r, K)), k


def stage_us(X, r, stage):
    pts = torch.from_numpy(X).to(DEV)
    n, d = X.shape
    ws = torch.empty(frnn.workspace_bytes(n, d), dtype=torch.uint8, device=DEV)
    out = torch.empty((2, 64 * n), dtype=torch.int64, device=DEV)
    times = []
    for _ in range(7):
        stats = frnn.FrnnStats()
        st, _ = frnn.build_into(pts, r, 64, ws, out[0], out[1], frnn.Config(timing=True), stats)
        assert st == frnn.FRNN_OK
        times.append(stats.as_dict()["stage_ms"][stage] * 1e3)
    return sorted(times)[3]


def test_a_crowded_tile_does_not_wait_for_one_workgroup():
    # One workgroup took 48 times as long for 120,000 points as 500 tiles, the parts 5 times:
    # the bound lies half way in ratio.
    rng = np.random.Generator(np.random.PCG64(9))
    spread = stage_us(rng.uniform(-1, 1, size=(120_000, 8)).astype(np.float32), 0.1, "scatter")
    one = stage_us(crowded(120_000, 8, 2, 2.0, 9), 0.1, "scatter")
    print(f"rows into cell order: {spread:.1f} us spread, {one:.1f} us crowded", flush=True)
    assert one <= 15 * spread
