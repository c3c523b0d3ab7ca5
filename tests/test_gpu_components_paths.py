"""Labeling of chains inside and across waves, and of edge lists off the builder's order.

A lane of the union-find pass whose smaller root is the larger root of the joining lane
before or after it hooks under the end of their chain in the wave: paths with lengths
around 64 edges, in rising, falling and turning order, with edges dropped, repeated and
pointing either way, cross every edge of that rule.  Labels against the CPU oracle, byte
for byte.  Two times are compared within one process: edges that all join one large tree
against edges inside small ones (19 times as long when every edge swapped without looking,
4 times now), and a path of 200 against one of 20 (1.8 times as long with 256 edges a wave).
"""

import numpy as np
import pytest
import torch

from oracle import components as cc_oracle
from paper_2202_06929_amd import frnn

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def to(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to(DEV)


def check(src, dst, n, scores=None):
    src, dst = np.asarray(src, dtype=np.int64), np.asarray(dst, dtype=np.int64)
    got, count = frnn.components(to(src), to(dst), n, None if scores is None else to(scores), 0.5)
    want = cc_oracle.labels(src, dst, n, scores, 0.5)
    assert np.array_equal(got.cpu().numpy(), want)
    assert count == len(np.unique(want))


@pytest.mark.parametrize("n", [2, 3, 63, 64, 65, 66, 127, 129, 257, 5000])
@pytest.mark.parametrize("order", ["rising", "falling", "turning", "inside_out", "both_ways", "repeated", "twos"])
def test_paths_around_a_wave(n, order):
    print(f"path {order} n={n}", flush=True)
    rng = np.random.Generator(np.random.PCG64(n))
    a = np.arange(n - 1)
    if order == "falling":
        a = a[::-1]
    elif order == "turning":  # up, then down, in runs of 20
        a = np.concatenate([r if k % 2 else r[::-1] for k, r in enumerate(np.array_split(a, n // 20 + 1))])
    elif order == "inside_out":  # neighbouring lanes come from both ends
        a = np.stack([a, a[::-1]], axis=1).ravel()[: n - 1]
    elif order == "repeated":
        a = np.repeat(a, rng.integers(1, 4, size=n - 1))
    elif order == "twos":  # every second edge first: chains of two trees a lane apart
        a = np.concatenate([a[::2], a[1::2]])
    src, dst = a.copy(), a + 1
    if order == "both_ways":
        flip = rng.random(a.size) < 0.5
        src, dst = np.where(flip, dst, src), np.where(flip, src, dst)
    check(src, dst, n)
    check(src, dst, n, np.where(rng.random(a.size) < 0.05, 0.2, 0.9).astype(np.float32))


@pytest.mark.parametrize("seed", range(6))
def test_paths_among_other_edges(seed):
    # Many short paths over shuffled names, their edges in runs, loops and random edges between.
    rng = np.random.Generator(np.random.PCG64(seed))
    n = 6000
    name = rng.permutation(n) if seed % 2 else np.arange(n)
    src, dst = [], []
    for at in range(0, n - 70, 70):
        r = np.arange(at, at + int(rng.integers(2, 70)))
        r = r[::-1] if rng.random() < 0.5 else r
        src += [name[r[:-1]], name[rng.integers(0, n, 2)], name[[at]]]
        dst += [name[r[1:]], name[rng.integers(0, n, 2)], name[[at]]]
    src, dst = np.concatenate(src), np.concatenate(dst)
    check(src, dst, n, np.where(rng.random(src.size) < 0.1, 0.2, 0.9).astype(np.float32))


def call_us(src, dst, n):
    """Smallest of five means over ten calls, enqueued in a row."""
    src, dst = to(src), to(dst)
    for _ in range(3):
        frnn.components(src, dst, n)
    begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    times = []
    for _ in range(5):
        begin.record()
        for _ in range(10):
            frnn.components(src, dst, n)
        end.record()
        torch.cuda.synchronize()
        times.append(begin.elapsed_time(end) * 100.0)
    return min(times)


def test_edges_that_join_the_same_trees_do_not_wait_for_each_other():
    # 1M edges sorted by source, to a random vertex or one of the source's ten.
    rng = np.random.Generator(np.random.PCG64(3))
    n = 200_000
    src = np.sort(rng.integers(0, n, 10**6))
    near = call_us(src, src // 10 * 10 + rng.integers(0, 10, 10**6), n)
    far = call_us(src, rng.integers(0, n, 10**6), n)
    print(f"1M edges: near {near:.1f} us, far {far:.1f} us", flush=True)
    assert far <= 12 * near


def test_a_path_of_200_takes_no_longer_than_one_of_20():
    a = np.arange(199)
    short, long = call_us(a[:19], a[:19] + 1, 20), call_us(a, a + 1, 200)
    print(f"path of 20: {short:.1f} us, of 200 {long:.1f} us", flush=True)
    assert long <= 1.3 * short
