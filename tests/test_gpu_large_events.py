"""Calls whose largest event has more than 1,048,576 rows.

They are binned by atomics on a histogram instead of through tiles, and only they are: the
scan that cuts the search's pieces, the scatter into whole and split rows, from float4 and
from single floats, the histogram's memory as the search's extension, and the queues of
long lists run here behind that binning.  Clumps whose points all lie within r of one
another give lists of every kind (up to 16, 17 to 32, longer, above 512 hits), beside
isolated points.  An event is two halves a long way apart along coordinate 0, so its edges
are those of the halves, byte for byte; the halves go through the tiles, which are
compared with the CPU oracle at every size they take (one event of this size is, too).
"""

import pytest
import torch

from paper_2202_06929_amd import frnn

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
N = (1 << 20) + 1
HALF = 1 << 19
R = 0.02


def clumps(n, d, seed):
    """n points, most alone, the others in clumps within balls of R / 2, shuffled."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    sizes = [1200, 700, 513] + [1, 2, 3, 12, 17, 20, 32, 33, 120] * (n // 2000)
    sizes = torch.tensor(sizes + [1] * (n - sum(sizes)), device=DEV)
    which = torch.repeat_interleave(torch.arange(len(sizes), device=DEV), sizes)[:n]
    at = (torch.rand((len(sizes), d), generator=g, device=DEV) * 2 - 1)[which]
    step = torch.randn((n, d), generator=g, device=DEV)
    step *= 0.49 * R * torch.rand((n, 1), generator=g, device=DEV) / step.norm(dim=1, keepdim=True)
    return (at + step)[torch.randperm(n, generator=g, device=DEV)].contiguous()


def event(d, seed):
    """N points: HALF of them, then the others 10 apart; and the two parts."""
    a, b = clumps(HALF, d, seed), clumps(N - HALF, d, seed + 1)
    b[:, 0] += 10.0
    return torch.cat([a, b]), a, b


def edges_of(a, b, K, config=None):
    ea, eb = frnn.build(a, R, K, config), frnn.build(b, R, K, config)
    return torch.cat([ea, eb + len(a)], dim=1)


@pytest.mark.parametrize("d,K", [(3, 8), (4, 64), (5, 4096), (8, 16), (10, 64), (12, 8), (12, 256), (16, 64), (20, 64),
                                 (32, 24), (48, 8), (64, 64)])
def test_every_row_width_and_cap(d, K):
    X, a, b = event(d, d + K)
    print(f"n={N} d={d} K={K}", flush=True)
    got = frnn.build(X, R, K)
    assert torch.equal(got, edges_of(a, b, K))
    kept = torch.bincount(got[0], minlength=N)
    for lo, hi in ((1, 16), (17, 32), (33, 512), (513, 4096)):
        if d > 3 and K >= hi:
            assert ((kept >= lo) & (kept <= hi)).any(), (lo, hi)


@pytest.mark.parametrize("config", [frnn.Config(axes=3), frnn.Config(axes=3, cell_div=2),
                                    frnn.Config(axes=3, cell_div=3), frnn.Config(dims=(6, 0, 3, 1), grid_mult=1)])
def test_other_grids(config):
    X, a, b = event(7, 3)
    print(f"n={N} d=7 {config}", flush=True)
    assert torch.equal(frnn.build(X, R, 64, config), edges_of(a, b, 64))


def test_an_unaligned_first_row():
    X, a, b = event(8, 5)
    off = torch.empty(N * 8 + 1, dtype=torch.float32, device=DEV)[1:].view(N, 8)
    off.copy_(X)
    print("rows off 16 bytes", flush=True)
    assert torch.equal(frnn.build(off, R, 64), edges_of(a, b, 64))


@pytest.mark.parametrize("sizes", [[0, 5, N, 0, 3000, 1, 0], [40_000, N], [N] + [7] * 50, [N, N]])
@pytest.mark.parametrize("d,K", [(6, 64), (12, 8)])
def test_batches_beside_small_and_empty_events(sizes, d, K):
    print(f"batch {sizes[:8]} d={d} K={K}", flush=True)
    X, a, b = event(d, 9)
    evs = [X if m == N else clumps(m, d, m) if m >= 3000 else
           torch.rand((m, d), generator=torch.Generator(device=DEV).manual_seed(m), device=DEV) * R for m in sizes]
    offsets = [0]
    for m in sizes:
        offsets.append(offsets[-1] + m)
    edges, eo = frnn.build_batch(torch.cat(evs), offsets, R, K)
    for e, points in enumerate(evs):
        got = edges[:, int(eo[e]):int(eo[e + 1])]
        if len(points) == 0:
            assert got.shape[1] == 0
        else:
            want = edges_of(a, b, K) if len(points) == N else frnn.build(points, R, K)
            assert torch.equal(got, want), e


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -float("inf")])
def test_a_bad_coordinate_is_reported(bad):
    X, a, b = event(10, 1)
    for at in (0, 9, N * 10 - 1, 5_000_003):
        print(f"coordinate {at} is {bad}", flush=True)
        Y = X.clone()
        Y.view(-1)[at] = bad
        with pytest.raises(frnn.FrnnError) as err:
            frnn.build(Y, R, 8)
        assert err.value.status == frnn.FRNN_ERR_NONFINITE, at
    assert torch.equal(frnn.build(X, R, 8), edges_of(a, b, 8))  # and the next call is whole again


def test_too_small_outputs_report_the_edges_needed():
    X, a, b = event(6, 2)
    E = edges_of(a, b, 64).shape[1]
    print(f"E={E}", flush=True)
    ws = torch.empty(frnn.workspace_bytes(N, 6), dtype=torch.uint8, device=DEV)
    out = torch.full((2, E), -7, dtype=torch.int64, device=DEV)
    st, need = frnn.build_into(X, R, 64, ws, out[0, :E - 1], out[1, :E - 1])
    assert st == frnn.FRNN_ERR_CAPACITY and need == E
    st, need = frnn.build_into(X, R, 64, ws, out[0], out[1])
    assert st == frnn.FRNN_OK and need == E and torch.equal(out, edges_of(a, b, 64))
