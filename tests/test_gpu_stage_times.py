"""Stage times: a stage without a kernel reads 0, the others are positive and add up to no
more than the call takes."""

import time

import pytest
import torch

from paper_2202_06929_amd import frnn

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("n", [1, 5000, 120_000, (1 << 20) + 1])
def test_stages(n):
    print(f"n={n}", flush=True)
    pts = torch.rand((n, 4), generator=torch.Generator(device=DEV).manual_seed(n), device=DEV)
    for timing in (True, False, True):
        torch.cuda.synchronize()
        begin = time.perf_counter()
        _, stats = frnn.build(pts, 0.01, 16, frnn.Config(timing=timing), return_stats=True)
        took = (time.perf_counter() - begin) * 1e3
        ms = stats["stage_ms"]
        assert list(ms) == list(frnn.STAGES)
        if not timing:
            assert not any(ms.values())
            continue
        assert all(v > 0 for k, v in ms.items() if k != "cells")
        assert (ms["cells"] == 0.0) == (n <= 1 << 20)
        assert sum(ms.values()) <= took
