"""Re-sorting the live particles between launches changes nothing but their
order: one-step launches with and without it give the same bits, for seed
counts around a wavefront, and when whole segments have emptied."""

import sys

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2004_02003_amd import _lib

    _lib.load()


@pytest.mark.parametrize("P", [1, 63, 65, 511, 5000])
def test_resorted_particles_end_where_they_did(P):
    from paper_2004_02003_amd import Context

    n, N = (70, 19, 23), 9
    g = torch.Generator(device="cuda").manual_seed(P)
    grids = [torch.randn((n[2], n[1], n[0], 3), device="cuda", generator=g) + 1.5 for _ in range(N + 1)]
    times = np.arange(N + 1) * 0.5
    hi = torch.tensor([v - 1.0 for v in n], dtype=torch.float64, device="cuda")
    seeds = torch.rand((P, 3), dtype=torch.float64, device="cuda", generator=g) * hi
    print(f"[gpu-case] rebin {P}", file=sys.stderr, flush=True)
    out = []
    for every in (0, 2):
        with Context(n, P) as ctx:
            ctx.set_tuning(steps_per_launch=1, rebin_every=every)
            ctx.seed_explicit(seeds)
            ctx.advect(grids, times)
            fm = ctx.flowmap()
            torch.cuda.synchronize()
            out.append({k: v.clone() for k, v in fm.items()})
    for k in out[0]:
        assert torch.equal(out[0][k], out[1][k]), k
    if P > 100:
        assert 0 < int((out[0]["flag"] == 0).sum()) < P
