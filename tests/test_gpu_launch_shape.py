"""The advection's launch shapes -- a workgroup per 256 particles, two on a CU
at a time (sparse FP32 particles, launches of 2 or 8 steps on), or a capped number
that loops -- move the same particles by the same bits."""

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


# per segment (an eighth of the particles): under a workgroup, a few, and more
# than 6 x 32 (from where launches of 2 steps go in pairs)
@pytest.mark.parametrize("P,n", [(5, (40, 30, 20)), (2049, (9, 8, 7)), (2047, (40, 30, 20)), (420_001, (130, 121, 119))])
@pytest.mark.parametrize("K", [1, 2, 4, 9])
@pytest.mark.parametrize("dtype,fp64,lanes", [(torch.float32, False, 1), (torch.float16, False, 1),
                                              (torch.float32, True, 1), (torch.float32, False, 2)])
def test_launch_shapes_agree(P, n, K, dtype, fp64, lanes):
    from paper_2004_02003_amd import Context

    N = 9
    g = torch.Generator(device="cuda").manual_seed(P + K)
    grids = [(torch.randn((n[2], n[1], n[0], 3), device="cuda", generator=g) + 0.5).to(dtype) for _ in range(N + 1)]
    times = np.arange(N + 1) * 0.3
    hi = torch.tensor([v - 1.0 for v in n], dtype=torch.float64, device="cuda")
    seeds = torch.rand((P, 3), dtype=torch.float64, device="cuda", generator=g) * hi
    print(f"[gpu-case] launch shape {P} {K} {dtype} {fp64} {lanes}", file=sys.stderr, flush=True)
    out = []
    for cap in (0, 1):
        with Context(n, P) as ctx:
            ctx.set_tuning(steps_per_launch=K, blocks_per_cu=cap, lanes_per_particle=lanes)
            ctx.seed_explicit(seeds)
            ctx.advect(grids, times, fp64=fp64, record_exit=True)
            fm = ctx.flowmap()
            fm["face"] = ctx.exit_points()
            torch.cuda.synchronize()
            out.append({k: v.clone() for k, v in fm.items()})
    for k in out[0]:
        assert torch.equal(torch.nan_to_num(out[0][k]), torch.nan_to_num(out[1][k])), k
