"""Intervals swept in groups of checkpoint segments (the tape holds 1 GiB, 64
bytes per step and seed): what one group leaves to the next."""

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


def _say(msg):
    print(f"[gpu-case] {msg}", file=sys.stderr, flush=True)


def test_seeds_dropped_in_a_later_group():
    """360,000 seeds x 50 steps, checkpoints every 10: segments 4 to 1 are one
    group, segment 0 the next.  A flow along x, fast in the rows y <= 1 (three
    cells per step: four flushes, so the 99 record slots of a seed run out in
    the first group and the rest goes to the grids with atomics) and slow in the
    rows y >= 2 (one flush per level).  The adjoint is called with grids whose
    first ten levels flow back, so the seeds near the low face leave in the
    recomputed segment 0, after the first group has swept them: a slow one's
    records are all withdrawn (BTO_ADJ_DROPPED), a fast one's atomics cannot be
    (BTO_ADJ_DROPPED_PARTIAL).  The flow is uniform where the seeds are, so the
    others keep their cotangents, and the grid gradients sum to the kept
    cotangents times the interval: up to 3,000 terms per cell and level of one
    sign, each addition rounded to 2^-24.  The partly dropped seeds have zero
    cotangents, so that what they left adds nothing to that sum."""
    from paper_2004_02003_amd import Context, _lib

    n, N, k, P = (256, 4, 4), 50, 10, 360_000

    def grid(fast, slow):
        g = torch.zeros((n[2], n[1], n[0], 3), device="cuda")
        g[:, :2, :, 0] = fast
        g[:, 2:, :, 0] = slow
        return g

    fwd = grid(3.0, 0.05)
    back = grid(-6.0, -1.0)
    times = np.arange(N + 1, dtype=np.float64)
    gen = torch.Generator(device="cuda").manual_seed(5)
    u = torch.rand((P, 3), dtype=torch.float64, device="cuda", generator=gen)
    kind = torch.arange(P, device="cuda") % 4  # 0, 1: fast, 2, 3: slow; 0, 2: leave
    x0 = torch.tensor([40.0, 70.0, 1.0, 40.0], dtype=torch.float64, device="cuda")[kind]
    dx = torch.tensor([10.0, 30.0, 1.0, 60.0], dtype=torch.float64, device="cuda")[kind]
    seeds = torch.stack([x0 + dx * u[:, 0], torch.where(kind < 2, 0.2, 2.2) + 0.6 * u[:, 1], 0.5 + 2.0 * u[:, 2]], 1)
    cot = 0.5 + torch.rand((P, 1, 3), device="cuda", generator=gen)
    cot[kind == 0] = 0.0
    _say("seeds dropped in a later group")
    with Context(n, P) as ctx:
        ctx.set_tuning(ckpt_every=k)
        ctx.seed_explicit(seeds.contiguous())
        ctx.advect([fwd] * (N + 1), times, record_ckpt=True)
        grids = [back] * k + [fwd] * (N + 1 - k)
        gg = [torch.zeros_like(fwd) for _ in grids]
        st = torch.empty(P, dtype=torch.uint8, device="cuda")
        g = ctx.adjoint(grids, times, cot, grad_grids=gg, ckpt_every=k, status=st, recorded=True)
        torch.cuda.synchronize()
    assert torch.all(st[kind == 0] == _lib.BTO_ADJ_DROPPED_PARTIAL), torch.bincount(st[kind == 0].long())
    assert torch.all(st[kind == 2] == _lib.BTO_ADJ_DROPPED), torch.bincount(st[kind == 2].long())
    kept = (kind == 1) | (kind == 3)
    assert torch.all(st[kept] == 0)
    assert torch.all(g[~kept] == 0)
    assert float((g[kept] - cot[kept].reshape(g[kept].shape)).abs().max()) <= 1e-6
    total = torch.stack([x.double().reshape(-1, 3).sum(0) for x in gg]).sum(0)
    want = cot[kept].double().reshape(-1, 3).sum(0) * (times[-1] - times[0])
    assert float((total - want).abs().max() / want.abs().max()) <= 3000 * 2.0 ** -24


def _block(P, N, dtype, seed):
    """A flow of one sign (a seed crosses each cell face once, so none runs out
    of record slots), seeds anywhere: most leave at the high faces or stay."""
    n = (27, 22, 17)
    g = torch.Generator(device="cuda").manual_seed(seed)
    grids = [(0.1 + 0.4 * torch.rand((n[2], n[1], n[0], 3), device="cuda", generator=g)).to(dtype)
             for _ in range(N + 1)]
    hi = torch.tensor([v - 1.0 for v in n], dtype=torch.float64, device="cuda")
    seeds = torch.rand((P, 3), dtype=torch.float64, device="cuda", generator=g) * hi
    return n, grids, np.arange(N + 1) * 0.1, seeds, g


def _sweep(n, grids, times, seeds, cot, k, recorded, grid_grad):
    from paper_2004_02003_amd import Context

    P = len(seeds)
    with Context(n, P) as ctx:
        ctx.set_tuning(ckpt_every=k)
        ctx.seed_explicit(seeds)
        if recorded:
            ctx.advect(grids, times, record_ckpt=True)
        gg = [torch.zeros(v.shape, dtype=torch.float32, device="cuda") for v in grids] if grid_grad else None
        st = torch.empty(P, dtype=torch.uint8, device="cuda")
        out = ctx.adjoint(grids, times, cot, grad_grids=gg, ckpt_every=k, status=st, recorded=recorded)
        torch.cuda.synchronize()
    return out, st, gg


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_grid_gradients_do_not_depend_on_the_groups(dtype):
    """Groups of 4 + 1 segments of 10 steps, of 1 + 1 segments of 25, and one
    segment of 50 steps swept for a part of the seeds at a time: the same
    records in the same order, so the same bits."""
    P, N = 360_000, 50
    n, grids, times, seeds, g = _block(P, N, dtype, 3)
    cot = 0.5 + torch.rand((P, 1, 3), device="cuda", generator=g)
    _say(f"grid gradients by group {dtype}")
    a, sa, ga = _sweep(n, grids, times, seeds, cot, 50, False, True)
    assert 0.5 * P < int((sa == 0).sum()) < P
    for k in (10, 25):
        b, sb, gb = _sweep(n, grids, times, seeds, cot, k, False, True)
        assert torch.equal(sa, sb) and torch.equal(a, b), k
        assert all(torch.equal(x, y) for x, y in zip(ga, gb)), k


@pytest.mark.parametrize("k", [10, 25])
def test_recorded_groups_sum_to_their_seed_subsets(k):
    """Grid gradients from recorded checkpoints over several groups against
    three subsets of the seeds that each fit one sweep: the same terms, up to
    2,000 of one sign per point, added in another order.  Seed gradients are
    the subsets' bits, also with three cotangents."""
    P, N = 360_000, 50
    n, grids, times, seeds, g = _block(P, N, torch.float16, 4)
    cot = 0.5 + torch.rand((P, 1, 3), device="cuda", generator=g)
    cot3 = torch.randn((P, 3, 3), device="cuda", generator=g)
    _say(f"recorded groups, checkpoints every {k}")
    a, sa, ga = _sweep(n, grids, times, seeds, cot, k, True, True)
    j, sj, _ = _sweep(n, grids, times, seeds, cot3, k, True, False)
    assert torch.equal(sa, sj) and int((sa == 0).sum()) > P // 2
    total = [torch.zeros(v.shape, dtype=torch.float64, device="cuda") for v in grids]
    for lo, hi in ((0, 100_000), (100_000, 230_000), (230_000, P)):
        s, ss, gs = _sweep(n, grids, times, seeds[lo:hi].contiguous(), cot[lo:hi].contiguous(), k, True, True)
        assert torch.equal(ss, sa[lo:hi]) and torch.equal(s, a[lo:hi]), (lo, hi)
        for t, v in zip(total, gs):
            t += v
        s, ss, _ = _sweep(n, grids, times, seeds[lo:hi].contiguous(), cot3[lo:hi].contiguous(), k, True, False)
        assert torch.equal(ss, sj[lo:hi]) and torch.equal(s, j[lo:hi]), (lo, hi)
    top = max(float(t.abs().max()) for t in total)
    assert top > 0
    for t, v in zip(total, ga):
        assert float((t - v).abs().max()) <= 2000 * 2.0 ** -24 * top
