"""The adjoint's tape (1 GiB, 64 bytes per step and seed): an interval that
passes it is swept in groups of checkpoint segments, a single segment that
passes it in parts of the seeds.  Both give the gradients of seed sets that
fit, recomputed or recorded."""

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


def _grads(n, grids, times, seeds, cot, ckpt, recorded, grid_grad=False):
    from paper_2004_02003_amd import Context

    with Context(n, len(seeds)) as ctx:
        ctx.set_tuning(ckpt_every=ckpt)
        ctx.seed_explicit(seeds)
        if recorded:
            ctx.advect(grids, times, record_ckpt=True)
        gg = [torch.zeros(g.shape, dtype=torch.float32, device="cuda") for g in grids] if grid_grad else None
        st = torch.empty(len(seeds), dtype=torch.uint8, device="cuda")
        out = ctx.adjoint(grids, times, cot, grad_grids=gg, ckpt_every=ckpt, status=st, recorded=recorded)
        torch.cuda.synchronize()
    return out.cpu(), st.cpu(), None if gg is None else torch.stack(gg).cpu()


# 360,000 seeds x 50 steps: 1.07 GiB of tape; ckpt 10: groups of 4 + 1
# segments, ckpt 50: one segment, 335,544 seeds and the rest
@pytest.mark.parametrize("dtype,recorded", [(torch.float32, False), (torch.float16, True)])
def test_intervals_beyond_the_tape(dtype, recorded):
    n, N, P = (27, 22, 17), 50, 360_000
    g = torch.Generator(device="cuda").manual_seed(7)
    grids = [(0.3 * torch.randn((n[2], n[1], n[0], 3), device="cuda", generator=g)).to(dtype) for _ in range(N + 1)]
    times = np.arange(N + 1) * 0.1
    hi = torch.tensor([v - 1.0 for v in n], dtype=torch.float64, device="cuda")
    seeds = torch.rand((P, 3), dtype=torch.float64, device="cuda", generator=g) * hi
    cot = 0.5 + torch.rand((P, 1, 3), device="cuda", generator=g)  # one sign: no cancelled sums
    print(f"[gpu-case] tape {dtype} recorded={recorded}", file=sys.stderr, flush=True)
    runs = {k: _grads(n, grids, times, seeds, cot, k, recorded, True) for k in (10, 50)}
    for k, (a, sa, _) in runs.items():
        assert 0.3 * P < int((sa == 0).sum()) < P
        for lo, m in ((0, 777), (335_000, 1500), (P - 65, 65)):
            s, ss, _ = _grads(n, grids, times, seeds[lo:lo + m].contiguous(), cot[lo:lo + m].contiguous(), k, recorded)
            assert torch.equal(ss, sa[lo:lo + m]) and torch.equal(s, a[lo:lo + m]), (k, lo, m)
    if not recorded:  # (a recorded forward is rounded at its launches, which the spacing cuts)
        (a, sa, ga), (b, sb, gb) = runs[10], runs[50]
        assert torch.equal(sa, sb) and torch.equal(a, b)
        # about 50 seeds per cell and level: each grid sum has fewer than 2,000
        # terms of one sign up to the flow's shear, added in different groupings
        assert (ga - gb).abs().max() <= 2e-5 * ga.abs().max()


# Record slots around the sort's tile of 4,096 (2 (N + 1) + 2 per seed, in
# sixteens), one to a hundred seeds per cell; 512^3 x 2 steps: 32 key bits, the
# marker of unused slots needs 64-bit keys.  A flow of one sign: a seed crosses
# each cell face once, so none runs out of record slots (the flushes beyond
# them are atomics, in no fixed order).
@pytest.mark.parametrize("n,N,P", [((5, 6, 7), 1, 1), ((9, 8, 7), 1, 682), ((9, 8, 7), 1, 683), ((4, 3, 5), 2, 2400),
                                   ((40, 30, 20), 5, 30_000), ((512, 512, 512), 2, 5000)])
def test_grid_gradient_reduction_at_its_sizes(n, N, P, monkeypatch):
    g = torch.Generator(device="cuda").manual_seed(P)
    grids = []
    for _ in range(N + 1):
        v = torch.rand((n[2], n[1], n[0], 3), device="cuda", generator=g)
        grids.append(v.mul_(0.4).add_(0.1).to(torch.float16))
        del v
    times = np.arange(N + 1) * 0.1
    hi = torch.tensor([v - 1.0 for v in n], dtype=torch.float64, device="cuda")
    seeds = torch.rand((P, 3), dtype=torch.float64, device="cuda", generator=g) * hi * 0.8 + 0.1 * hi
    cot = 0.5 + torch.rand((P, 1, 3), device="cuda", generator=g)
    print(f"[gpu-case] reduction {n} {N} {P}", file=sys.stderr, flush=True)
    from paper_2004_02003_amd import Context

    def run():
        gg = [torch.zeros(v.shape, dtype=torch.float32, device="cuda") for v in grids]
        with Context(n, P) as ctx:
            ctx.seed_explicit(seeds)
            ctx.adjoint(grids, times, cot, grad_grids=gg, ckpt_every=2)
            torch.cuda.synchronize()
        return gg

    a, b = run(), run()
    assert all(torch.equal(x, y) for x, y in zip(a, b))
    del b
    monkeypatch.setenv("BTO_GRAD_ATOMICS", "1")
    c = run()
    # fewer than 200 terms of (nearly) one sign per point, added in two orders
    top = max(float(x.abs().max()) for x in c)
    assert top > 0
    for x, y in zip(a, c):
        assert float((x - y).abs().max()) <= 2e-5 * top
        assert torch.equal(x != 0, y != 0)


@pytest.mark.parametrize("mode", ["linear", "frozen"])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float16, torch.bfloat16])
@pytest.mark.parametrize("P", [1, 65, 3000])
def test_tangent_sweep_equals_the_reverse_sweep(P, dtype, mode):
    """Three cotangents: carried forward from the seeds, and backwards from
    recorded checkpoints.  Two orders of the same FP32 products: N steps of
    four stages with eight roundings each, relative to the gradients' norm."""
    from paper_2004_02003_amd import Context

    n, N = (30, 21, 26), 13
    g = torch.Generator(device="cuda").manual_seed(P)
    grids = [(0.4 * torch.randn((n[2], n[1], n[0], 3), device="cuda", generator=g)).to(dtype) for _ in range(N + 1)]
    times = np.arange(N + 1) * 0.1
    hi = torch.tensor([v - 1.0 for v in n], dtype=torch.float64, device="cuda")
    sp = torch.tensor([0.5, 1.0, 0.25], dtype=torch.float64, device="cuda")
    seeds = (torch.rand((P, 3), dtype=torch.float64, device="cuda", generator=g) * 0.96 + 0.02) * hi * sp
    seeds[1::17] -= 100.0  # outside from the start
    cot = torch.randn((P, 3, 3), device="cuda", generator=g)
    print(f"[gpu-case] tangent {P} {dtype} {mode}", file=sys.stderr, flush=True)
    with Context(n, P, spacing=sp.tolist()) as ctx:
        ctx.set_tuning(ckpt_every=N, steps_per_launch=N)  # one launch: the recorded forward is the recomputed one
        st = [torch.empty(P, dtype=torch.uint8, device="cuda") for _ in range(2)]
        ctx.seed_explicit(seeds)
        ctx.advect(grids, times, mode=mode, record_ckpt=True)
        a = ctx.adjoint(grids, times, cot, ckpt_every=N, mode=mode, status=st[0], recorded=True)
        b = ctx.adjoint(grids, times, cot, ckpt_every=N, mode=mode, status=st[1])
        torch.cuda.synchronize()
    assert torch.equal(st[0], st[1])
    assert torch.equal(b[st[1] != 0], torch.zeros_like(b[st[1] != 0]))
    assert P < 100 or (st[1] == 1).any()
    assert float((a - b).norm()) <= N * 32 * 2.0 ** -24 * float(a.norm())


@pytest.mark.parametrize("dtype,n", [(torch.float16, (1024, 1023, 701)), (torch.float32, (1024, 701, 513))])
def test_adjoint_on_grids_beyond_4_gib(dtype, n):
    """A flow that lives in the last 60 x 50 x 40 points of a grid beyond 4 GiB
    (zero elsewhere, so a wrong address shows) against the same flow on a grid
    of those points alone: Jacobians (carried forward) and seed gradients
    (reverse sweep).  The same FP32 arithmetic on FP64 positions shifted by
    whole cells: offsets to 2^-24, four stages of two steps."""
    from paper_2004_02003_amd import Context

    g = torch.Generator(device="cuda").manual_seed(2)
    m = (60, 50, 40)
    big, small = [], []
    for _ in range(3):
        s = (0.3 * torch.randn((m[2], m[1], m[0], 3), device="cuda", generator=g)).to(dtype)
        b = torch.zeros((n[2], n[1], n[0], 3), dtype=dtype, device="cuda")
        assert b.numel() * b.element_size() > 1 << 32
        b[-m[2]:, -m[1]:, -m[0]:] = s
        big.append(b)
        small.append(s)
    P = 3000
    off = torch.tensor([a - b for a, b in zip(n, m)], dtype=torch.float64, device="cuda")
    hi = torch.tensor([v - 1.0 for v in m], dtype=torch.float64, device="cuda")
    x0 = 3.0 + torch.rand((P, 3), dtype=torch.float64, device="cuda", generator=g) * (hi - 4.0)  # up to the last cells
    cot = torch.randn((P, 3, 3), device="cuda", generator=g)
    out = []
    print(f"[gpu-case] adjoint beyond 4 GiB {dtype} {n}", file=sys.stderr, flush=True)
    for size, grids, seeds in ((n, big, x0 + off), (m, small, x0)):
        with Context(size, P) as ctx:
            ctx.seed_explicit(seeds.contiguous())
            st = torch.empty(P, dtype=torch.uint8, device="cuda")
            j = ctx.adjoint(grids, [0.0, 0.5, 1.0], cot, ckpt_every=2, status=st)
            r = ctx.adjoint(grids, [0.0, 0.5, 1.0], cot[:, :1].contiguous(), ckpt_every=2)
            torch.cuda.synchronize()
            out.append((st.cpu(), j.cpu(), r.cpu()))
    (sb, jb, rb), (ss, js, rs) = out
    assert int((ss == 0).sum()) > P // 2
    ok = (sb == 0) & (ss == 0)
    assert int((sb != ss).sum()) <= 2  # an end point within rounding of a face
    for a, b in ((jb, js), (rb, rs)):
        assert float((a[ok] - b[ok]).norm()) <= 2 * 32 * 2.0 ** -24 * 4 * float(b[ok].norm())
