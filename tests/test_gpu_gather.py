"""The gathering step (register windows of 16-bit rows, 32-bit offsets) against
the LDS-staged layout, whose step loads, addresses and samples another way with
the same arithmetic: flow maps equal bit for bit.

Sizes where a row window can go wrong: the smallest grids (every row is one of
the grid's last), odd and even points per axis (a row starts on a dword or
between two), an odd number of points (the last window starts 2 bytes early),
sizes around a tile's edge, and grids beyond 4 GiB (64-bit offsets)."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")


def _run(n, grids, seeds, tiles, mode="linear", fp64=False):
    from paper_2004_02003_amd import Context

    with Context(n, len(seeds)) as c:
        c.set_tuning(tiles=tiles, steps_per_launch=1)
        c.seed_explicit(seeds)
        for q in range(len(grids) - 1):
            c.advect(grids[q:q + 2], [0.5 * q, 0.5 * q + 0.5], mode=mode, record_exit=True, fp64=fp64)
        fm = c.flowmap(with_seeds=False)
        face = c.exit_points()
        st = c.stats()
        return [fm["end"].cpu(), fm["flag"].cpu(), fm["exit"].cpu(), face.cpu()], st


def _same(a, b, label):
    for u, v, nm in zip(a[0], b[0], ("end", "flag", "exit", "exit point")):
        assert torch.equal(u.nan_to_num(nan=-7.0), v.nan_to_num(nan=-7.0)) if u.is_floating_point() else torch.equal(u, v), \
            f"{label}: {nm} differs"
    assert a[1] == b[1], label


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16, torch.bfloat16])
@pytest.mark.parametrize("n", [(2, 2, 2), (3, 2, 2), (2, 3, 2), (3, 3, 3), (5, 4, 3), (33, 9, 9), (34, 10, 8),
                               (63, 17, 9)])
def test_gathered_rows_equal_staged_rows(n, dtype):
    rng = np.random.default_rng([n[0], n[1], n[2], 5])
    grids = [torch.from_numpy(rng.standard_normal((n[2], n[1], n[0], 3)) * 0.4).to("cuda", dtype) for _ in range(4)]
    hi = np.array(n) - 1.0
    corners = np.stack(np.meshgrid(*[[0.0, h] for h in hi], indexing="ij"), -1).reshape(-1, 3)
    near = np.clip(hi - rng.uniform(0, 1, (64, 3)), 0, hi)          # the last cells
    seeds = np.concatenate([corners, near, rng.uniform(0, 1, (300, 3)) * hi])
    seeds = torch.from_numpy(seeds).to("cuda")
    for mode, fp64 in (("linear", False), ("frozen", False), ("linear", True)):
        want = _run(n, grids, seeds, 1, mode, fp64)
        for tiles in (0, 2):
            _same(_run(n, grids, seeds, tiles, mode, fp64), want, f"{n} {dtype} {mode} fp64={fp64} tiles={tiles}")


@pytest.mark.parametrize("dtype,n", [(torch.float16, (1024, 1023, 701)), (torch.float32, (1024, 701, 513))])
def test_grids_beyond_4_gib(dtype, n):
    # one grid for both levels; values that differ from point to point, so a wrong address shows
    g = torch.empty((n[2], n[1], n[0], 3), dtype=dtype, device="cuda")
    assert g.numel() * g.element_size() > 1 << 32
    x = torch.arange(n[0], device="cuda", dtype=torch.float32).view(1, 1, -1)
    y = torch.arange(n[1], device="cuda", dtype=torch.float32).view(1, -1, 1)
    for k in range(0, n[2], 64):
        z = torch.arange(k, min(k + 64, n[2]), device="cuda", dtype=torch.float32).view(-1, 1, 1)
        g[k:k + 64, ..., 0] = 0.5 + 0.001 * z + 0 * (x + y)
        g[k:k + 64, ..., 1] = 0.25 + 0.0005 * x + 0 * (y + z)
        g[k:k + 64, ..., 2] = -0.5 + 0.0005 * y + 0 * (x + z)
    hi = torch.tensor([v - 1.0 for v in n], dtype=torch.float64, device="cuda")
    gen = torch.Generator(device="cuda").manual_seed(3)
    seeds = torch.rand((20000, 3), dtype=torch.float64, device="cuda", generator=gen) * hi
    seeds[:64] = hi - torch.rand((64, 3), dtype=torch.float64, device="cuda", generator=gen)  # the last points
    want = _run(n, [g, g, g], seeds, 1)
    for tiles in (0, 2):
        _same(_run(n, [g, g, g], seeds, tiles), want, f"{n} {dtype} tiles={tiles}")
