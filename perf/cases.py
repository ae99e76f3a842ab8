"""The work that a program has this library do, as cases with sizes.

Each case goes through the public entry points only.  Four kinds:

* ``insitu``  -- one interval of the in situ form: seed the lattice, one RK4
  step per call with that cycle's two grids, write the flow map.  With
  ``driver`` the interval runs through ``InSituDriver`` (one ``cycle`` call per
  simulation cycle).
* ``fused``   -- one interval with every cycle resident: seed, one ``advect``
  call, flow map (and the exit points where they are recorded).
* ``grad``    -- differentiable flow map: forward, and the gradients of the end
  positions with respect to the seeds and every grid.
* ``jacobian``-- flow-map Jacobians and FTLE of explicit seeds.
* ``posthoc`` -- per-block flow maps placed into one lattice, terminated
  entries rebuilt, the result scored against the communicating flow map.

Inputs are synthetic and made on the GPU from the seed alone: Fourier-mode
turbulence (1.5 cells of rms displacement per step, the turbulent blocks), an
ABC flow with noise (slow: about 0.15 cells per step), and for ``posthoc`` a
smooth displacement of the lattice.  An in situ interval longer than its
resident grids walks them back and forth, so that consecutive calls always see
consecutive cycles.
"""

from __future__ import annotations

import math

import numpy as np
import torch

from paper_2004_02003_amd import Context, InSituDriver, advect_autograd, jacobian_ftle
from paper_2004_02003_amd.posthoc import flowmap_error, place_block, reconstruct_lattice

_DT = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
_ITEM = {"f32": 4, "f16": 2, "bf16": 2}
_GRID_CAP = 6 << 30      # bytes of resident grids of an in situ case
_DEV = "cuda"


def _case(kind, n, stride, steps, dtype="f32", flow="turb", mode="linear", tiles=0, fp64=False, exits=False,
          driver=False, lanes=1, rebin=0, name=None):
    c = dict(kind=kind, nx=n[0], ny=n[1], nz=n[2], stride=stride, steps=steps, dtype=dtype, flow=flow, mode=mode,
             tiles=tiles, fp64=fp64, exits=exits, driver=driver, lanes=lanes, rebin=rebin)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # a rank's 64^3 block of the ABC run at 1:27, one cycle per call through the driver: latency and host time
        _case("insitu", (64, 64, 64), 3, 25, flow="abc", driver=True, name="rank64_f32_driver"),
        # a ragged block, FROZEN time stepping (one grid per step in use), exit points recorded and read back
        _case("fused", (97, 61, 83), 2, 25, "bf16", "turb", mode="frozen", exits=True, name="ragged_bf16_frozen_exits"),
        # the 128^3 ABC block with all cycles resident
        _case("fused", (128, 128, 128), 2, 100, flow="abc", name="abc128_f32_fused"),
        # the same block, one cycle per call
        _case("insitu", (128, 128, 128), 2, 50, flow="abc", name="abc128_f32_insitu"),
        # turbulent 256^3 block in FP32, one cycle per call, particles kept by tile
        _case("insitu", (256, 256, 256), 2, 25, tiles=2, name="turb256_f32_insitu"),
        # the same with extended-precision sampling, on a block that no tile divides
        _case("insitu", (201, 150, 177), 2, 25, tiles=2, fp64=True, name="turb201_f32_fp64_insitu"),
        # bfloat16 storage, one cycle per call
        _case("insitu", (256, 256, 256), 2, 25, "bf16", tiles=2, name="turb256_bf16_insitu"),
        # the largest block: 512^3 in FP16, 16.7 million particles, one cycle per call
        _case("insitu", (512, 512, 512), 2, 20, "f16", tiles=2, name="turb512_f16_insitu"),
        # turbulent 256^3 block in FP16 with every cycle resident, re-sorted every 5 steps
        _case("fused", (256, 256, 256), 2, 25, "f16", rebin=5, name="turb256_f16_fused"),
        # a training step: forward with checkpoints, then seed and grid gradients
        _case("grad", (128, 128, 128), 4, 50, flow="abc", name="abc128_f32_grad"),
        # flow-map Jacobians and FTLE of a sparse lattice in FP16 turbulence
        _case("jacobian", (160, 144, 136), 4, 50, "f16", name="turb160_f16_jacobian"),
        # eight blocks' flow maps into one 128^3 lattice, rebuilt and scored
        _case("posthoc", (64, 64, 64), 2, 50, name="posthoc_128_lattice"),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["insitu", "insitu", "insitu", "fused", "fused", "grad", "jacobian", "posthoc"])
    if kind == "posthoc":
        return _case("posthoc", [_logint(rng, 12, 96) for _ in range(3)], rng.choice([2, 3]), rng.randint(10, 100))
    if kind in ("grad", "jacobian"):
        n = [_logint(rng, 32, 144) for _ in range(3)]
        return _case(kind, n, rng.choice([3, 4, 5]), rng.randint(8, 50),
                     "f32" if kind == "grad" else rng.choice(["f32", "f16", "bf16"]), rng.choice(["abc", "turb"]),
                     rng.choice(["linear", "linear", "linear", "frozen"]))
    dtype = rng.choice(["f32", "f32", "f16", "bf16"])
    if kind == "fused":
        n = [_logint(rng, 24, 224) for _ in range(3)]
        flow = rng.choice(["abc", "turb"])
        return _case("fused", n, rng.choice([1, 2, 2, 3]), rng.randint(5, 60), dtype, flow,
                     rng.choice(["linear", "linear", "linear", "frozen"]), fp64=rng.random() < 0.2,
                     exits=rng.random() < 0.25, lanes=2 if dtype == "f32" and flow == "turb" else 1,
                     rebin=5 if flow == "turb" else 0)
    n = [_logint(rng, 24, 384) for _ in range(3)]
    flow = rng.choice(["abc", "turb", "turb"])
    # the turbulent blocks keep their particles by tile, the slow ones in seed order
    return _case("insitu", n, rng.choice([1, 2, 2, 3]) if max(n) < 256 else rng.choice([2, 3]), rng.randint(5, 25),
                 dtype, flow, rng.choice(["linear", "linear", "linear", "frozen"]), tiles=2 if flow == "turb" else 0,
                 fp64=rng.random() < 0.2, exits=rng.random() < 0.2, driver=flow == "abc" and rng.random() < 0.5)


# ---------------------------------------------------------------------------
# Inputs.
# ---------------------------------------------------------------------------
def _n(case):
    return int(case["nx"]), int(case["ny"]), int(case["nz"])


def _lattice(n, stride):
    off = (stride - 1) / 2.0
    return tuple(int(math.floor((d - 1 - off) / stride)) + 1 for d in n)


def _seeds(case):
    return int(np.prod(_lattice(_n(case), case["stride"])))


def _dt(case):
    return 0.05 if case["flow"] == "abc" else 0.02


def _turb_modes(rng, L, dt, M=64):
    """Divergence-free modes, |k| in 1..16 periods of L, rms displacement 1.5 cells per dt."""
    km = rng.uniform(1.0, 16.0, M)
    d = rng.standard_normal((M, 3))
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    r = rng.standard_normal((M, 3))
    r -= (r * d).sum(1, keepdims=True) * d
    r /= np.linalg.norm(r, axis=1, keepdims=True)
    a = km[:, None] ** (-5.0 / 6.0) * r
    a *= (1.5 / dt) / math.sqrt(0.5 * float((a * a).sum()))
    k = (2 * math.pi / L) * km[:, None] * d
    return k, a, rng.uniform(0, 2 * math.pi, M), 0.1 * (1.5 / dt) * np.linalg.norm(k, axis=1)


def _grids(case, seed, count):
    """`count` consecutive cycles: contiguous (nz, ny, nx, 3) device tensors in the storage type."""
    nx, ny, nz = _n(case)
    dt, dtype = _dt(case), _DT[case["dtype"]]
    rng = np.random.default_rng(seed)
    ax = [torch.arange(m, dtype=torch.float64, device=_DEV) for m in (nx, ny, nz)]
    out = []
    if case["flow"] == "turb":
        k, a, ph, om = _turb_modes(rng, max(nx, ny, nz), dt)
        k, a, ph, om = (torch.from_numpy(np.ascontiguousarray(v)).to(_DEV) for v in (k, a, ph, om))
        ang = [k[:, d, None] * ax[d][None, :] for d in range(3)]
        # u(z, y, x, c) = Re sum_m a_mc e^{i(kx x + ky y + kz z + om t + ph)} as one product of real matrices
        right = torch.cat([a[:, None, :] * torch.cos(ang[0])[:, :, None],
                           -a[:, None, :] * torch.sin(ang[0])[:, :, None]]).reshape(-1, 3 * nx).float()
        for c in range(count):
            yz = ang[2][:, :, None] + ang[1][:, None, :] + (om * (c * dt) + ph)[:, None, None]
            left = torch.cat([torch.cos(yz).reshape(len(om), -1), torch.sin(yz).reshape(len(om), -1)]).t().float()
            out.append((left.contiguous() @ right).view(nz, ny, nx, 3).to(dtype))
            del yz, left
        return out
    g = torch.Generator(device=_DEV).manual_seed(seed)
    k, sh = 2 * math.pi / (2 * max(nx, ny, nz)), rng.uniform(0, 2 * math.pi, 3)
    X, Y, Z = (k * ax[d] + sh[d] for d in range(3))
    A, B, C = math.sqrt(3.0), math.sqrt(2.0), 1.0
    u = A * torch.sin(Z)[:, None, None] + C * torch.cos(Y)[None, :, None] + 0 * X
    v = B * torch.sin(X)[None, None, :] + A * torch.cos(Z)[:, None, None] + 0 * Y[None, :, None]
    w = C * torch.sin(Y)[None, :, None] + B * torch.cos(X)[None, None, :] + 0 * Z[:, None, None]
    base = torch.stack([u, v, w], dim=-1).float()
    for c in range(count):
        noise = torch.randn(base.shape, generator=g, device=_DEV, dtype=torch.float32)
        out.append(((1.0 + 0.1 * math.sin(c * dt)) * base + 0.01 * noise).to(dtype))
    return out


def _resident(case):
    """Grids held by the case: every cycle where all are resident, else what fits the cap (at least 4)."""
    per = int(np.prod(_n(case))) * 3 * _ITEM[case["dtype"]]
    if case["kind"] != "insitu":
        return case["steps"] + 1
    return min(case["steps"] + 1, max(4, min(26, _GRID_CAP // per)))


def _walk(case):
    """Grid index of each cycle: 0, 1, .., G-1, G-2, .., 0, 1, .."""
    G, N = _resident(case), case["steps"] + 1
    period = 2 * (G - 1)
    return [min(c % period, period - c % period) for c in range(N)]


def _explicit_seeds(case, seed):
    """A jittered lattice, (P, 3) float64 in cell units."""
    n, s = _n(case), case["stride"]
    m = _lattice(n, s)
    z, y, x = torch.meshgrid(*[torch.arange(m[d], dtype=torch.float64, device=_DEV) for d in (2, 1, 0)], indexing="ij")
    p = (s - 1) / 2.0 + s * torch.stack([x, y, z], dim=-1).reshape(-1, 3)
    g = torch.Generator(device=_DEV).manual_seed(seed + 77)
    p = p + 0.45 * (torch.rand(p.shape, generator=g, device=_DEV, dtype=torch.float64) * 2 - 1)
    hi = torch.tensor([v - 1.0 for v in n], dtype=torch.float64, device=_DEV)
    return torch.minimum(p.clamp_min(0.0), hi).contiguous()


def _posthoc_maps(case, seed):
    """Per-block flow maps (block coordinates, flags) and the communicating one
    (domain coordinates), for 2 x 2 x 2 blocks: a smooth displacement of a few
    cells per axis, terminated where it leaves the block (the domain)."""
    m, s = _n(case), case["stride"]
    rng = np.random.default_rng(seed)
    cells = [v * s for v in m]
    M = tuple(2 * v for v in m)
    off = (s - 1) / 2.0
    z, y, x = torch.meshgrid(*[off + s * torch.arange(M[d], dtype=torch.float64, device=_DEV) for d in (2, 1, 0)],
                             indexing="ij")
    x0 = torch.stack([x, y, z], dim=-1)
    u = torch.zeros_like(x0)
    for _ in range(8):
        k = torch.from_numpy(2 * math.pi * rng.uniform(-3, 3, 3) / (2 * max(cells))).to(_DEV)
        a = torch.from_numpy(rng.standard_normal(3) * (0.05 * case["steps"])).to(_DEV)
        u = u + torch.sin(x0 @ k + rng.uniform(0, 2 * math.pi))[..., None] * a
    end = x0 + u

    def kept(lo, hi, e):
        return ((e >= torch.tensor(lo, dtype=torch.float64, device=_DEV)) &
                (e <= torch.tensor(hi, dtype=torch.float64, device=_DEV))).all(-1)

    blocks = []
    for b in range(8):
        o = [b & 1, (b >> 1) & 1, b >> 2]
        sl = tuple(slice(o[d] * m[d], (o[d] + 1) * m[d]) for d in (2, 1, 0))
        lo = [float(o[d] * cells[d]) for d in range(3)]
        e = end[sl]
        ok = kept(lo, [lo[d] + cells[d] for d in range(3)], e)
        local = (e - torch.tensor(lo, dtype=torch.float64, device=_DEV)).reshape(-1, 3).contiguous()
        blocks.append((local, (~ok).to(torch.uint8).reshape(-1).contiguous(), [o[d] * m[d] for d in range(3)], lo))
    ref = (end + 1e-6 * torch.sin(7 * end)).reshape(-1, 3).contiguous()
    rflag = (~kept([0.0] * 3, [2.0 * c for c in cells], end)).to(torch.uint8).reshape(-1).contiguous()
    return M, blocks, ref, rflag


def prepare(case, seed):
    if case["kind"] == "posthoc":
        M, blocks, ref, rflag = _posthoc_maps(case, seed)
        P = int(np.prod(M))
        return dict(case=case, M=M, blocks=blocks, ref=ref, rflag=rflag,
                    end=torch.empty((P, 3), dtype=torch.float64, device=_DEV),
                    flag=torch.empty(P, dtype=torch.uint8, device=_DEV))
    n = _n(case)
    ctx = Context(n, _seeds(case))
    ctx.set_tuning(tiles=case["tiles"], lanes_per_particle=case["lanes"], rebin_every=case["rebin"])
    grids = _grids(case, seed, _resident(case))
    dt = _dt(case)
    st = dict(case=case, ctx=ctx, grids=grids, times=[c * dt for c in range(case["steps"] + 1)])
    if case["kind"] == "insitu":
        st["cycles"] = [grids[i] for i in _walk(case)]
    if case["kind"] in ("grad", "jacobian"):
        st["seeds"] = _explicit_seeds(case, seed)
    if case["kind"] == "grad":
        g = torch.Generator(device=_DEV).manual_seed(seed + 5)
        st["cot"] = torch.randn(st["seeds"].shape, generator=g, device=_DEV, dtype=torch.float64)
        st["seeds"].requires_grad_(True)
        for v in grids:
            v.requires_grad_(True)
    return st


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "posthoc":
        m = _n(case)
        for end, flag, off, shift in st["blocks"]:
            place_block(end, flag, m, st["end"], st["flag"], st["M"], off, shift=shift)
        state = reconstruct_lattice(st["end"], st["flag"], st["M"])
        err = flowmap_error(st["end"], state, st["ref"], st["rflag"], cell=1.0)
        return dict(end=st["end"], flag=st["flag"], state=state, **err)
    ctx, times = st["ctx"], st["times"]
    if kind == "jacobian":
        J, sigma, status = jacobian_ftle(ctx, st["seeds"], st["grids"], times, mode=case["mode"])
        return dict(jac=J, ftle=sigma, status=status)
    if kind == "grad":
        end, flag, exit_step = advect_autograd(ctx, st["seeds"], st["grids"], times, mode=case["mode"])
        gr = torch.autograd.grad(end, [st["seeds"], *st["grids"]], grad_outputs=st["cot"])
        return dict(end=end.detach(), flag=flag, exit=exit_step, grad_seed=gr[0], grad_grids=list(gr[1:]))
    if kind == "fused":
        ctx.seed(case["stride"])
        ctx.advect(st["grids"], times, mode=case["mode"], record_exit=case["exits"], fp64=case["fp64"])
        fm = ctx.flowmap()
    elif case["driver"]:
        got = []
        d = InSituDriver(ctx, interval=case["steps"], stride=case["stride"], mode=case["mode"],
                         on_flowmap=lambda i, f, t0, t1: got.append(f))
        for g, t in zip(st["cycles"], times):
            d.cycle(g, t)
        return got[0]
    else:
        ctx.seed(case["stride"])
        cyc = st["cycles"]
        for s in range(case["steps"]):
            ctx.advect([cyc[s], cyc[s + 1]], times[s:s + 2], mode=case["mode"], record_exit=case["exits"],
                       fp64=case["fp64"])
        fm = ctx.flowmap()
    if case["exits"]:
        fm["face"] = ctx.exit_points()
    return fm


def work(case):
    """Bytes: every grid that a call is given, as far as the seeds touch it
    (at most 8 points per seed), once per call, and every output once.  Flops:
    about 340 per RK4 step of a particle (four trilinear samples of three
    components, two of them over two levels, and the FP64 stage points), with
    three quarters of the seeds advancing on average."""
    if case["kind"] == "posthoc":
        P = 8 * int(np.prod(_n(case)))
        return dict(bytes=P * (25 + 25 + 1 + 25), flops=P * 20)
    P, S = _seeds(case), case["steps"]
    npts = int(np.prod(_n(case)))
    level = min(npts, 8 * P) * 3
    per = 1 if case["mode"] == "frozen" else 2
    reads = {"insitu": per * S, "fused": S + 1, "grad": 2 * (S + 1), "jacobian": S + 1}[case["kind"]]
    out = {"insitu": 53 * P, "fused": 53 * P, "grad": (29 + 24 + 24) * P + 4 * npts * 3 * (S + 1),
           "jacobian": (36 + 4 + 1 + 24) * P}[case["kind"]]
    flops = 340.0 * 0.75 * P * S * {"insitu": 1, "fused": 1, "grad": 5, "jacobian": 7}[case["kind"]]
    return dict(bytes=reads * level * _ITEM[case["dtype"]] + out + (24 * P if case["exits"] else 0), flops=flops)


# ---------------------------------------------------------------------------
# The same in 64 bits, in plain torch.
# ---------------------------------------------------------------------------
def _sample(flat, n, p):
    """Trilinear sample of one grid (points x 3, storage type) at p (P, 3)."""
    top = torch.tensor([v - 2 for v in n], dtype=torch.float64, device=p.device)
    i = torch.minimum(torch.floor(p.detach()), top)
    f = p - i
    i = i.long()
    base = i[:, 0] + n[0] * (i[:, 1] + n[1] * i[:, 2])
    v = 0.0
    for c in range(8):
        b = (c & 1, (c >> 1) & 1, c >> 2)
        w = 1.0
        for d in range(3):
            w = w * (f[:, d] if b[d] else 1.0 - f[:, d])
        v = v + w[:, None] * flat[base + (b[0] + n[0] * (b[1] + n[1] * b[2]))].double()
    return v


def _step(A, B, h, n, x, hi):
    """One RK4 step (A: level n, B: level n + 1, or None when frozen): end
    point, the first outside point, and whether one was found."""
    def mid(y):
        return _sample(A, n, y) if B is None else 0.5 * (_sample(A, n, y) + _sample(B, n, y))

    bad = torch.zeros(len(x), dtype=torch.bool, device=x.device)
    face = torch.full_like(x, math.nan)

    def check(y):
        nonlocal bad, face
        out = ~((y >= 0) & (y <= hi)).all(-1) & ~bad
        face = torch.where(out[:, None], y, face)
        bad = bad | out
        return torch.where(bad[:, None], x, y)

    k1 = _sample(A, n, x)
    k2 = mid(check(x + 0.5 * h * k1))
    k3 = mid(check(x + 0.5 * h * k2))
    k4 = _sample(A if B is None else B, n, check(x + h * k3))
    y = check(x + h / 6 * (k1 + 2 * k2 + 2 * k3 + k4))
    return y, face, bad


def _advance(case, cycles, times, x, hi, keep=None):
    """The interval from x (P, 3): end, flag, exit step and outside point."""
    n, S = _n(case), case["steps"]
    flat = [g.reshape(-1, 3) for g in cycles]
    P = len(x)
    end = x.clone()
    inside = ((x >= 0) & (x <= hi)).all(-1)
    flag = (~inside).to(torch.uint8)
    step = torch.where(inside, S, 0).to(torch.int32)
    face = torch.full_like(x, math.nan)
    for q in range(0, P, 1 << 21):
        ids = torch.nonzero(inside[q:q + (1 << 21)]).flatten() + q
        y = x[ids]
        for s in range(S):
            if not len(ids):
                break
            B = None if case["mode"] == "frozen" else flat[s + 1]
            z, f, bad = _step(flat[s], B, times[s + 1] - times[s], n, y, hi)
            dead = ids[bad]
            end[dead], face[dead] = y[bad], f[bad]
            flag[dead] = 1
            step[dead] = s
            ids, y = ids[~bad], z[~bad]
        end[ids] = y
    return end, flag, step, face


def _exit_face(x, y, hi):
    """Where the segment from x (inside) to y (outside) meets the box."""
    lo = y < 0
    over = y > hi
    fv = torch.where(lo, torch.zeros_like(y), hi.expand_as(y))
    t = torch.where(lo | over, (fv - x) / (y - x), torch.full_like(y, math.inf))
    tau, ax = t.min(-1)
    p = torch.minimum((x + tau[:, None] * (y - x)).clamp_min(0.0), hi)
    at = torch.zeros_like(lo).scatter_(1, ax[:, None], True)
    return torch.where(at, fv, p)


def _exact_posthoc(case, seed):
    M, blocks, ref, rflag = _posthoc_maps(case, seed)
    m = _n(case)
    end = torch.empty((M[2], M[1], M[0], 3), dtype=torch.float64, device=_DEV)
    flag = torch.empty((M[2], M[1], M[0]), dtype=torch.uint8, device=_DEV)
    for e, f, off, shift in blocks:
        sl = tuple(slice(off[d], off[d] + m[d]) for d in (2, 1, 0))
        end[sl] = e.view(m[2], m[1], m[0], 3) + torch.tensor(shift, dtype=torch.float64, device=_DEV)
        flag[sl] = f.view(m[2], m[1], m[0])
    known = flag == 0
    state = known.to(torch.uint8)
    end[~known] = math.nan
    for dim in (2, 1, 0):
        L = end.shape[dim]
        shape = [1, 1, 1]
        shape[dim] = L
        idx = torch.arange(L, device=_DEV).view(shape).expand(known.shape)
        lo = torch.where(known, idx, -1).cummax(dim).values
        hi = torch.where(known, idx, L).flip(dim).cummin(dim).values.flip(dim)
        fill = ~known & (lo >= 0) & (hi < L)
        pick = lambda i: torch.gather(end, dim, i.clamp(0, L - 1)[..., None].expand(end.shape))  # noqa: E731
        span = (hi - lo).double()
        val = ((idx - lo) / span)[..., None] * pick(hi) + ((hi - idx) / span)[..., None] * pick(lo)
        end = torch.where(fill[..., None], val, end)
        state[fill] = 2
        known = known | fill
    end, state, flag = end.reshape(-1, 3), state.reshape(-1), flag.reshape(-1)
    use = rflag == 0
    cov = use & (state != 0)
    d = (end - ref)[cov].norm(dim=-1)
    mean = float(d.mean()) if len(d) else 0.0
    return dict(end=end, flag=flag, state=state, mean_l2=mean, max_l2=float(d.max()) if len(d) else 0.0,
                n=int(cov.sum()), uncovered=int((use & (state == 0)).sum()), accuracy_pct=(1.0 - mean) * 100.0)


def exact(case, seed):
    if case["kind"] == "posthoc":
        return _exact_posthoc(case, seed)
    if _seeds(case) * case["steps"] > (1 << 26):
        return None
    n, S = _n(case), case["steps"]
    hi = torch.tensor([v - 1.0 for v in n], dtype=torch.float64, device=_DEV)
    grids = _grids(case, seed, _resident(case))
    times = [c * _dt(case) for c in range(S + 1)]
    if case["kind"] in ("insitu", "fused"):
        cycles = [grids[i] for i in _walk(case)] if case["kind"] == "insitu" else grids
        m, s = _lattice(n, case["stride"]), case["stride"]
        z, y, x = torch.meshgrid(*[torch.arange(m[d], dtype=torch.float64, device=_DEV) for d in (2, 1, 0)],
                                 indexing="ij")
        x0 = (s - 1) / 2.0 + s * torch.stack([x, y, z], dim=-1).reshape(-1, 3)
        end, flag, step, face = _advance(case, cycles, times, x0, hi)
        out = dict(end=end, flag=flag, exit=step, seed=x0)
        if case["exits"]:
            out["face"] = torch.where((flag == 1)[:, None], _exit_face(end, face, hi), math.nan)
        return out
    seeds = _explicit_seeds(case, seed)
    end, flag, step, _ = _advance(case, grids, times, seeds, hi)
    ids = torch.nonzero(flag == 0).flatten()
    # gradients over the seeds that stay inside, by autograd, one step's graph at a time
    want = case["kind"] == "grad"
    P, nc = len(seeds), 1 if want else 3
    xs = [seeds[ids]]
    with torch.no_grad():
        for s in range(S):
            B = None if case["mode"] == "frozen" else grids[s + 1].reshape(-1, 3)
            xs.append(_step(grids[s].reshape(-1, 3), B, times[s + 1] - times[s], n, xs[-1], hi)[0])
    if want:
        g = torch.Generator(device=_DEV).manual_seed(seed + 5)
        lam = torch.randn(seeds.shape, generator=g, device=_DEV, dtype=torch.float64)[ids][None]
    else:
        lam = torch.eye(3, dtype=torch.float64, device=_DEV)[:, None, :].expand(3, len(ids), 3)
    # sums in 64 bits, written as the float32 nearest to them (a grid's sum is whole once its two steps are through)
    gg = [None] * (S + 1)
    for s in range(S - 1, -1, -1):
        x = xs[s].clone().requires_grad_(True)
        A = grids[s].reshape(-1, 3).double().requires_grad_(want)
        B = None if case["mode"] == "frozen" else grids[s + 1].reshape(-1, 3).double().requires_grad_(want)
        y = _step(A, B, times[s + 1] - times[s], n, x, hi)[0]
        ask = [x] + ([A] + ([B] if B is not None else []) if want else [])
        new = []
        for c in range(nc):
            r = torch.autograd.grad(y, ask, grad_outputs=lam[c], retain_graph=c + 1 < nc)
            new.append(r[0])
            if want:
                gg[s] = r[1] if gg[s] is None else gg[s] + r[1]
                if B is not None:
                    gg[s + 1] = r[2] if gg[s + 1] is None else gg[s + 1] + r[2]
        lam = torch.stack(new)
    J = torch.zeros((P, nc, 3), dtype=torch.float64, device=_DEV)
    J[ids] = lam.permute(1, 0, 2)
    if want:
        shape = tuple(grids[0].shape)
        zero = torch.zeros(int(np.prod(shape)) // 3, 3, dtype=torch.float64, device=_DEV)
        return dict(end=end, flag=flag, exit=step, grad_seed=J.view(P, 3),
                    grad_grids=[(zero if v is None else v).view(shape) for v in gg])
    C = (J.transpose(1, 2) @ J).cpu().numpy()
    top = np.linalg.eigvalsh(C)[:, 2]
    with np.errstate(divide="ignore"):
        sigma = 0.5 * np.log(np.where(top > 0, top, 0.0)) / (times[-1] - times[0])
    return dict(jac=J, ftle=torch.from_numpy(sigma), status=flag)
