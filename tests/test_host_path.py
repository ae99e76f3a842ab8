"""The library's host code on a card that is short of memory, seen from outside:
the library is loaded behind a HIP runtime without a device (fake_hip.c), which
logs allocations, copies, waits and launches and refuses what it is told to.
Each case runs in a process of its own.  No GPU."""

import ctypes
import os
import re
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
STREAM = 7


class Host:
    """The library behind the fake runtime."""

    def __init__(self, fake):
        self.f = ctypes.CDLL(fake, mode=ctypes.RTLD_GLOBAL)
        self.f.fake_log.restype = ctypes.c_char_p
        self.f.fake_memory.argtypes = [ctypes.c_size_t]
        sys.path.insert(0, os.path.join(ROOT, "paper_2004_02003_amd"))
        import _lib

        self.lib, self.L = _lib, _lib.load()

    def create(self, n, cap):
        b = self.lib.Block()
        b.n[:], b.spacing[:] = n, [1.0] * 3
        h = ctypes.c_void_p()
        assert self.L.bto_create(ctypes.byref(b), cap, 0, ctypes.byref(h)) == 0
        return h

    def seed(self, h, P):
        assert self.L.bto_seed_explicit(h, 1 << 50, P, STREAM) == 0

    def tune(self, h, **kw):
        t = self.lib.Tuning()
        assert self.L.bto_get_tuning(h, ctypes.byref(t)) == 0
        for k, v in kw.items():
            setattr(t, k, v)
        assert self.L.bto_set_tuning(h, ctypes.byref(t)) == 0

    @staticmethod
    def grids(N, at=1 << 51):
        return (ctypes.c_void_p * (N + 1))(*[at + (q << 32) for q in range(N + 1)])

    @staticmethod
    def times(N):
        return (ctypes.c_double * (N + 1))(*range(N + 1))

    def logged(self, call):
        """(status, log lines) of a call."""
        self.f.fake_clear()
        rc = call()
        return rc, self.f.fake_log().decode().splitlines()

    def advect(self, h, N, dtype=0, flags=0):
        return self.logged(lambda: self.L.bto_advect_interval(h, self.grids(N), self.times(N), N, dtype, flags, STREAM))

    def adjoint(self, h, N, k, grads=False):
        return self.logged(lambda: self.L.bto_adjoint_interval(
            h, self.grids(N), self.times(N), N, 0, 0, 1 << 50, 1, 1 << 50,
            self.grids(N, 1 << 52) if grads else None, None, k, STREAM))


def launches(log):
    return [ln for ln in log if ln.startswith("launch")]


def memory_calls(log):
    return [ln for ln in log if re.match("malloc|free|sync|memset|copy", ln)]


def case_adjoint_keeps_the_tape_it_got(grads):
    """The first call settles for a shorter tape; the next ones use it without
    asking again."""
    host = Host(sys.argv[1])
    h = host.create((27, 22, 17), 400_000)
    host.seed(h, 400_000)
    if grads:  # the records are in place; the scratch of one position per seed has to grow
        assert host.adjoint(h, 50, 50, True)[0] == 0
    host.f.fake_memory(0 if grads else 640 << 20)
    rc, first = host.adjoint(h, 50, 10, grads)
    assert rc == 0, rc
    tried = [ln for ln in first if ln.startswith("malloc")]
    assert any("failed" in ln for ln in tried) and "ok" in tried[-1], first
    for _ in range(2):
        rc, again = host.adjoint(h, 50, 10, grads)
        assert rc == 0
        assert not memory_calls(again), again
        assert launches(again) == launches(first)


def case_adjoint_recovers(_):
    host = Host(sys.argv[1])
    h = host.create((27, 22, 17), 400_000)
    host.seed(h, 360_000)
    host.f.fake_memory(1 << 20)
    assert host.adjoint(h, 50, 10)[0] == host.lib.BTO_ENOMEM
    host.f.fake_memory(4 << 30)
    rc, log = host.adjoint(h, 50, 10)
    assert rc == 0 and [ln for ln in log if ln.startswith("malloc")] == [log[0]] and "ok" in log[0], log
    assert host.L.bto_destroy(h) == 0 and host.f.fake_blocks() == 0


def case_rebin_buffers(_):
    """A re-sort whose second buffer cannot be had leaves nothing behind; the
    next one gets both and clears the bin counts on the caller's stream, ahead
    of the kernel that counts into them (the null stream would not be ordered
    with a stream created non-blocking)."""
    host = Host(sys.argv[1])
    h = host.create((64, 64, 64), 40_000)
    host.tune(h, rebin_every=1)
    host.seed(h, 40_000)
    held = host.f.fake_blocks()
    host.f.fake_fail(1)
    rc, log = host.advect(h, 4)
    assert rc == host.lib.BTO_ENOMEM and host.f.fake_blocks() == held, (rc, log)
    rc, log = host.advect(h, 4)
    assert rc == 0 and len([ln for ln in log if ln.startswith("malloc") and "ok" in ln]) == 2, log
    assert not [ln for ln in log if ln.startswith("memset")], log
    kernels = launches(log)
    assert all(ln.endswith("stream 0x7") for ln in kernels), log
    fill = next(i for i, ln in enumerate(kernels) if "tile_fill_kernel" in ln)
    assert fill < next(i for i, ln in enumerate(kernels) if "rebin_count_kernel" in ln)
    assert len([ln for ln in kernels if "tile_fill_kernel" in ln]) == 1
    assert host.L.bto_destroy(h) == 0 and host.f.fake_blocks() == 0


def case_launches_of_many_particles(lanes):
    """2.15 thousand million particles, 215 GB of state: with two lanes each a
    launch of one batch per workgroup would pass 2^32 threads."""
    host = Host(sys.argv[1])
    P = 2_150_000_000
    h = host.create((64, 64, 64), P)
    host.tune(h, lanes_per_particle=lanes)
    host.seed(h, P)
    rc, log = host.advect(h, 2)
    assert rc == 0, (rc, log)
    blocks, threads = map(int, re.search(r"advect_kernel.* grid (\d+) 1 block (\d+)", log[-1]).groups())
    assert 2 ** 31 < blocks * threads < 2 ** 32


def case_pairs_of_workgroups(_):
    """Which FP32 launches keep all but two workgroups off a CU (by LDS they do
    not use): lattices of stride 2, launches of `steps`, re-sorted or not."""
    host = Host(sys.argv[1])
    for n, steps, rebin, pair in [
            (112, 24, 0, False), (112, 24, 24, False), (128, 8, 0, False), (128, 12, 0, True), (132, 32, 0, False),
            (146, 24, 0, False), (146, 31, 0, True), (146, 2, 2, False), (150, 2, 2, True), (150, 2, 0, False), (174, 8, 0, False),
            (174, 24, 0, True), (256, 2, 0, False), (256, 5, 0, False), (256, 6, 0, True), (256, 2, 2, True),
            (256, 1, 1, False)]:
        h = host.create((n, n, n), (n // 2) ** 3)
        host.tune(h, rebin_every=rebin, steps_per_launch=32)
        host.seed(h, (n // 2) ** 3)
        rc, log = host.advect(h, steps)
        assert rc == 0
        lds = [int(re.search(r" lds (\d+)", ln).group(1)) for ln in launches(log) if "advect_kernel" in ln]
        assert len(lds) == 1 and (lds[0] > 0) == pair, (n, steps, rebin, log)
        assert host.L.bto_destroy(h) == 0


def case_two_lanes_loop_in_long_launches(_):
    """Two lanes per particle: a batch per workgroup, but from 20 steps on a grid
    that fills the chip once (four workgroups on each of 256 CUs here)."""
    host = Host(sys.argv[1])
    h = host.create((200, 200, 200), 10 ** 6)
    host.tune(h, lanes_per_particle=2, steps_per_launch=24)
    for steps, dtype, blocks in [(1, 0, None), (19, 0, None), (20, 0, 1024), (48, 0, 1024), (20, 1, None)]:
        host.seed(h, 10 ** 6)
        rc, log = host.advect(h, steps, dtype)
        grids = [int(re.search(r" grid (\d+)", ln).group(1)) for ln in launches(log) if "advect_kernel" in ln]
        batch = 256 if dtype else 128
        want = blocks or 8 * -(-125_000 // batch)
        assert rc == 0 and grids == [want] * len(grids), (steps, dtype, grids)


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    from paper_2004_02003_amd import _lib

    if not os.path.exists(_lib.LIB_PATH):
        pytest.skip("libbto.so not built")
    out = str(tmp_path_factory.mktemp("fake") / "fake_hip.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-I", os.path.join(ROCM, "include"),
                    os.path.join(HERE, "fake_hip.c"), "-o", out], check=True)
    return out


@pytest.mark.parametrize("case,arg", [("adjoint_keeps_the_tape_it_got", 0), ("adjoint_keeps_the_tape_it_got", 1),
                                      ("adjoint_recovers", 0), ("rebin_buffers", 0), ("launches_of_many_particles", 1),
                                      ("launches_of_many_particles", 2), ("pairs_of_workgroups", 0),
                                      ("two_lanes_loop_in_long_launches", 0)])
def test_host(fake, case, arg):
    r = subprocess.run([sys.executable, os.path.abspath(__file__), fake, case, str(arg)], capture_output=True,
                       text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


if __name__ == "__main__":
    globals()["case_" + sys.argv[2]](int(sys.argv[3]))
