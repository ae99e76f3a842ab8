"""The lattice rebuild at the edges of its kernels (lines around half a
wavefront, two chunks and the longest; pieces of eight entries; workgroups of
64 lines), and the accuracy metric called by more threads at once than it keeps
scratch sets for."""

import sys
import threading

import numpy as np
import pytest

from oracle import reconstruct as orc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2004_02003_amd import _lib

    _lib.load()


def _t(a):
    import torch

    return torch.as_tensor(np.ascontiguousarray(a), device="cuda")


@pytest.mark.parametrize("known", [0.03, 0.7])
@pytest.mark.parametrize("m", [(31, 9, 70), (32, 8, 9), (33, 65, 7), (128, 17, 16), (129, 3, 25), (1024, 2, 3),
                               (65, 1024, 1)])
def test_rebuild_at_the_kernels_edges(m, known):
    from paper_2004_02003_amd import posthoc

    rng = np.random.default_rng(sum(m))
    P = int(np.prod(m))
    end = rng.normal(size=(P, 3)) * 10
    flag = np.where(rng.random(P) < known, 0, 1).astype(np.uint8)
    print(f"[gpu-case] rebuild {m} {known}", file=sys.stderr, flush=True)
    g_end = _t(end)
    st = posthoc.reconstruct_lattice(g_end, _t(flag), m)
    o_end, o_st = orc.reconstruct(end, flag == 0, m)
    assert np.array_equal(st.cpu().numpy(), o_st)
    assert np.array_equal(g_end.cpu().numpy(), o_end, equal_nan=True)


def test_metric_from_many_threads():
    import torch
    from paper_2004_02003_amd import posthoc

    rng = np.random.default_rng(5)
    inputs, want = [], []
    for k in range(12):
        P = 20_000 + 7 * k
        b = rng.normal(size=(P, 3))
        m = b + rng.normal(size=(P, 3)) * 0.01 * (k + 1)
        bs = rng.choice([0, 1, 2], size=P).astype(np.uint8)
        mf = rng.choice([0, 1], size=P, p=[0.9, 0.1]).astype(np.uint8)
        inputs.append([_t(v) for v in (b, bs, m, mf)])
        want.append(posthoc.flowmap_error(*inputs[-1]))
        o = orc.flowmap_error(b, bs, m, mf, cell=1.0)
        assert want[-1]["n"] == o["n"] and want[-1]["mean_l2"] == pytest.approx(o["mean_l2"], rel=1e-12)
    torch.cuda.synchronize()
    got = [[] for _ in inputs]
    print("[gpu-case] metric, 12 threads", file=sys.stderr, flush=True)

    def work(k):
        s = torch.cuda.Stream()
        for _ in range(20):
            got[k].append(posthoc.flowmap_error(*inputs[k], stream=s))

    ts = [threading.Thread(target=work, args=(k,)) for k in range(len(inputs))]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for k, w in enumerate(want):
        assert len(got[k]) == 20 and all(r == w for r in got[k]), k
