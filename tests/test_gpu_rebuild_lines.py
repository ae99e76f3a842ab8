"""The lattice rebuild's y and z passes on both sides of their rule (fewer than
4,096 lines: a wavefront per line; otherwise 64 lines per workgroup, a lane per
line in pieces of eight entries), bit for bit against the oracle."""

import sys

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


# few lines: short and long (chunks of 64 entries, two and more), single ones;
# many: pieces cut short, the last workgroup of 64 lines not full, the longest
@pytest.mark.parametrize("known", [0.03, 0.7])
@pytest.mark.parametrize("m", [(4, 1000, 4), (3, 130, 90), (1, 64, 65), (1, 1, 1024), (2, 1024, 200), (63, 9, 65),
                               (64, 9, 64), (64, 65, 66), (1024, 9, 4), (300, 7, 70)])
def test_rebuild_by_number_of_lines(m, known):
    import torch
    from paper_2004_02003_amd import posthoc

    rng = np.random.default_rng(sum(m))
    P = int(np.prod(m))
    end = rng.normal(size=(P, 3)) * 10
    flag = np.where(rng.random(P) < known, 0, 1).astype(np.uint8)
    print(f"[gpu-case] rebuild {m} {known}", file=sys.stderr, flush=True)
    g_end = torch.as_tensor(end, device="cuda").clone()
    st = posthoc.reconstruct_lattice(g_end, torch.as_tensor(flag, device="cuda"), m)
    o_end, o_st = orc.reconstruct(end, flag == 0, m)
    assert np.array_equal(st.cpu().numpy(), o_st)
    assert np.array_equal(g_end.cpu().numpy(), o_end, equal_nan=True)
