"""The selection at the edges of its thread layouts, with scores that are distinct
(the search ends early), few-valued (ties at every threshold) and all equal,
against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2606_03928_amd import vase

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.fixture(autouse=True)
def _lib(gpu_lib):
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("K,B,Nv", [
    (1, 1, 0), (2, 1, 1), (63, 20, 43), (255, 1, 254), (256, 100, 60), (257, 16, 1), (511, 511, 0),
    (512, 64, 32), (513, 64, 32), (2048, 128, 128), (2049, 1, 5), (6145, 256, 300), (8192, 128, 8064),
])
def test_select_layouts(K, B, Nv):
    rng = np.random.default_rng(K + B)
    n = 6
    attn, vr = rng.random((n, K), np.float32), rng.random((n, K), np.float32) + 1
    attn[1], vr[1] = rng.integers(1, 4, K), rng.integers(1, 3, K)
    attn[2], vr[2] = 0.5, 2.0
    attn[3] = 0.0
    attn[4], vr[4] = attn[4] * np.float32(2.0 ** -60), rng.integers(0, 2, K)
    a, r = torch.from_numpy(attn).to(DEV), torch.from_numpy(vr).to(DEV)
    for det in (0, vase.DETERMINISTIC):
        src = vase.select(a, r, K, B, Nv, seed=9, round=4, flags=det)
        want = oracle.select(attn, vr, K, B, Nv, 9, 4, flags=det)
        np.testing.assert_array_equal(src.cpu().numpy(), want)
