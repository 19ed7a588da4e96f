"""Selection of slices beyond 32 rows a thread: the row counts at which the
rows held by a thread change (36, 48 and 64), aligned and unaligned
capacities, per slice and head-shared, against the oracle's keep sets."""
import numpy as np
import pytest
import torch

import oracle
from paper_2506_15745_amd import ipv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [0, ipv.HEAD_SHARED])
@pytest.mark.parametrize("n,S", [(32768, 32768), (32769, 32769), (32928, 32928), (36864, 36866), (36865, 36868),
                                 (49152, 49152), (49153, 49155), (65536, 65536)])
def test_long_slices(n, S, mode):
    print("rows", n, "capacity", S, "mode", mode, flush=True)
    rng = np.random.default_rng(n)
    H, budget, r, gh = 2, n // 2 + 3, 2, 14
    # few distinct values: ties run through every digit
    tar = -rng.choice(np.linspace(0.1, 0.99, 5000, dtype=np.float32), (1, 1, H, S)).astype(np.float32)
    van = rng.choice(np.linspace(0.5, 30, 3000, dtype=np.float32), (1, 1, H, S)).astype(np.float32)
    fr = np.broadcast_to((np.arange(S) // (gh * gh)).astype(np.int32), (1, 1, H, S)).copy()
    dev = [torch.from_numpy(x).to("cuda:0") for x in (tar, van, fr)]
    keep = torch.zeros((1, 1, H, budget), dtype=torch.int32, device="cuda:0")
    ws = ipv.alloc_workspace(ipv.Shape(1, 1, H, 32, S, gh, gh, ipv.F32), "cuda:0")
    ipv.ipv_select(*dev, n, budget, 0.4, r, keep, ws, gh, gh, head_dim=32, dtype=ipv.F32, mode=mode)
    assert ipv.ipv_read_device_errors(ws) == 0
    want = oracle.select(tar, van, fr, n, budget, 0.4, r, mode=mode).keep_idx
    assert np.array_equal(want, keep.cpu().numpy())
