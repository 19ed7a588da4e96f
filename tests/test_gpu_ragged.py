"""Streams of different row counts share launches: a ragged batch against each
of its streams alone, bit for bit, at the edges of the grouping (empty streams
first, inside and last, 64 and 65 streams, a grid just within and just beyond
twice the rows) and of the tiles (one row, one frame, partial frames)."""
import numpy as np
import pytest
import torch

import synth
from paper_2506_15745_amd import ipv
from tests import parity as P

pytestmark = pytest.mark.gpu

P4 = 16  # rows a frame of the 4x4 grid
#  L, H, D, counts, budget, r, capacity, dtype, mode, pooling
CASES = {
    "empty-first-inside-last": (2, 3, 128, (0, 90, 0, 0, 64, 80, 0), 48, 2, 96, "bf16", 0, None),
    "one-row-streams": (1, 1, 32, (1, 2, 1, 3, 2), 1, 1, 5, "f32", 0, None),
    "64-streams": (1, 2, 64, tuple(64 + b % 7 for b in range(64)), 40, 1, 71, "bf16", 0, (0.3, 0.5, 0.7)),
    "65-streams": (1, 1, 64, tuple(64 + b % 7 for b in range(65)), 40, 1, 71, "f32", ipv.HEAD_SHARED, None),
    "grid-twice-the-rows": (1, 2, 128, (96, 32, 32, 32, 160), 32, 1, 160, "bf16", 0, None),
    "adjacent-pooled": (2, 2, 128, (96, 70, 81), 50, 2, 97, "bf16", ipv.TAR_ADJACENT, (0.3, 0.5, 0.7)),
    "adjacent-shared-f32": (3, 3, 256, (49, 80, 64, 64), 40, 2, 80, "f32", ipv.TAR_ADJACENT | ipv.HEAD_SHARED, None),
    "uniform": (2, 2, 32, (96, 0, 70, 81), 50, 2, 97, "bf16", ipv.UNIFORM_SELECT, None),
    # several rows a selection thread, several compaction chunks, more slices than XCDs
    "long": (3, 3, 64, (4500, 3000, 6000, 2600), 2000, 3, 6001, "bf16", 0, (0.3, 0.5, 0.7)),
}


@pytest.mark.parametrize("name", CASES)
def test_ragged_batch_equals_its_streams(name):
    L, H, D, counts, budget, r, S, dtype, mode, tau = CASES[name]
    B = len(counts)
    print(name, counts[:8], flush=True)
    sd, kind, bits = (synth.BF16, "bf16", torch.int16) if dtype == "bf16" else (synth.F32, "raw", torch.int32)
    sts = [synth.fresh_cache(400 + b, L, H, S, D, 4, 4, max(n, 1), sd, synth.RhoSpec(0.0, 0.95, 0.2), (0.1, 0.55, 1.0))
           for b, n in enumerate(counts)]

    def fresh():
        st = lambda a: P.to_device(np.ascontiguousarray(np.stack([getattr(x, a) for x in sts])),  # noqa: E731
                                   kind if a in "KV" else "raw")
        K, V = st("K"), st("V")
        comp = ipv.Compressor(K, 4, 4, budget)
        for t in (comp.tar, comp.van, comp.keep_idx):
            t.fill_(-7)
        return K, V, st("frame_idx"), st("patch_idx"), comp

    def results(K, V, fr, pa, comp):
        return [K.view(bits), V.view(bits), fr, pa, comp.keep_idx, comp.tar.view(torch.int32), comp.van.view(torch.int32)]

    def whole(K, V, fr, pa, comp, n):
        comp.compress(K, V, fr, pa, n, 0.5, r, tau, mode=mode)

    def steps(K, V, fr, pa, comp, n):
        pool = torch.full((B, L), -7, dtype=torch.int32, device="cuda:0")
        ipv.ipv_tar_scores(K, fr, pa, n, r, comp.tar, comp.ws, 4, 4, mode=mode)
        ipv.ipv_van_scores(V, fr, pa, n, tau, comp.van, pool, comp.ws, 4, 4)
        ipv.ipv_select(comp.tar, comp.van, fr, n, budget, 0.5, r, comp.keep_idx, comp.ws, 4, 4, head_dim=D,
                       dtype=ipv.BF16 if dtype == "bf16" else ipv.F32, mode=mode)
        ipv.ipv_compact(K, V, fr, pa, n, comp.keep_idx, budget, comp.ws, 4, 4)
        return [pool]

    for call in (whole, steps):
        one, many = fresh(), fresh()
        got = call(*many, list(counts)) or []
        want = None
        for b, n in enumerate(counts):
            pools = call(*one, [n if i == b else 0 for i in range(B)]) or []
            want = [w.clone() for w in pools] if want is None else [torch.where(p != -7, p, w) for p, w in zip(pools, want)]
        torch.cuda.synchronize()
        # one row of budget does not hold a window of two: reported alike
        assert one[4].device_errors() == many[4].device_errors() == (ipv.DEV_RECENT_OVER if budget == 1 else 0)
        for x, y in zip(results(*one) + want, results(*many) + got):
            assert torch.equal(x, y)
