"""Passes of small slices, which go out as one launch, against the step entry
points (launches of their own), bit for bit: the edges of the rule (256 and
257 rows, 64 KB of keys and just beyond, 256 and 257 slices, frames of 24 KB and
beyond, windows of 32 and 33 frames), every row size, one row, ragged batches, a window of the whole cache, reversed stages."""
import numpy as np
import pytest
import torch

import synth
from paper_2506_15745_amd import ipv
from tests import parity as P

pytestmark = pytest.mark.gpu

#  counts, L, H, D, grid, budget, r, capacity, dtype, mode
CASES = {
    "256-rows": ((256,), 1, 2, 128, (4, 4), 128, 2, 256, "bf16", 0),
    "257-rows": ((257,), 1, 2, 64, (4, 4), 128, 2, 257, "bf16", 0),
    "64KB": ((128,), 2, 2, 128, (5, 7), 70, 2, 129, "f32", 0),
    "beyond-64KB": ((129,), 2, 2, 128, (5, 7), 70, 2, 129, "f32", 0),
    "256-slices": ((64,), 64, 4, 32, (4, 4), 33, 2, 64, "bf16", 0),
    "257-slices": ((64,), 257, 1, 32, (4, 4), 33, 2, 64, "bf16", 0),
    "one-row": ((1,), 1, 1, 64, (3, 3), 1, 1, 3, "f32", 0),
    "whole-window": ((120,), 2, 2, 256, (3, 5), 120, 8, 120, "bf16", ipv.TAR_REVERSE),
    "wide-rows": ((64,), 1, 3, 256, (2, 3), 32, 3, 67, "f32", ipv.VAN_REVERSE),
    "long-window": ((250,), 1, 2, 32, (1, 5), 200, 33, 250, "bf16", 0),
    # the most LDS that the rule admits: 256 positions a round, 32 frames a position
    "most-lds": ((250,), 1, 2, 32, (1, 5), 200, 32, 250, "bf16", 0),
    "24KB-frames": ((256,), 1, 2, 64, (8, 12), 200, 1, 256, "f32", 0),
    "beyond-24KB-frames": ((256,), 1, 2, 64, (1, 97), 200, 1, 256, "f32", 0),
    "ragged": ((90, 0, 250, 131, 90), 2, 2, 64, (6, 7), 88, 2, 251, "bf16", ipv.TAR_REVERSE | ipv.VAN_REVERSE),
    "two-table-rounds": ((240,), 1, 2, 32, (10, 15), 239, 1, 240, "f32", ipv.TAR_REVERSE),
    "wide-grid": ((240,), 1, 2, 32, (8, 15), 239, 1, 240, "f32", 0),
}


@pytest.mark.parametrize("name", CASES)
def test_one_launch_equals_the_steps(name):
    counts, L, H, D, (gh, gw), budget, r, S, dtype, mode = CASES[name]
    print(name, flush=True)
    sd, kind, bits = (synth.BF16, "bf16", torch.int16) if dtype == "bf16" else (synth.F32, "raw", torch.int32)
    sts = [synth.fresh_cache(600 + b, L, H, S, D, gh, gw, max(n, 1), sd, synth.RhoSpec(0.0, 0.95, 0.2), (0.5,))
           for b, n in enumerate(counts)]

    def fresh():
        st = lambda a: P.to_device(np.ascontiguousarray(np.stack([getattr(x, a) for x in sts])),  # noqa: E731
                                   kind if a in "KV" else "raw")
        K, V = st("K"), st("V")
        return K, V, st("frame_idx"), st("patch_idx"), ipv.Compressor(K, gh, gw, budget)

    n = list(counts)
    K1, V1, f1, p1, c1 = fresh()
    c1.compress(K1, V1, f1, p1, n, 0.5, r, mode=mode)
    K2, V2, f2, p2, c2 = fresh()
    ipv.ipv_tar_scores(K2, f2, p2, n, r, c2.tar, c2.ws, gh, gw, mode=mode)
    ipv.ipv_van_scores(V2, f2, p2, n, None, c2.van, None, c2.ws, gh, gw)
    ipv.ipv_select(c2.tar, c2.van, f2, n, budget, 0.5, r, c2.keep_idx, c2.ws, gh, gw, head_dim=D,
                   dtype=ipv.BF16 if dtype == "bf16" else ipv.F32, mode=mode)
    ipv.ipv_compact(K2, V2, f2, p2, n, c2.keep_idx, budget, c2.ws, gh, gw)
    torch.cuda.synchronize()
    assert c1.device_errors() == 0 and c2.device_errors() == 0
    for x, y in ((K1.view(bits), K2.view(bits)), (V1.view(bits), V2.view(bits)), (f1, f2), (p1, p2),
                 (c1.keep_idx, c2.keep_idx), (c1.tar.view(torch.int32), c2.tar.view(torch.int32)),
                 (c1.van.view(torch.int32), c2.van.view(torch.int32))):
        assert torch.equal(x, y)


@pytest.mark.parametrize("bad", ["frames", "patch", "window"])
def test_broken_metadata_is_reported_alike(bad):
    """Metadata that breaks the cache's invariants: the device error word and the rows left are those of the steps."""
    L, H, D, S, budget, r = 1, 2, 64, 128, 64, 1
    st = synth.fresh_cache(77, L, H, S, D, 4, 4, S, synth.F32, synth.RhoSpec(0.0, 0.95), (0.5,))
    out = []
    for steps in (False, True):
        K, V, fr, pa = (P.to_device(np.ascontiguousarray(getattr(st, a)[None])) for a in ("K", "V", "frame_idx", "patch_idx"))
        if bad == "frames":
            fr[0, 0, 1, 20] = 7
        elif bad == "patch":
            pa[0, 0, 0, 5] = 16
        else:
            fr[:] = 3
        c = ipv.Compressor(K, 4, 4, budget)
        if steps:
            ipv.ipv_tar_scores(K, fr, pa, S, r, c.tar, c.ws, 4, 4)
            ipv.ipv_van_scores(V, fr, pa, S, None, c.van, None, c.ws, 4, 4)
            ipv.ipv_select(c.tar, c.van, fr, S, budget, 0.5, r, c.keep_idx, c.ws, 4, 4, head_dim=D, dtype=ipv.F32)
            ipv.ipv_compact(K, V, fr, pa, S, c.keep_idx, budget, c.ws, 4, 4)
        else:
            c.compress(K, V, fr, pa, S, 0.5, r)
        torch.cuda.synchronize()
        out.append((c.device_errors(), c.keep_idx.clone(), K.clone(), V.clone(), fr, pa))
    print(bad, "error word", out[0][0], flush=True)
    assert out[0][0] == out[1][0] != 0
    for x, y in zip(out[0][1:], out[1][1:]):
        assert torch.equal(x, y)
