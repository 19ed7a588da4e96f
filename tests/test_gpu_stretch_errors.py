"""Entry rows that break the cache's invariants, and NaN, through ipv_ckv_stream:
the device error word, and what is left of every slice, are those of the loop
step by step (ipv_ckv_step), in every kind of pass that the call can take."""
import numpy as np
import pytest
import torch

import synth
from paper_2506_15745_amd import ipv
from tests import parity as P

pytestmark = pytest.mark.gpu

#  L, H, D, grid, entry rows, frames, cap, budget, r, capacity, dtype, mode, pooling
PATHS = {
    "small": (1, 2, 64, (4, 4), 48, 14, 128, 64, 1, 144, "f32", 0, None),
    "small-scanned-window": (1, 2, 64, (4, 4), 48, 14, 128, 112, 3, 144, "bf16", 0, None),
    "next-launch-beside": (2, 2, 128, (9, 13), 351, 40, 1700, 800, 3, 1819, "bf16", 0, None),
    "scanned-window": (1, 2, 128, (7, 7), 490, 30, 700, 650, 4, 751, "bf16", 0, None),
    "head-shared": (2, 3, 64, (9, 13), 351, 40, 1700, 800, 3, 1819, "f32", ipv.HEAD_SHARED, None),
    "adjacent": (2, 2, 128, (9, 13), 351, 40, 1700, 800, 3, 1819, "bf16", ipv.TAR_ADJACENT, None),
    "adjacent-shared": (1, 4, 64, (9, 13), 351, 40, 1700, 800, 3, 1819, "f32", ipv.TAR_ADJACENT | ipv.HEAD_SHARED, None),
    "pooled": (2, 2, 64, (9, 13), 351, 40, 1700, 800, 3, 1819, "bf16", 0, (0.3, 0.5, 0.7)),
    "uniform": (2, 2, 64, (9, 13), 351, 40, 1700, 800, 3, 1819, "bf16", ipv.UNIFORM_SELECT, None),
    "in-the-cache": (2, 2, 128, (9, 13), 1638, 3, 1700, 800, 3, 1819, "bf16", 0, None),
}
FRAMES, PATCH, NAN = ipv.DEV_BAD_FRAMES, ipv.DEV_BAD_PATCH, ipv.DEV_NAN


def decreasing(K, V, fr, pa, p):
    fr[0, 0, 1, 20] = 7


def far_ahead(K, V, fr, pa, p):
    fr[0, 0, 0, 21] = 1000000


def outside(K, V, fr, pa, p):
    pa[0, 0, 0, 5] = p
    pa[0, 0, 1, 6] = -3


def twice(K, V, fr, pa, p):
    pa[0, 0, 0, 3] = pa[0, 0, 0, 4].item()


def heads_apart(K, V, fr, pa, p):
    fr[0, 0, 1] -= 1


def nan_key(K, V, fr, pa, p):
    K[0, 0, 0, 7] = float("nan")


def nan_value(K, V, fr, pa, p):
    V[0, 0, 0, 9, 3] = float("nan")


def errors_of(breaks, mode, tau):
    """The bits that must be raised; None: this mode does not look at what is broken."""
    scored = not mode & ipv.UNIFORM_SELECT
    if breaks in (decreasing, far_ahead):
        return FRAMES
    if breaks is outside:
        return PATCH if scored else None
    if breaks is twice:
        return FRAMES if mode & ipv.TAR_ADJACENT else None
    if breaks is heads_apart:
        return FRAMES if mode & ipv.HEAD_SHARED else None
    return NAN if scored and not tau else None


BREAKS = (decreasing, far_ahead, outside, twice, heads_apart, nan_key, nan_value)
CASES = [(path, f) for path, c in PATHS.items() for f in BREAKS if errors_of(f, c[11], c[12])]


@pytest.mark.parametrize("path,breaks", CASES, ids=lambda x: getattr(x, "__name__", x))
def test_broken_entry_rows_are_reported_as_step_by_step(path, breaks):
    L, H, D, (gh, gw), entry, frames, cap, budget, r, S, dtype, mode, tau = PATHS[path]
    bits = errors_of(breaks, mode, tau)
    print(path, breaks.__name__, flush=True)
    p = gh * gw
    sd, kind, word = (synth.BF16, "bf16", torch.int16) if dtype == "bf16" else (synth.F32, "raw", torch.int32)
    sigma = (0.1, 0.35) if tau else (0.5,)
    src = synth.fresh_cache(31, L, H, frames * p, D, gh, gw, frames * p, sd, synth.RhoSpec(0.0, 0.95, 0.2), sigma)
    old = synth.fresh_cache(32, L, H, S, D, gh, gw, entry, sd, synth.RhoSpec(0.0, 0.95), sigma)
    by_frame = lambda a: P.to_device(np.ascontiguousarray(np.stack(  # noqa: E731
        [getattr(src, a)[None, :, :, f * p:(f + 1) * p] for f in range(frames)])), kind)
    fK, fV = by_frame("K"), by_frame("V")
    out = []
    for stream in (False, True):
        K, V = (P.to_device(np.ascontiguousarray(getattr(old, a)[None]), kind) for a in "KV")
        fr, pa = (P.to_device(np.ascontiguousarray(getattr(old, a)[None])) for a in ("frame_idx", "patch_idx"))
        fr -= 1000
        breaks(K, V, fr, pa, p)
        c = ipv.Compressor(K, gh, gw, budget)
        args = (cap, budget, 0.5, r, tau, c.tar, c.van, c.keep_idx, c.ws, gh, gw)
        if stream:
            n, passes = ipv.ipv_ckv_stream(K, V, fr, pa, entry, fK, fV, 0, *args, mode=mode)
        else:
            n, passes = entry, 0
            for f in range(frames):
                n, fired = ipv.ipv_ckv_step(K, V, fr, pa, n, fK[f], fV[f], f, 0, *args, mode=mode)
                passes += int(fired)
        torch.cuda.synchronize()
        out.append((c.device_errors(), n, passes, c.keep_idx.view(L, H, budget),
                    [t[0, :, :, :n] for t in (K.view(word), V.view(word), fr, pa)]))
    (e1, n1, ps1, keep1, rows1), (e2, n2, ps2, keep2, rows2) = out
    assert e1 == e2 and e1 & bits == bits and (n1, ps1) == (n2, ps2) and ps1 >= 1
    for l in range(L):
        for h in range(H):
            if bits == NAN and l == 0 and (h == 0 or mode & ipv.HEAD_SHARED):
                k = keep2[l, h]  # a NaN's rank is unspecified: the keep set is still one
                assert k[0] >= 0 and bool((k[1:] > k[:-1]).all())
                continue
            assert torch.equal(keep1[l, h], keep2[l, h])
            for x, y in zip(rows1, rows2):
                assert torch.equal(x[l, h], y[l, h])
