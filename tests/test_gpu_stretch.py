"""Passes over resident frames (ipv_ckv_stream) against the loop that appends
every frame and compacts at every pass (ipv_ckv_step): caches, metadata and
row counts, and the last pass's scores and keep sets, bit for bit."""
import numpy as np
import pytest
import torch

import synth
from paper_2506_15745_amd import ipv
from tests import parity as P

pytestmark = pytest.mark.gpu

#  L, H, D, grid, rows a frame, entry rows per stream, frames, cap, budget, r, capacity, dtype, mode, pooling
CASES = {
    # entry rows and budget over several 512-row chunks: the gather's waits
    "entry-chunks": (2, 2, 128, (7, 7), 49, (1100, 1100), 60, 2000, 1600, 4, 2052, "bf16", 0, None),
    # every pass brings one or two frames: the window reaches into old rows, places read through the index
    "few-new-frames": (1, 2, 64, (5, 5), 25, (0, 75), 40, 301, 270, 3, 333, "f32", 0, None),
    # frames of fewer rows than the grid; streams with passes at different frames; one that never fires
    "partial-frames": (2, 1, 128, (6, 7), 31, (0, 310, 42), 37, 700, 400, 4, 731, "bf16", 0, None),
    # streams that enter with different counts (none, too) and are alike from a later pass on, the last one's gather included
    "entries-join": (2, 2, 128, (7, 7), 49, (0, 1760, 1775), 60, 2000, 1600, 4, 2052, "bf16", 0, None),
    "entries-join-adjacent": (1, 2, 64, (7, 7), 49, (1775, 0, 1760), 70, 2000, 1600, 2, 2051, "f32", ipv.TAR_ADJACENT, None),
    "pooled": (4, 2, 64, (4, 4), 16, (0, 64), 30, 130, 70, 2, 146, "bf16", ipv.VAN_REVERSE, (0.3, 0.5, 0.7)),
    "adjacent": (2, 2, 128, (9, 13), 117, (234,), 40, 1300, 700, 3, 1417, "bf16", ipv.TAR_ADJACENT, None),
    "adjacent-shared-f32": (2, 4, 256, (3, 5), 15, (15,), 40, 150, 91, 2, 165, "f32",
                            ipv.TAR_ADJACENT | ipv.HEAD_SHARED, None),
    "adjacent-pooled": (2, 2, 32, (4, 4), 16, (0,), 40, 130, 70, 2, 146, "bf16", ipv.TAR_ADJACENT, (0.3, 0.5, 0.7)),
    "uniform": (2, 2, 128, (7, 7), 49, (0, 600), 60, 1300, 700, 2, 1349, "bf16", ipv.UNIFORM_SELECT, None),
    "uniform-shared": (2, 2, 64, (7, 7), 49, (98,), 60, 1300, 700, 2, 1349, "f32",
                       ipv.UNIFORM_SELECT | ipv.HEAD_SHARED, None),
    # budget equal to the cap: one pass, at the last frame
    "budget-is-cap": (1, 1, 32, (4, 4), 16, (3,), 8, 128, 128, 2, 144, "bf16", 0, None),
    # more rows than 32 a selection thread, keep set over several stages
    "long": (1, 1, 32, (14, 14), 196, (0,), 180, 33000, 30000, 5, 33196, "bf16", 0, None),
    # the work of the next pass beside a selection: 4, 8, 12 and 16 rows a selection thread, odd capacities, windows as
    # long as the new frames and longer (nothing ahead), the largest number of selections it is done for and one more,
    # frames narrower than the grid, rows left in the cache above the budget (not in the first pass then)
    "ahead-4-rows": (2, 2, 128, (9, 13), 117, (0,), 60, 1700, 800, 3, 1819, "bf16", 0, None),
    "ahead-8-rows": (1, 3, 64, (14, 14), 196, (0,), 90, 5000, 2500, 4, 5199, "f32", 0, None),
    "ahead-12-rows": (1, 2, 32, (14, 14), 196, (0, 0), 120, 10000, 5000, 4, 10196, "bf16", ipv.TAR_REVERSE, None),
    "ahead-16-rows": (1, 2, 32, (14, 14), 196, (0,), 150, 15000, 8000, 4, 15197, "f32", ipv.HEAD_SHARED, None),
    "ahead-window-is-the-new-frames": (2, 2, 256, (5, 5), 25, (0,), 60, 500, 400, 4, 525, "bf16", 0, None),
    "ahead-176-selections": (88, 2, 64, (6, 7), 42, (0,), 40, 600, 300, 2, 642, "bf16", 0, None),
    "ahead-185-selections": (185, 1, 32, (6, 7), 42, (0,), 40, 600, 300, 2, 642, "bf16", 0, None),
    # TaR tiles of frames, 4 and 8 slices in turn, slices left over
    "4-slices-in-turn": (113, 2, 32, (5, 5), 25, (0,), 24, 300, 200, 2, 325, "bf16", 0, None),
    "8-slices-in-turn": (449, 1, 32, (5, 5), 25, (0,), 24, 300, 200, 2, 325, "bf16", 0, None),
    "ahead-64-selections-of-1KB-rows": (32, 2, 256, (6, 7), 42, (0,), 20, 400, 200, 2, 442, "f32", 0, None),
    "ahead-narrow-frames": (1, 2, 64, (8, 8), 41, (20, 20), 60, 900, 400, 2, 943, "f32", ipv.VAN_REVERSE, None),
    "ahead-rows-above-the-budget": (1, 2, 128, (7, 7), 49, (900,), 80, 1000, 500, 2, 1049, "bf16", 0, None),
    # the first pass has 260 rows, the later ones 250 and go out as one launch each
    "ahead-then-small": (1, 2, 64, (4, 5), 20, (0,), 40, 250, 230, 2, 270, "bf16", 0, None),
    # passes of one launch each: the most LDS that its rule admits, windows scanned; two rounds of the table
    "small-most-lds": (1, 2, 32, (1, 5), 5, (0, 100), 60, 240, 190, 32, 250, "bf16", 0, None),
    "small-32KB-frames": (1, 2, 128, (8, 16), 40, (0, 60), 30, 200, 150, 1, 250, "bf16", 0, None),
    "beyond-32KB-frames": (1, 2, 128, (3, 43), 40, (0, 60), 30, 200, 150, 1, 250, "bf16", 0, None),
    "small-two-table-rounds": (1, 2, 128, (9, 9), 40, (0, 33), 30, 200, 150, 1, 250, "bf16", ipv.VAN_REVERSE, None),
    # one pass with few new rows in a call, then frames without one
    "in-cache": (2, 2, 128, (7, 7), 49, (1990, 1960, 1960), 6, 2000, 1600, 4, 2051, "bf16", ipv.HEAD_SHARED, None),
    "in-cache-pooled": (4, 1, 64, (7, 7), 30, (1990, 0, 1870), 8, 2000, 1600, 4, 2030, "f32", 0, (0.3, 0.5, 0.7)),
    # the consecutive-frame mode: the norms only, where the walks take most of the CUs and the selections do not
    "ahead-adjacent-half-the-slices": (224, 2, 32, (6, 7), 42, (0,), 40, 900, 400, 2, 943, "bf16",
                                       ipv.TAR_ADJACENT | ipv.HEAD_SHARED, None),
    # all passes of a call in the cache: much metadata on one workgroup
    "call-in-cache": (1, 8, 32, (14, 14), 196, (0, 500), 60, 5000, 3800, 4, 5199, "bf16", ipv.HEAD_SHARED, None),
    "call-in-cache-uniform": (1, 4, 32, (14, 14), 150, (2900,), 70, 8000, 6000, 3, 8150, "f32",
                              ipv.HEAD_SHARED | ipv.UNIFORM_SELECT, None),
    "call-in-cache-pooled": (1, 8, 32, (7, 7), 49, (0, 0, 4900), 120, 5000, 4000, 4, 5049, "bf16",
                             ipv.HEAD_SHARED | ipv.VAN_REVERSE, (0.3, 0.5, 0.7)),
    "call-in-cache-long-pooled": (1, 2, 32, (14, 14), 196, (0, 20000), 240, 26000, 13000, 4, 26195, "bf16", 0,
                                  (0.3, 0.5, 0.7)),
    "ahead-adjacent": (2, 2, 256, (9, 13), 117, (0,), 60, 1700, 800, 3, 1819, "f32", ipv.TAR_ADJACENT, None),
    "ahead-adjacent-shared": (3, 2, 64, (9, 13), 117, (0, 0), 60, 1700, 1500, 4, 1817, "bf16",
                        ipv.TAR_ADJACENT | ipv.HEAD_SHARED, None),
}


@pytest.mark.parametrize("name", CASES)
@pytest.mark.parametrize("cut", [0, 1])
def test_stream_passes_equal_step_by_step(name, cut):
    L, H, D, (gh, gw), rows, entry, frames, cap, budget, r, S, dtype, mode, tau = CASES[name]
    p, B = gh * gw, len(entry)
    sd, kind, bits = (synth.BF16, "bf16", torch.int16) if dtype == "bf16" else (synth.F32, "raw", torch.int32)
    sigma = (0.1, 0.35, 0.55, 1.0) if tau else (0.5,)
    src = [synth.fresh_cache(900 + b, L, H, frames * p, D, gh, gw, frames * p, sd, synth.RhoSpec(0.0, 0.95, 0.2), sigma)
           for b in range(B)]
    old = [synth.fresh_cache(950 + b, L, H, S, D, gh, gw, max(n, 1), sd, synth.RhoSpec(0.0, 0.95), sigma)
           for b, n in enumerate(entry)]
    fr_of = lambda a, f: np.stack([getattr(s, a)[:, :, f * p:f * p + rows] for s in src])  # noqa: E731
    fK = P.to_device(np.ascontiguousarray(np.stack([fr_of("K", f) for f in range(frames)])), kind)
    fV = P.to_device(np.ascontiguousarray(np.stack([fr_of("V", f) for f in range(frames)])), kind)

    def fresh():
        K = torch.zeros((B, L, H, S, D), dtype=torch.bfloat16 if dtype == "bf16" else torch.float32, device="cuda:0")
        V = torch.zeros_like(K)
        fr = torch.full((B, L, H, S), -1, dtype=torch.int32, device="cuda:0")
        pa = torch.full_like(fr, -1)
        for b, n in enumerate(entry):
            if n:
                K[b, :, :, :n] = P.to_device(np.ascontiguousarray(old[b].K[:, :, :n]), kind)
                V[b, :, :, :n] = P.to_device(np.ascontiguousarray(old[b].V[:, :, :n]), kind)
                fr[b, :, :, :n] = P.to_device(np.ascontiguousarray(old[b].frame_idx[:, :, :n] - 1000))
                pa[b, :, :, :n] = P.to_device(np.ascontiguousarray(old[b].patch_idx[:, :, :n]))
        return K, V, fr, pa, ipv.Compressor(K, gh, gw, budget)

    args = (cap, budget, 0.5, r, tau)
    if name == "budget-is-cap":  # the count after the pass admits no further frame
        frames = -(-(cap - entry[0]) // rows)
    K1, V1, f1, p1, c1 = fresh()
    n1, passes1 = list(entry), [0] * B
    at = [0] * B  # rows at each stream's last pass
    for f in range(frames):
        before = n1
        n1, fired = ipv.ipv_ckv_step(K1, V1, f1, p1, n1, fK[f], fV[f], f, 0, *args, c1.tar, c1.van, c1.keep_idx, c1.ws,
                                     gh, gw, mode=mode)
        for b in range(B):
            passes1[b] += int(fired[b])
            at[b] = before[b] + rows if fired[b] else at[b]
    K2, V2, f2, p2, c2 = fresh()
    n2, passes2 = list(entry), [0] * B
    cuts = [0, frames // 3, frames // 3 + 1, frames] if cut else [0, frames]
    for a, b in zip(cuts, cuts[1:]):
        n2, ps = ipv.ipv_ckv_stream(K2, V2, f2, p2, n2, fK[a:b], fV[a:b], a, *args, c2.tar, c2.van, c2.keep_idx, c2.ws,
                                    gh, gw, mode=mode)
        passes2 = [x + y for x, y in zip(passes2, ps)]
    torch.cuda.synchronize()
    assert c1.device_errors() == 0 and c2.device_errors() == 0
    assert n2 == n1 and passes2 == passes1 and max(passes1) >= 1
    for b in range(B):
        m = n1[b]
        for x, y in ((K1, K2), (V1, V2)):
            assert torch.equal(x[b, :, :, :m].view(bits), y[b, :, :, :m].view(bits))
        assert torch.equal(f1[b, :, :, :m], f2[b, :, :, :m]) and torch.equal(p1[b, :, :, :m], p2[b, :, :, :m])
        if passes1[b]:
            assert torch.equal(c1.keep_idx[b], c2.keep_idx[b])
            if not mode & ipv.UNIFORM_SELECT:
                for x, y in ((c1.tar, c2.tar), (c1.van, c2.van)):
                    assert torch.equal(x[b, :, :, :at[b]].view(torch.int32), y[b, :, :, :at[b]].view(torch.int32))
    print(name, "passes", passes1, "rows", n1, flush=True)


def test_frames_in_the_caches_own_rows():
    """A program that writes frames where they will be appended: the same as with the frames in a buffer of their own."""
    gh = gw = 7
    p, D, n0, frames, cap, budget, r = 49, 64, 98, 39, 2000, 1000, 4
    S = n0 + frames * p
    st = synth.fresh_cache(77, 1, 1, S, D, gh, gw, S, synth.F32, synth.RhoSpec(0.0, 0.95), (0.5,))
    out = []
    for own in (False, True):
        K, V, fr, pa = (P.to_device(np.ascontiguousarray(getattr(st, a)[None])) for a in ("K", "V", "frame_idx", "patch_idx"))
        fK, fV = (t[0, 0, 0, n0:].view(frames, 1, 1, 1, p, D) for t in (K, V))
        if own:
            fK, fV = fK.clone(), fV.clone()
        c = ipv.Compressor(K, gh, gw, budget)
        n, passes = ipv.ipv_ckv_stream(K, V, fr, pa, n0, fK, fV, 2, cap, budget, 0.5, r, None, c.tar, c.van, c.keep_idx,
                                       c.ws, gh, gw)
        torch.cuda.synchronize()
        assert passes == 1 and c.device_errors() == 0
        out.append([t[..., :n, :] for t in (K, V)] + [t[..., :n] for t in (fr, pa)] + [c.keep_idx])
    for x, y in zip(*out):
        assert torch.equal(x, y)
