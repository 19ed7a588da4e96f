"""What calls launch, on a host-only build that writes the launches down."""
import ctypes

import pytest

from paper_2506_15745_amd import ipv
from tests.recorder import BASE, Stream, recorder, recorder_library  # noqa: F401

# 16 streams below the cap at counts of their own, all at it within the first frame
FIRE_TOGETHER = dict(L=2, H=2, D=64, grid=(14, 14), cap=6272, budget=3136, r=4, entry=[6076 + b for b in range(16)])


@pytest.mark.parametrize("mode,tau,chain", [(0, None, 3), (ipv.TAR_ADJACENT, None, 3), (0, (0.3, 0.5, 0.7), 4),
                                            (ipv.UNIFORM_SELECT, None, 1)])
def test_streams_alike_after_a_pass_share_its_launches(recorder, mode, tau, chain):  # noqa: F811
    """Streams that enter a call with different counts and are compressed at the same frame
    are at the budget together from then on: only that first pass takes launches for each."""
    s = Stream(**FIRE_TOGETHER)
    passes = 6
    recorder.start()
    rc, n, ps = s.call(1 + 16 * (passes - 1), mode, tau)
    assert rc == ipv.OK and ps == [passes] * 16 and n == [3136] * 16
    got = recorder.launches()
    assert len(got) <= 16 * chain + (passes - 1) * chain + 1
    assert [x.kernel for x in got].count("k_stretch_gather") == 1


@pytest.mark.parametrize("frames,mode,tau,where", [
    (3, 0, None, "cache"), (4, 0, None, "frames"), (3, ipv.HEAD_SHARED, None, "cache"), (4, 0, (0.3, 0.5, 0.7), "cache"),
    (5, 0, (0.3, 0.5, 0.7), "frames"), (1, ipv.TAR_ADJACENT, None, "cache"), (1, ipv.UNIFORM_SELECT, None, "cache")])
def test_a_pass_with_few_new_rows_runs_in_the_cache(recorder, frames, mode, tau, where):  # noqa: F811
    s = Stream(L=28, H=4, D=128, grid=(14, 14), cap=6272, budget=3136, r=4, entry=[6272 - 196 * frames])
    recorder.start()
    rc, n, ps = s.call(frames, mode, tau)
    assert rc == ipv.OK and ps == [1] and n == [3136]
    kernels = recorder.kernels()
    assert ("k_append" in kernels and "k_compact" in kernels) == (where == "cache")
    assert ("k_stretch_gather" in kernels) == (where == "frames")


@pytest.mark.parametrize("L,H,D,cap,mode,in_cache", [
    (1, 8, 64, 6272, ipv.HEAD_SHARED, True), (1, 2, 64, 6272, ipv.HEAD_SHARED, False), (28, 4, 128, 6272, ipv.HEAD_SHARED, False),
    (1, 8, 256, 6272, ipv.HEAD_SHARED, False), (1, 4, 64, 31000, ipv.HEAD_SHARED | ipv.UNIFORM_SELECT, True),
    (1, 1, 64, 46000, ipv.UNIFORM_SELECT, True), (1, 1, 64, 12000, ipv.UNIFORM_SELECT, False), (1, 1, 64, 12000, 0, False),
    (1, 8, 64, 20000, ipv.HEAD_SHARED | ipv.TAR_ADJACENT, True), (1, 4, 64, 20000, ipv.HEAD_SHARED | ipv.TAR_ADJACENT, False)])
def test_a_call_with_much_metadata_on_few_workgroups_runs_in_the_cache(recorder, L, H, D, cap, mode, in_cache):  # noqa: F811
    budget = cap * 3 // 4
    s = Stream(L=L, H=H, D=D, grid=(14, 14), cap=cap, budget=budget, r=4, entry=[0])
    first, later = -(-cap // 196), -(-(cap - budget) // 196)
    recorder.start()
    rc, n, passes = s.call(first + 2 * later + 1, mode)
    assert rc == ipv.OK and passes == [3] and n == [budget + 196]
    kernels = recorder.kernels()
    assert kernels.count("k_append") == (4 if in_cache else 1) and kernels.count("k_compact") == (3 if in_cache else 0)
    assert any("stretch" in k for k in kernels) != in_cache


@pytest.mark.parametrize("L,H,D,cap,mode,in_cache", [
    (1, 2, 64, 50000, 0, True), (1, 1, 64, 26000, 0, True), (1, 1, 64, 9000, 0, False), (6, 8, 64, 50000, 0, False),
    (2, 1, 64, 50000, ipv.TAR_ADJACENT, True), (1, 1, 64, 16000, ipv.TAR_ADJACENT, False), (28, 4, 128, 6272, 0, False)])
def test_a_call_with_pooling_over_few_long_slices_runs_in_the_cache(recorder, L, H, D, cap, mode, in_cache):  # noqa: F811
    budget = cap // 2
    s = Stream(L=L, H=H, D=D, grid=(14, 14), cap=cap, budget=budget, r=4, entry=[0])
    recorder.start()
    rc, n, passes = s.call(-(-cap // 196) + 2 * -(-(cap - budget) // 196), mode, (0.3, 0.5, 0.7))
    assert rc == ipv.OK and passes == [3] and n == [budget]
    kernels = recorder.kernels()
    assert kernels.count("k_append") == (3 if in_cache else 0) and any("stretch" in k for k in kernels) != in_cache


@pytest.mark.parametrize("apart", [196, 1, 0])
def test_streams_that_are_compressed_apart_count_apart(recorder, apart):  # noqa: F811
    """What the passes over the frames save is set against the selections of as many launches as the streams take
    (streams of different counts take launches of their own also in a pass at the same frame)."""
    s = Stream(L=1, H=8, D=64, grid=(14, 14), cap=6272, budget=4704, r=4, entry=[apart * b for b in range(8)])
    recorder.start()
    rc, n, passes = s.call(32, ipv.HEAD_SHARED)
    assert rc == ipv.OK and passes == [1] * 8
    assert any("stretch" in k for k in recorder.kernels()) == (apart == 0)


@pytest.mark.parametrize("frames_at,cache,apart", [
    ("fK", "K", False), ("fV", "V", False), ("fK", "V", False), ("fV", "K", False), ("fK", "K", True), ("fV", "V", True)])
def test_frames_in_the_caches_memory_go_frame_by_frame(recorder, frames_at, cache, apart):  # noqa: F811
    """Passes over frames where they lie would read what the gather has overwritten."""
    s = Stream(L=1, H=1, D=64, grid=(14, 14), cap=6272, budget=3136, r=4, entry=[196])
    # the frames begin in the cache's last row, or where the cache ends
    s.at[frames_at] = s.at[cache] + (s.shape.capacity - (0 if apart else 1)) * 64 * 2
    recorder.start()
    rc, n, ps = s.call(64)
    assert rc == ipv.OK and ps == [3] and n == [3136 + 196]
    kernels = recorder.kernels()
    assert any("stretch" in k for k in kernels) == apart
    assert kernels.count("k_append") == (1 if apart else 64)


@pytest.mark.parametrize("own_memory", [True, False])
def test_a_call_that_the_runtime_stops_reports_what_it_came_with(recorder, own_memory):  # noqa: F811
    s = Stream(L=1, H=1, D=64, grid=(14, 14), cap=6272, budget=3136, r=4, entry=[196, 3136, 0])
    if not own_memory:
        s.at["fK"] = s.at["K"]
    recorder.start()
    assert s.call(40)[0] == ipv.OK
    total = len(recorder.launches())
    assert total > 10
    for stop in range(total):
        recorder.start(fail=stop)
        assert s.call(40) == (ipv.ERR_HIP, [196, 3136, 0], [0, 0, 0])
        assert len(recorder.launches()) == stop  # nothing is launched after the refusal


@pytest.mark.parametrize("slices,D,grid,padded", [
    (57, 128, (14, 14), 57), (113, 128, (14, 14), 114), (225, 128, (14, 14), 228), (449, 128, (14, 14), 456),
    (113, 256, (24, 24), 114), (449, 256, (24, 24), 450), (449, 256, (48, 48), 449), (449, 128, (24, 24), 452)])
def test_tar_tiles_share_the_cache_with_as_many_tables_as_fit(recorder, slices, D, grid, padded):  # noqa: F811
    """The TaR tiles of a pass without old rows are numbered for whole groups of slices (1, 2, 4 or 8)."""
    p = grid[0] * grid[1]
    s = Stream(L=slices, H=1, D=D, grid=grid, cap=4 * p, budget=2 * p, r=1, entry=[0])
    recorder.start()
    assert s.call(4)[0] == ipv.OK
    tar, = [x for x in recorder.launches() if x.kernel == "k_stretch_tar"]
    tiles = -(-p // (256 * 16 // (2 * D)))  # a group of 256 threads: 256 / lanes a row columns of 4 frames
    assert tar.grid_x == -(-padded * tiles // 8) * 8


@pytest.mark.parametrize("L,H,D,dtype,cap,budget,r,mode,ahead", [
    (80, 8, 128, ipv.BF16, 6272, 3136, 4, ipv.HEAD_SHARED, True),
    (28, 4, 128, ipv.BF16, 1568, 784, 4, 0, False),  # the window is all 4 new frames, 3 of them
    (28, 4, 128, ipv.BF16, 1568, 784, 3, 0, True),
    (160, 1, 128, ipv.BF16, 6272, 3136, 4, 0, True), (161, 1, 128, ipv.BF16, 6272, 3136, 4, 0, False),
    (64, 1, 256, ipv.F32, 6272, 3136, 4, 0, True), (65, 1, 256, ipv.F32, 6272, 3136, 4, 0, False),
    (1, 4, 128, ipv.BF16, 16200, 8000, 4, 0, True), (1, 4, 128, ipv.BF16, 16600, 8000, 4, 0, False),
    (28, 4, 128, ipv.BF16, 6272, 3136, 4, ipv.TAR_ADJACENT, False),
    (28, 4, 128, ipv.BF16, 6272, 3136, 4, ipv.TAR_ADJACENT | ipv.HEAD_SHARED, True),
    (28, 4, 128, ipv.BF16, 2352, 1176, 4, ipv.TAR_ADJACENT | ipv.HEAD_SHARED, False),
    (4, 4, 128, ipv.BF16, 12544, 6272, 4, ipv.TAR_ADJACENT | ipv.HEAD_SHARED, False)])
def test_the_next_passs_launch_goes_beside_few_selections(recorder, L, H, D, dtype, cap, budget, r, mode, ahead):  # noqa: F811
    s = Stream(L=L, H=H, D=D, grid=(14, 14), cap=cap, budget=budget, r=r, entry=[0], dtype=dtype)
    recorder.start()
    rc, _, passes = s.call(-(-cap // 196) + 2 * -(-(cap - budget) // 196), mode)
    assert rc == ipv.OK and passes == [3]
    kernels = recorder.kernels()
    assert kernels.count("k_select_ahead") == (2 if ahead else 0)
    # without it each pass has a first launch of its own; with it only the first one, or the walks stay
    walks = bool(mode & ipv.TAR_ADJACENT)
    assert kernels.count("k_stretch_prev_van" if walks else "k_stretch_table_van") == (1 if ahead and not walks else 3)


def compress_kernels(recorder, n, L, H, D, grid, r, dtype):  # noqa: F811
    """The kernels of one ipv_compress of n rows a slice."""
    s = ipv.Shape(1, L, H, D, n, *grid, dtype)
    a = {k: BASE * (i + 1) for i, k in enumerate("K V fr pa tar van keep ws".split())}
    recorder.start()
    assert ipv.lib().ipv_compress(ctypes.byref(s), a["K"], a["V"], a["fr"], a["pa"], (ctypes.c_int32 * 1)(n), n // 2, 0.5, r, 0,
                                  None, a["tar"], a["van"], a["keep"], a["ws"], ipv.workspace_bytes(s), None) == ipv.OK
    return recorder.launches()


@pytest.mark.parametrize("n,D,dtype,grid,one", [
    (256, 128, ipv.BF16, (8, 8), True), (256, 128, ipv.BF16, (8, 12), True), (256, 128, ipv.BF16, (1, 97), False),
    (256, 128, ipv.BF16, (24, 24), False), (64, 256, ipv.F32, (4, 6), True), (64, 256, ipv.F32, (5, 5), False),
    (64, 256, ipv.F32, (64, 64), False), (256, 32, ipv.BF16, (16, 24), True), (256, 32, ipv.BF16, (90, 90), False)])
def test_a_wide_grid_has_the_launches_of_large_slices(recorder, n, D, dtype, grid, one):  # noqa: F811
    """In one workgroup the recent-key table and the tiles take rounds in proportion to the grid."""
    kernels = [x.kernel for x in compress_kernels(recorder, n, 1, 2, D, grid, 1, dtype)]
    assert kernels == (["k_small_pass"] if one else ["k_table_van", "k_score_sweep", "k_select", "k_compact"])


def test_a_small_pass_fits_the_lds(recorder):  # noqa: F811
    """The dynamic part of the largest request; the static part (the selection's, and the places of a
    stretch) is below 64 KB, and a CU has 160 KB."""
    most = 0
    for D, dtype in ((32, ipv.BF16), (64, ipv.BF16), (32, ipv.F32), (256, ipv.BF16), (256, ipv.F32)):
        for x in compress_kernels(recorder, 64, 1, 2, D, (1, 2), 32, dtype):
            assert x.kernel == "k_small_pass"
            most = max(most, x.lds)
    assert most == 32 << 10
