"""What calls launch, on a host-only build that writes the launches down."""
import pytest

from paper_2506_15745_amd import ipv
from tests.recorder import Stream, recorder, recorder_library  # noqa: F401

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
