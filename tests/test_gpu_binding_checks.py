"""The binding reads a pass's whole buffer set at once when everything fits;
what does not fit is refused with the same status as on host tensors."""
import numpy as np
import pytest
import torch

from paper_2506_15745_amd import ipv

pytestmark = pytest.mark.gpu

B, L, H, S, D, GH, GW, C = 1, 2, 2, 64, 32, 4, 4, 32
ROWS = (B, L, H, S)


def bufs():
    z = lambda *s, dt=torch.float32: torch.zeros(s, dtype=dt, device="cuda:0")  # noqa: E731
    i32 = torch.int32
    return dict(K=z(*ROWS, D, dt=torch.bfloat16), V=z(*ROWS, D, dt=torch.bfloat16), fr=z(*ROWS, dt=i32),
                pa=z(*ROWS, dt=i32), tar=z(*ROWS), van=z(*ROWS), keep=z(B, L, H, C, dt=i32),
                ws=z(1 << 20, dt=torch.uint8), Kn=z(B, L, H, 16, D, dt=torch.bfloat16),
                Vn=z(B, L, H, 16, D, dt=torch.bfloat16))


def compress(b):
    ipv.ipv_compress(b["K"], b["V"], b["fr"], b["pa"], S, C, 0.5, 1, None, b["tar"], b["van"], b["keep"], b["ws"], GH, GW)


def step(b):
    ipv.ipv_ckv_step(b["K"], b["V"], b["fr"], b["pa"], 0, b["Kn"], b["Vn"], 0, 0, S, C, 0.5, 1, None, b["tar"], b["van"],
                     b["keep"], b["ws"], GH, GW)


def stream(b):
    ipv.ipv_ckv_stream(b["K"], b["V"], b["fr"], b["pa"], 0, b["Kn"][None], b["Vn"][None], 0, S, C, 0.5, 1, None,
                       b["tar"], b["van"], b["keep"], b["ws"], GH, GW)


BAD = {
    "keep-short": ("keep", lambda t: t[..., :C - 1].contiguous(), ipv.ERR_SHAPE),
    "keep-int64": ("keep", lambda t: t.long(), ipv.ERR_DTYPE),
    "tar-short": ("tar", lambda t: t[..., :S - 1].contiguous(), ipv.ERR_SHAPE),
    "van-double": ("van", lambda t: t.double(), ipv.ERR_DTYPE),
    "van-strided": ("van", lambda t: torch.zeros(B, L, S, H, device="cuda:0").transpose(2, 3), ipv.ERR_SHAPE),
    "K-strided": ("K", lambda t: torch.zeros(B, L, H, D, S, dtype=t.dtype, device="cuda:0").transpose(3, 4), ipv.ERR_SHAPE),
    "K-half": ("K", lambda t: t.half(), ipv.ERR_DTYPE),
    "V-float": ("V", lambda t: t.float(), ipv.ERR_DTYPE),
    "V-short": ("V", lambda t: t[:, :, :, :S - 8].contiguous(), ipv.ERR_SHAPE),
    "fr-float": ("fr", lambda t: t.float(), ipv.ERR_DTYPE),
    "pa-host": ("pa", lambda t: t.cpu(), ipv.ERR_ARG),
    "ws-host": ("ws", lambda t: t.cpu(), ipv.ERR_ARG),
    "V-none": ("V", lambda t: None, ipv.ERR_NULL),
    "fr-none": ("fr", lambda t: None, ipv.ERR_NULL),
    "pa-none": ("pa", lambda t: None, ipv.ERR_NULL),
    "ws-small": ("ws", lambda t: t[:512].clone(), ipv.ERR_WORKSPACE),
}


@pytest.mark.parametrize("name", BAD)
def test_mismatched_gpu_tensors_are_refused(name):
    key, make, want = BAD[name]
    b = bufs()
    b[key] = make(b[key])
    for call in (compress, step, stream):
        if call is not compress and name == "ws-small":
            continue  # one frame fires no pass, which needs no workspace
        with pytest.raises(ipv.IpvError) as e:
            call(b)
        assert e.value.status == want, call.__name__


@pytest.mark.parametrize("key,make,want", [
    ("Kn", lambda t: t.float(), ipv.ERR_DTYPE), ("Vn", lambda t: t[:, :, :, :8].contiguous(), ipv.ERR_SHAPE),
    ("Kn", lambda t: t[:, :1].contiguous(), ipv.ERR_SHAPE), ("Vn", lambda t: t.cpu(), ipv.ERR_ARG),
    ("Kn", lambda t: torch.zeros(B, L, H, D, 16, dtype=t.dtype, device="cuda:0").transpose(3, 4), ipv.ERR_SHAPE)])
def test_mismatched_frames_are_refused(key, make, want):
    b = bufs()
    b[key] = make(b[key])
    for call in (step, stream):
        with pytest.raises(ipv.IpvError) as e:
            call(b)
        assert e.value.status == want, call.__name__


def test_grid_sizes_are_taken_as_a_fresh_shape_takes_them():
    """Also after a call with the same grid has been seen: floats refused, anything with an index accepted, by its value now."""
    b = bufs()
    run = lambda gh: ipv.ipv_compress(b["K"], b["V"], b["fr"], b["pa"], S, C, 0.5, 1, None, b["tar"], b["van"],  # noqa: E731
                                      b["keep"], b["ws"], gh, GW)
    run(GH)
    with pytest.raises(TypeError):
        run(float(GH))
    run(np.array(GH))
    changing = torch.tensor(GH)
    run(changing)
    changing.fill_(0)
    with pytest.raises(ipv.IpvError) as e:
        run(changing)
    assert e.value.status == ipv.ERR_SHAPE


def test_calls_follow_the_current_stream():
    b = bufs()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert ipv._stream(None) == side.cuda_stream == torch.cuda.current_stream().cuda_stream
        step(b)
    assert ipv._stream(None) == torch.cuda.current_stream().cuda_stream
    torch.cuda.synchronize()
