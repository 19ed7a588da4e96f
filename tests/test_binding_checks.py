"""The Python binding refuses companion tensors that do not match the cache.

The C ABI only sees pointers, so a score, keep-index or metadata tensor
smaller than the cache implies would be written past its end; the binding
checks shape, dtype and device of every tensor first. These checks run before
any pointer is taken, so host tensors exercise them without a GPU (a fully
consistent set of host tensors is then refused for not being in GPU memory).
"""
import pytest
import torch

from paper_2506_15745_amd import ipv

B, L, H, S, D, GH, GW, C = 1, 2, 2, 64, 32, 4, 4, 32


def bufs(dtype=torch.bfloat16):
    K = torch.zeros(B, L, H, S, D, dtype=dtype)
    return dict(K=K, V=torch.zeros_like(K), fr=torch.zeros(B, L, H, S, dtype=torch.int32),
                pa=torch.zeros(B, L, H, S, dtype=torch.int32), tar=torch.zeros(B, L, H, S),
                van=torch.zeros(B, L, H, S), keep=torch.zeros(B, L, H, C, dtype=torch.int32),
                ws=torch.zeros(1 << 16, dtype=torch.uint8), pool=torch.zeros(B, L, dtype=torch.int32))


def compress(b, budget=C):
    ipv.ipv_compress(b["K"], b["V"], b["fr"], b["pa"], S, budget, 0.5, 1, None, b["tar"], b["van"], b["keep"],
                     b["ws"], GH, GW)


def status(fn, *a, **kw):
    with pytest.raises(ipv.IpvError) as e:
        fn(*a, **kw)
    return e.value.status


@pytest.mark.parametrize("key,bad,st", [
    ("keep", torch.zeros(B, L, H, C - 1, dtype=torch.int32), ipv.ERR_SHAPE),   # shorter than the budget
    ("keep", torch.zeros(B, L, H, C, dtype=torch.int64), ipv.ERR_DTYPE),
    ("tar", torch.zeros(B, L, H, S - 1), ipv.ERR_SHAPE),                       # fewer rows than the cache
    ("van", torch.zeros(B, L, 1, S), ipv.ERR_SHAPE),
    ("van", torch.zeros(B, L, H, S, dtype=torch.float64), ipv.ERR_DTYPE),
    ("V", torch.zeros(B, L, H, S, D, dtype=torch.float32), ipv.ERR_DTYPE),     # fp32 V with a bf16 K
    ("V", torch.zeros(B, L, H, S - 8, D, dtype=torch.bfloat16), ipv.ERR_SHAPE),
    ("fr", torch.zeros(B, L, H, S, dtype=torch.int64), ipv.ERR_DTYPE),
    ("pa", torch.zeros(B, L, H, S // 2, dtype=torch.int32), ipv.ERR_SHAPE),
    ("keep", None, ipv.ERR_NULL),
    ("ws", None, ipv.ERR_WORKSPACE),
])
def test_compress_refuses_mismatched_tensors(key, bad, st):
    b = bufs()
    b[key] = bad
    assert status(compress, b) == st


def test_consistent_host_tensors_reach_the_device_check():
    assert status(compress, bufs()) == ipv.ERR_ARG


def test_keep_width_follows_the_budget():
    b = bufs()
    assert status(compress, b, budget=C - 1) == ipv.ERR_SHAPE


def test_step_entry_points_check_their_tensors():
    b = bufs()
    assert status(ipv.ipv_tar_scores, b["K"], b["fr"], b["pa"], S, 1, torch.zeros(B, L, H, 8), b["ws"], GH,
                  GW) == ipv.ERR_SHAPE
    assert status(ipv.ipv_van_scores, b["V"], b["fr"], b["pa"], S, None, b["van"], torch.zeros(B, L + 1,
                  dtype=torch.int32), b["ws"], GH, GW) == ipv.ERR_SHAPE
    assert status(ipv.ipv_select, b["tar"], b["van"], b["fr"], S, C, 0.5, 1, torch.zeros(B, L, H, 8,
                  dtype=torch.int32), b["ws"], GH, GW) == ipv.ERR_SHAPE
    assert status(ipv.ipv_select, b["tar"], torch.zeros(B, L, H, S, dtype=torch.float16), b["fr"], S, C, 0.5, 1,
                  b["keep"], b["ws"], GH, GW) == ipv.ERR_DTYPE
    assert status(ipv.ipv_compact, b["K"], b["V"], b["fr"], b["pa"], S, b["keep"], C + 1, b["ws"], GH,
                  GW) == ipv.ERR_SHAPE


def test_append_and_loop_check_new_rows():
    b = bufs()
    Kn = torch.zeros(B, L, H, 16, D, dtype=torch.float32)   # fp32 rows into a bf16 cache
    assert status(ipv.ipv_append, b["K"], b["V"], b["fr"], b["pa"], 0, Kn, Kn, 0, 0, GH, GW) == ipv.ERR_DTYPE
    Kn = torch.zeros(B, L, H + 1, 16, D, dtype=torch.bfloat16)
    assert status(ipv.ipv_append, b["K"], b["V"], b["fr"], b["pa"], 0, Kn, Kn, 0, 0, GH, GW) == ipv.ERR_SHAPE
    Kn = torch.zeros(B, L, H, 16, D, dtype=torch.bfloat16)
    assert status(ipv.ipv_ckv_step, b["K"], b["V"], b["fr"], b["pa"], 0, Kn, Kn, 0, 0, 48, C, 0.5, 1, None,
                  b["tar"], b["van"], torch.zeros(B, L, H, C + 4, dtype=torch.int32), b["ws"], GH,
                  GW) == ipv.ERR_SHAPE
    Fk = torch.zeros(3, B, L, H, 16, D, dtype=torch.float32)
    assert status(ipv.ipv_ckv_stream, b["K"], b["V"], b["fr"], b["pa"], 0, Fk, Fk, 0, 48, C, 0.5, 1, None,
                  b["tar"], b["van"], b["keep"], b["ws"], GH, GW) == ipv.ERR_DTYPE


class OnGpu:
    """Answers the binding's questions as a contiguous GPU tensor would."""
    is_cuda, device = True, torch.device("cuda:0")

    def __init__(self, *shape, dtype=torch.float32):
        self.shape, self.dtype = torch.Size(shape), dtype

    def dim(self):
        return len(self.shape)

    def get_device(self):
        return 0

    def is_contiguous(self):
        return True

    def data_ptr(self):
        return 4096


def gpu_buffers():
    rows, i32, bf16 = (1, 2, 2, 64), torch.int32, torch.bfloat16
    return [OnGpu(*rows, 32, dtype=bf16), OnGpu(*rows, 32, dtype=bf16), OnGpu(*rows, dtype=i32), OnGpu(*rows, dtype=i32),
            OnGpu(*rows), OnGpu(*rows), OnGpu(1, 2, 2, 32, dtype=i32)]


@pytest.mark.parametrize("missing", [1, 2, 3])  # V, frame_idx, patch_idx
def test_missing_buffers_of_a_gpu_cache_are_refused(missing):
    b = gpu_buffers()
    b[missing] = None
    with pytest.raises(ipv.IpvError) as e:
        ipv._checked_ptrs(*b, 32, OnGpu(1 << 20, dtype=torch.uint8), 4, 4, 0)
    assert e.value.status == ipv.ERR_NULL


def test_a_grid_is_read_by_its_value_and_type_in_each_call():
    run = lambda g: ipv._checked_ptrs(*gpu_buffers(), 32, OnGpu(1 << 20, dtype=torch.uint8), g, 4, 0)[0].grid_h  # noqa: E731
    assert run(4) == 4 and run(torch.tensor(4)) == 4
    with pytest.raises(TypeError):
        run(4.0)
    changing = torch.tensor(4)
    assert run(changing) == 4
    changing.fill_(5)
    assert run(changing) == 5
