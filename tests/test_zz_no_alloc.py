"""hvdx_ring_allreduce_noalloc and hvdx_ring_allreduce_whole (the ring in one launch without a
workspace argument) against hvdx_ring_allreduce_steps (other kernels: a launch per step, the
messages through memory and, compressed, through a caller's workspace): the same bits, through
the C-ABI, on calls in a row, compressed and not, and the former's limit refused."""
import numpy as np
import pytest
import torch

import paper_1802_05799_amd as hv
from _gpu import assert_bits_equal, say

pytestmark = pytest.mark.gpu


def rows(x):
    return [torch.from_numpy(np.ascontiguousarray(r)).cuda() for r in x]


def in_steps(x, op, compress):
    n, count = x.shape
    r = rows(x)
    wsb = hv.hvdx_ring_workspace_bytes(n, count, hv.FLOAT32, compress)
    ws = torch.empty(max(wsb, 1), dtype=torch.uint8, device="cuda")
    hv.hvdx_ring_allreduce_steps([t.data_ptr() for t in r], n, count, hv.FLOAT32, op, compress,
                                 ws.data_ptr() if wsb else 0, wsb, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    return np.stack([t.cpu().numpy() for t in r])


def without_workspace(call, x, op, compress):
    n, count = x.shape
    r = rows(x)
    call([t.data_ptr() for t in r], n, count, hv.FLOAT32, op, compress, stream=torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    return np.stack([t.cpu().numpy() for t in r])


CALLS = [  # (ranks, elements) of consecutive calls; the first just under the 64 MiB limit
    (8, 4_194_304 - 128),  # 8 x 4,194,176 binary16 elements = 64 MiB - 2 KiB
    (5, 100_003),  # not a power of two: a true division; chunks not 16-byte aligned
    (3, 1_001),
    (1, 4_099),  # one rank: rounded to binary16 when compressed
]


@pytest.mark.parametrize("compress", [hv.COMPRESS_FP16, hv.COMPRESS_NONE], ids=["fp16-wire", "no-compression"])
def test_noalloc_matches_the_ring_in_steps(compress):
    assert hv.hvdx_ring_noalloc_max_bytes() == 64 << 20
    rng = np.random.default_rng(2024)
    for k, (n, count) in enumerate(CALLS):
        for op in (hv.AVERAGE, hv.SUM):
            say(f"noalloc call {k}: N={n} count={count} op={op} compress={compress}")
            x = (rng.standard_normal((n, count)) * 0.01).astype(np.float32)
            x[:, :6] = np.array([0.0, -0.0, 2.0 ** -24, 65504.0, 1e-8, -3.0], np.float32)
            want = in_steps(x, op, compress)
            assert all(np.array_equal(want[r].view(np.uint32), want[0].view(np.uint32)) for r in range(n))
            for call in (hv.hvdx_ring_allreduce_noalloc, hv.hvdx_ring_allreduce_whole):
                got = without_workspace(call, x, op, compress)
                assert_bits_equal(got, want, f"{call.__name__} call {k} N={n} count={count} op={op}")


def test_noalloc_refuses_more_than_its_limit():
    n, count = 8, 4_194_304 + 1  # one element past 64 MiB in binary16
    assert hv.hvdx_ring_workspace_bytes(n, count, hv.FLOAT32, hv.COMPRESS_FP16) > hv.hvdx_ring_noalloc_max_bytes()
    x = [torch.zeros(count, device="cuda") for _ in range(n)]
    with pytest.raises(hv.HvdxError) as e:
        hv.hvdx_ring_allreduce_noalloc([t.data_ptr() for t in x], n, count, hv.FLOAT32, hv.AVERAGE,
                                       hv.COMPRESS_FP16, torch.cuda.current_stream().cuda_stream)
    assert e.value.status == hv.ERR_WORKSPACE and "static" in str(e.value)
