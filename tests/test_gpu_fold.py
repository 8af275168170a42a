"""The one-launch kernels at the edges of their shapes: bursts of 8, 16 and 32 ranks and
their remainders, stretches of 64 vectors that a chunk ends inside, buffers aligned to
their elements only.  Bit for bit against the oracle's ring (no tolerance: the order of
additions and every rounding are the ring's)."""
import numpy as np
import pytest
import torch

import paper_1802_05799_amd as hv
from _gpu import NP_TO_HV, OPS, assert_bits_equal, from_gpu_rows, say, to_gpu_rows
from test_gpu_ring import inputs, oracle_ring

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [np.float32, np.float16], ids=["f32", "f16"])
@pytest.mark.parametrize("n", [2, 7, 8, 9, 15, 16, 17, 31, 32, 33, 48, 63, 64, 65, 128])
def test_flat_buffers(n, dtype):
    stretch = 64 * 16 // np.dtype(dtype).itemsize
    rng = np.random.default_rng(5000 + n)
    for count in (n, n * stretch, n * stretch + 1, n * (2 * stretch - 3) + n - 1, 3 * stretch * n - 5):
        for op in ("sum", "average"):
            for offset in (0, 1):
                say(f"one-launch ring n={n} count={count} {np.dtype(dtype).name} {op} offset={offset}")
                x = inputs(rng, n, count, dtype)
                want = oracle_ring(x, op)
                for fold in (False, True):
                    rows, keep = to_gpu_rows(x, offset)
                    args = ([r.data_ptr() for r in rows], n, count, NP_TO_HV[x.dtype], OPS[op])
                    stream = torch.cuda.current_stream().cuda_stream
                    if fold:
                        hv.hvdx_fold_allreduce(*args, hv.COMPRESS_NONE, stream)
                    else:
                        hv.hvdx_ring_allreduce_small(*args, stream)
                    assert_bits_equal(from_gpu_rows(rows), want, f"n={n} count={count} {op} fold={fold}")


@pytest.mark.parametrize("n", [1, 3, 8, 17, 40])
def test_flat_buffers_compressed(n):
    rng = np.random.default_rng(5100 + n)
    for count in (n * 256, n * 700 + 3):
        for offset in (0, 3):
            say(f"compressed fold n={n} count={count} offset={offset}")
            x = inputs(rng, n, count, np.float32)
            want = oracle_ring(x, "average", True)
            rows, keep = to_gpu_rows(x, offset)
            hv.hvdx_fold_allreduce([r.data_ptr() for r in rows], n, count, hv.FLOAT32, hv.AVERAGE, hv.COMPRESS_FP16,
                                   torch.cuda.current_stream().cuda_stream)
            assert_bits_equal(from_gpu_rows(rows), want, f"n={n} count={count}")
