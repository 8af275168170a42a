"""The ring with a launch per step: hvdx_ring_allreduce_steps against the oracle, and, at full
size, the ring on the tensors and the compressed ring of a direct tensor against the one-launch
path (which test_gpu_workloads.py and test_gpu_large.py hold to the oracle), bit for bit."""
import numpy as np
import pytest
import torch

import paper_1802_05799_amd as hv
from _gpu import NP_TO_HV, OPS, assert_bits_equal, from_gpu_rows, say, to_gpu_rows
from test_gpu_large import COUNT, N, filled
from test_gpu_ring import CASES, inputs, oracle_ring
from workloads import configs
from workloads import gpu as wgpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["f32", "f16", "compressed"])
def test_steps_match_oracle(kind):
    dtype = np.float16 if kind == "f16" else np.float32
    compress = hv.COMPRESS_FP16 if kind == "compressed" else hv.COMPRESS_NONE
    rng = np.random.default_rng(800)
    for n, count in CASES:
        for op in ("sum", "average"):
            for offset in (0, 3):
                say(f"ring in steps {kind} n={n} count={count} {op} offset={offset}")
                x = inputs(rng, n, count, dtype)
                rows, keep = to_gpu_rows(x, offset)
                need = hv.hvdx_ring_workspace_bytes(n, count, NP_TO_HV[x.dtype], compress)
                ws = torch.empty(max(need, 1), dtype=torch.uint8, device="cuda")
                hv.hvdx_ring_allreduce_steps([r.data_ptr() for r in rows], n, count, NP_TO_HV[x.dtype], OPS[op],
                                             compress, ws.data_ptr() if need else 0, need,
                                             torch.cuda.current_stream().cuda_stream)
                assert_bits_equal(from_gpu_rows(rows), oracle_ring(x, op, compress == hv.COMPRESS_FP16), f"n={n}")


@pytest.mark.parametrize("name,threshold", [("resnet50", 64 << 20), ("inceptionv3", 1 << 20), ("vgg16", 64 << 20),
                                            ("vgg16fp16", 64 << 20)])
def test_workloads_in_steps(name, threshold):
    w = configs.get(name)
    say(f"workload {name} in steps")
    per_rank, storage, _ = wgpu.make_rank_tensors(w)
    hv.FusedAllreduce(per_rank, op=w.op, compress=w.compress, threshold_bytes=threshold)()
    want = [storage[r].clone() for r in (0, w.nranks - 1)]
    del per_rank, storage
    per_rank, storage, _ = wgpu.make_rank_tensors(w)
    ar = hv.FusedAllreduce(per_rank, op=w.op, compress=w.compress, threshold_bytes=threshold, small_bucket_bytes=0)
    assert any(k == "rs" for k, _, _ in ar.kernel_sequence())
    ar()
    torch.cuda.synchronize()
    for x, r in zip(want, (0, w.nranks - 1)):
        assert torch.equal(x.view(torch.int32), storage[r].view(torch.int32)), f"rank {r}"
    assert all(torch.equal(x.view(torch.int32), storage[0].view(torch.int32)) for x in storage)
    del ar, per_rank, storage, want
    torch.cuda.empty_cache()


@pytest.mark.parametrize("path", ["flat", "tensors"])
def test_steps_beyond_2_to_31_elements(path):
    say(f"large ring in steps: {path}")
    stream = torch.cuda.current_stream().cuda_stream
    rows = filled()
    hv.hvdx_ring_allreduce([x.data_ptr() for x in rows], N, COUNT, hv.FLOAT32, hv.AVERAGE, 0, 0, 0, stream)
    want = rows[0]
    rows = filled()
    if path == "flat":
        hv.hvdx_ring_allreduce_steps([x.data_ptr() for x in rows], N, COUNT, hv.FLOAT32, hv.AVERAGE, 0, 0, 0, stream)
    else:
        ar = hv.FusedAllreduce([[x] for x in rows], op="average", threshold_bytes=4 * COUNT, small_bucket_bytes=0)
        assert not ar.buckets[0].direct and not ar.buckets[0].small
        ar()
    torch.cuda.synchronize()
    assert all(torch.equal(x.view(torch.int32), want.view(torch.int32)) for x in rows)
    del rows, want
    torch.cuda.empty_cache()
