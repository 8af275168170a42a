"""The one-launch kernels at the edges of their shapes: every burst (2 to 16 ranks' loads at once)
and its remainders, stretches of 64 vectors that a chunk ends inside, buffers aligned to
their elements only.  Bit for bit against the oracle's ring (no tolerance: the order of
additions and every rounding are the ring's)."""
import numpy as np
import pytest
import torch

import paper_1802_05799_amd as hv
from _gpu import NP_TO_HV, OPS, assert_bits_equal, from_gpu_rows, say, to_gpu_rows
from _writesets import BURST_RANKS, fold_burst
from oracle import allreduce, native
from test_gpu_ring import inputs, oracle_ring

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [np.float32, np.float16], ids=["f32", "f16"])
@pytest.mark.parametrize("n", [2, 7, 8, 9, 15, 16, 17, 24, 25, 27, 30, 31, 32, 33, 48, 63, 64, 65, 127, 128])
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


@pytest.mark.parametrize("n", BURST_RANKS)
def test_every_burst(n):
    """Each instantiation of either kernel: flat buffers and a list whose tensors lie differently
    to 16 bytes on each rank, binary32, binary16, and binary32 rounded to binary16."""
    rng = np.random.default_rng(5150 + n)
    numel = [n * 300 + 7, 513, 3]
    for half, compress in ((False, False), (True, False), (False, True)):
        dtype = np.float16 if half else np.float32
        say(f"burst of {fold_burst(n)}: n={n} half={half} compress={compress}")
        x = inputs(rng, n, n * 300 + 5, dtype)
        for offset in (0, 1):
            rows, keep = to_gpu_rows(x, offset)
            hv.hvdx_ring_allreduce_whole([r.data_ptr() for r in rows], n, x.shape[1], NP_TO_HV[x.dtype], hv.AVERAGE,
                                         hv.COMPRESS_FP16 if compress else hv.COMPRESS_NONE, offset,  # both loads
                                         torch.cuda.current_stream().cuda_stream)
            assert_bits_equal(from_gpu_rows(rows), oracle_ring(x, "average", compress), f"flat offset={offset}")
        for layout in ("packed", "unalike"):
            host, dev = rank_lists(rng, n, numel, dtype, layout)
            hv.FusedAllreduce(dev, compress=compress, threshold_bytes=2000)()
            torch.cuda.synchronize()
            want = native.allreduce(host, "average", compress=compress, threshold=2000)
            for r in range(n):
                for t in range(len(numel)):
                    assert_bits_equal(dev[r][t].cpu().numpy(), want[r][t], f"{layout} rank {r} tensor {t}")


def rank_lists(rng, n, numel, dtype, layout):
    """Host and device tensor lists; "packed": views end to end; "unalike": each rank's tensors
    at their own distance from a 16-byte boundary."""
    host = [[(rng.standard_normal(k) * 0.01).astype(dtype) for k in numel] for _ in range(n)]
    dev = []
    for r, row in enumerate(host):
        gap = r % 5 if layout == "unalike" else 0
        flat = torch.full((sum(numel) + gap * (len(numel) + 1) + 8,), 7.0, dtype=torch.from_numpy(row[0]).dtype,
                          device="cuda")
        at, ts = 0, []
        for x in row:
            at += gap
            ts.append(flat[at : at + x.size])
            ts[-1].copy_(torch.from_numpy(x))
            at += x.size
        dev.append(ts)
    return host, dev


LIST_CASES = [
    # (numel, ranks, threshold bytes, binary16 tensors, compress)
    ([1, 2, 3, 1023, 1024, 1025, 4099, 70001], 2, 64 << 20, False, False),
    ([255, 256, 257, 5, 30000, 0, 9], 7, 40000, False, False),  # fused and direct
    ([255, 256, 257, 5, 30000, 0, 9], 8, 0, False, False),  # every tensor by itself
    ([513, 64, 64, 64, 40007], 16, 64 << 20, True, False),  # binary16 tensors
    ([513, 64, 64, 64, 40007], 33, 50000, False, True),  # compressed, fused and direct
    ([3, 900, 20001], 128, 30000, False, True),
    ([2000, 1, 3001], 24, 4096, True, False),
]


@pytest.mark.parametrize("layout", ["packed", "unalike"])
@pytest.mark.parametrize("case", range(len(LIST_CASES)))
def test_default_cycle_in_one_launch(case, layout):
    numel, n, threshold, half, compress = LIST_CASES[case]
    rng = np.random.default_rng(5200 + case)
    for op in ("average", "sum"):
        say(f"one-launch cycle case {case} {layout} {op}")
        host, dev = rank_lists(rng, n, numel, np.float16 if half else np.float32, layout)
        want = allreduce.allreduce(host, op, compress=compress, threshold=threshold)
        ar = hv.FusedAllreduce(dev, op=op, compress=compress, threshold_bytes=threshold)
        assert {k for k, _, _ in ar.kernel_sequence()} <= {"cycle_small", "ring_small"}
        ar()
        torch.cuda.synchronize()
        for r in range(n):
            for t in range(len(numel)):
                assert_bits_equal(dev[r][t].cpu().numpy(), want[r][t], f"rank {r} tensor {t}")


def test_steps_of_a_one_launch_object():
    """The pieces a one-launch object offers for tracing still run: per bucket the copies and the
    ring's halves, or the whole cycle, on buffers allocated when first asked for."""
    numel, n, threshold = [3000, 5, 257, 90000], 5, 40000
    rng = np.random.default_rng(5300)
    for compress in (False, True):
        for whole in (False, True):
            say(f"pieces of a one-launch object compress={compress} whole={whole}")
            host, dev = rank_lists(rng, n, numel, np.float32, "packed")
            ar = hv.FusedAllreduce(dev, compress=compress, threshold_bytes=threshold)
            s = torch.cuda.current_stream().cuda_stream
            for b in ar.buckets:
                if whole and not b.direct:
                    ar.fused_cycle(b, s)
                    continue
                if not b.direct:
                    ar.pack(b, s)
                ar.ring_phase(b, hv.PHASE_REDUCE_SCATTER, s)
                ar.ring_phase(b, hv.PHASE_ALLGATHER, s)
                if not b.direct:
                    ar.unpack(b, s)
            torch.cuda.synchronize()
            want = allreduce.allreduce(host, "average", compress=compress, threshold=threshold)
            for r in range(n):
                for t in range(len(numel)):
                    assert_bits_equal(dev[r][t].cpu().numpy(), want[r][t], f"rank {r} tensor {t}")


@pytest.mark.parametrize("n", [2, 5])
def test_cached_and_streamed_loads(n):
    """hvdx_fold_allreduce, and the ring on 2 ranks, load through the caches up to 272 MiB in all:
    either side of it, against the ring in steps."""
    for count in ((272 << 18) // n, (272 << 18) // n + 1000):
        say(f"cached and streamed loads n={n} count={count}")
        g = torch.Generator(device="cuda").manual_seed(n)
        want = [torch.empty(count, device="cuda").normal_(0.0, 0.01, generator=g) for _ in range(n)]
        rows = [[x.clone() for x in want] for _ in range(2)]
        s = torch.cuda.current_stream().cuda_stream
        hv.hvdx_ring_allreduce_steps([x.data_ptr() for x in want], n, count, hv.FLOAT32, hv.AVERAGE, 0, 0, 0, s)
        hv.hvdx_fold_allreduce([x.data_ptr() for x in rows[0]], n, count, hv.FLOAT32, hv.AVERAGE, 0, s)
        hv.hvdx_ring_allreduce([x.data_ptr() for x in rows[1]], n, count, hv.FLOAT32, hv.AVERAGE, 0, 0, 0, s)
        torch.cuda.synchronize()
        for got in rows:
            assert all(torch.equal(a.view(torch.int32), b.view(torch.int32)) for a, b in zip(got, want))


ALONE_CASES = [
    # (numel, ranks, threshold, binary16 tensors, compress, elements off a 16-byte start, launches without a table)
    ([17_000_001], 2, 64 << 20, False, False, 0, [0]),  # above 64 MiB a rank
    ([5, 17_000_000, 3001], 3, 1 << 20, False, True, 0, [1]),  # compressed; the others in a fusion buffer
    ([700, 900, 1000], 3, 2000, False, False, 0, []),  # three direct tensors share a table
    ([300, 900, 200], 3, 2000, False, False, 0, [1]),  # the only direct one
    ([900, 200], 2, 1000, True, False, 0, [0]),
    ([900], 2, 0, False, False, 1, []),  # off a 16-byte start: only a table's tiles make up for it
    ([900], 4, 0, False, False, 0, []),  # more ranks: a table does not count
    ([17_000_000, 60_000_000], 2, 64 << 20, False, False, 0, [0, 1]),  # past the Infinity Cache together
]


@pytest.mark.parametrize("case", range(len(ALONE_CASES)))
def test_direct_tensors_in_launches_of_their_own(case):
    """On 2 or 3 ranks a direct tensor above 64 MiB a rank, or the last one, needs no table cut and
    uploaded (a call made once pays for it): same bits as in a table."""
    numel, n, threshold, half, compress, off, want_alone = ALONE_CASES[case]
    say(f"direct tensors alone, case {case}")
    rng = np.random.default_rng(5400 + case)
    dtype = np.float16 if half else np.float32
    host = [[(rng.standard_normal(k) * 0.01).astype(dtype) for k in numel] for _ in range(n)]
    dev = [[to_gpu_rows(x[None], off)[0][0] for x in row] for row in host]
    ar = hv.FusedAllreduce(dev, compress=compress, threshold_bytes=threshold)
    ar()
    torch.cuda.synchronize()
    alone = [t for c in ar._cycles if c.table is None for i in c.members for t in ar.buckets[i].tensors]
    assert alone == want_alone
    assert len(ar.kernel_sequence()) == len(ar._cycles) <= 2
    want = native.allreduce(host, "average", compress=compress, threshold=threshold)
    graph = ar.capture()
    for replay in range(4):  # the call, then replays on fresh inputs
        for r in range(n):
            for t in range(len(numel)):
                assert_bits_equal(dev[r][t].cpu().numpy(), want[r][t], f"replay {replay} rank {r} tensor {t}")
                dev[r][t].copy_(torch.from_numpy(host[r][t]))
        graph.replay()
        torch.cuda.synchronize()
