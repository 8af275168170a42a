"""The one-launch broadcasts at the edges of their shapes: buffers and tensors shorter than a
16-byte unit, just under and over a stretch, starting anywhere in a cache line and differently
on each rank, lists long enough for several rounds of the tensor search, and each number of
units per lane.  Every byte against the root's, and the bytes around every copy untouched."""
import numpy as np
import pytest
import torch

import paper_1802_05799_amd as hv
from _gpu import assert_bits_equal, say
from test_gpu_broadcast import host_state, rank_buffers, tensor_views

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,root", [(2, 1), (3, 0), (5, 3), (9, 8), (17, 4), (128, 127)])
def test_flat(n, root):
    rng = np.random.default_rng(600 + n)
    for nbytes in (1, 15, 16, 17, 31, 1023, 1024, 1025, 2048 * 3 + 5, 4096 * 2 - 1):
        for offset in (0, 5, 16, 100):
            say(f"flat broadcast n={n} nbytes={nbytes} offset={offset}")
            x = rng.integers(0, 256, size=(n, nbytes), dtype=np.uint8)
            bases, views = rank_buffers(x, offset)
            hv.hvdx_broadcast([v.data_ptr() for v in views], n, nbytes, root)
            torch.cuda.synchronize()
            got = np.stack([v.cpu().numpy() for v in views])
            assert_bits_equal(got, np.broadcast_to(x[root], x.shape).copy())
            for b in bases:
                g = b.cpu().numpy()
                assert np.all(g[: 64 + offset] == 0xA5) and np.all(g[64 + offset + nbytes :] == 0xA5)


SIZES = {
    "short": [0, 1, 2, 15, 16, 17, 3, 0, 31, 33, 1],
    "stretch": [1023, 1, 1024, 4097, 2048, 16, 4095, 8200],
    "many": None,  # 5000 tensors of 0 to 40 bytes: three rounds of the search
}


@pytest.mark.parametrize("offsets", ["aligned", "anywhere"])
@pytest.mark.parametrize("kind", list(SIZES))
@pytest.mark.parametrize("n", [2, 6, 20])
def test_tensors(n, kind, offsets):
    rng = np.random.default_rng(700 + n)
    sizes = SIZES[kind] or rng.integers(0, 41, size=5000 if n == 2 else 300).tolist()
    off = rng.integers(0, 48, size=len(sizes)).tolist() if offsets == "anywhere" else [0] * len(sizes)
    root = n // 2
    say(f"tensor broadcast n={n} {kind} {offsets}")
    x = [[rng.integers(0, 256, size=s, dtype=np.uint8) for s in sizes] for _ in range(n)]
    for layout in ("object", "dense", "pages"):  # the one it chose, and either through the C entries
        bases, views = tensor_views(x, sizes, off)
        tb = hv.TensorBroadcast(views)
        if layout == "dense":
            hv.hvdx_broadcast_tensors(*tb._args, root, tb._stream(None))
        elif layout == "pages":
            starts, extent = hv._call_layout(sizes, [v.data_ptr() for v in views[0]], None, 1 << 60)
            table = torch.tensor(starts, dtype=torch.int64, device="cuda")
            hv.hvdx_broadcast_tensors_placed(*tb._args[:2], table.data_ptr(), len(sizes), extent, tb.total, n, root,
                                             tb._stream(None))
        else:
            tb(root)
        torch.cuda.synchronize()
        got = host_state(views)
        for r in range(n):
            for t in range(len(sizes)):
                assert_bits_equal(got[r][t], x[root][t], f"{layout} rank {r} tensor {t}")
        everything = torch.cat([b for row in bases for b in row]).cpu().numpy()
        at = 0
        for _ in range(n):
            for s, o in zip(sizes, off):
                g = everything[at : at + s + o + 96]
                assert np.all(g[: 48 + o] == 0x5A) and np.all(g[48 + o + s :] == 0x5A)
                at += s + o + 96


@pytest.mark.parametrize("n", [2, 4, 5, 20])
def test_large_lists_take_every_shape(n):
    """32 MB and more: four units per lane for few ranks, two, and one for many."""
    say(f"large tensor broadcast n={n}")
    sizes = [20_000_003, 5, 13_000_000, 4096]
    g = torch.Generator(device="cuda").manual_seed(n)
    rows = [[torch.randint(0, 256, (s,), dtype=torch.uint8, device="cuda", generator=g) for s in sizes] for _ in range(n)]
    want = [x.clone() for x in rows[1]]
    hv.broadcast_(rows, root=1)
    flat = [torch.randint(0, 256, (33_000_001,), dtype=torch.uint8, device="cuda", generator=g) for _ in range(n)]
    want_flat = flat[0].clone()
    hv.hvdx_broadcast([x.data_ptr() for x in flat], n, flat[0].numel(), 0, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert all(torch.equal(x, w) for row in rows for x, w in zip(row, want))
    assert all(torch.equal(x, want_flat) for x in flat)


def test_placed_with_empty_tensors_between():
    """hvdx_broadcast_tensors_placed with starts that are no multiples of 16, an empty tensor's
    (whose pointers are NULL) among them."""
    n, root = 3, 1
    sizes, starts = [20, 0, 100, 0], [0, 40, 4104, 4208]
    say("placed broadcast with empty tensors")
    rng = np.random.default_rng(810)
    x = [[rng.integers(0, 256, size=s, dtype=np.uint8) for s in sizes] for _ in range(n)]
    bases, views = tensor_views(x, sizes, [0, 0, 8, 0])
    ptrs = [v.data_ptr() if s else 0 for row in views for v, s in zip(row, sizes)]
    table = torch.tensor(ptrs + sizes + starts, dtype=torch.int64, device="cuda")
    at = table.data_ptr()
    hv.hvdx_broadcast_tensors_placed(at, at + 8 * n * 4, at + 8 * (n + 1) * 4, 4, 4208, 120, n, root,
                                     torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    got = host_state(views)
    assert all(np.array_equal(got[r][t], x[root][t]) for r in range(n) for t in range(4))
    for row, szs in zip(bases, [sizes] * n):
        for b, s, off in zip(row, szs, [0, 0, 8, 0]):
            g = b.cpu().numpy()
            assert np.all(g[: 48 + off] == 0x5A) and np.all(g[48 + off + s :] == 0x5A)
