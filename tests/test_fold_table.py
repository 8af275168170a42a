"""The table of the one-launch cycle (hvdx_fuse_cycle_table), on the CPU: its tiles cover every
element of every tensor once, inside one ring chunk each, with the chunk's first rank, and a
tile marked aligned lies on a 16-byte boundary of every rank's tensor from its head's end on."""
import struct

import numpy as np
import pytest

import paper_1802_05799_amd as hv

LISTS = [[7, 64, 100, 1000, 4608, 4096, 513, 10000], [1], [0, 3, 0, 5], [2048 * 3, 5, 4096 * 2 + 3, 1, 9000],
         [33] * 90 + [12000], [100003]]
PAD = 16  # zero pointers after the tensors'
LAYOUTS = ["aligned", "packed", "unalike"]


def read_table(table, nt, n, ntiles):
    ptrs = np.frombuffer(table, dtype=np.uint64, count=nt * 2 * n).reshape(nt, 2 * n)
    tiles = []
    for i in range(ntiles):
        li, t, bits = struct.unpack_from("<qiI", table, (nt * 2 * n + PAD) * 8 + 16 * i)
        tiles.append((li, t, bits & 0xFFFF, bits >> 16 & 0xFF, bits >> 24 & 1, bits >> 28))
    assert not np.frombuffer(table, dtype=np.uint64, count=PAD, offset=nt * 2 * n * 8).any()
    return ptrs, tiles


def addresses(numel, n, es, layout):
    """Made-up device addresses, rank-major."""
    out = []
    for r in range(n):
        at = (r + 1) << 36
        for t, k in enumerate(numel):
            if layout == "aligned":
                at = -(-at // 256) * 256
            elif layout == "unalike":
                at += es * (r + t)
            out.append(at)
            at += k * es
    return out


@pytest.mark.parametrize("layout", LAYOUTS)
@pytest.mark.parametrize("types", [(4, 4), (4, 2), (2, 2)], ids=["f32", "f32-to-f16", "f16"])
def test_tiles_cover_every_element_once(types, layout):
    te, be = types
    dt = {4: hv.FLOAT32, 2: hv.FLOAT16}
    V = 16 // te
    seen = set()
    for numel in LISTS:
        for n in (2, 3, 8, 17, 128):
            for threshold in (0, 4096, 64 << 20):
                bucket_of, offset, counts, _ = hv.hvdx_fuse_plan(numel, dt[be], threshold)
                ptrs = addresses(numel, n, te, layout)
                table, ntiles, stretches = hv.hvdx_fuse_cycle_table(ptrs, numel, offset, bucket_of, counts, dt[te], dt[be], n)
                got, tiles = read_table(table, len(numel), n, ntiles)
                want = np.array(ptrs, dtype=np.uint64).reshape(n, len(numel)).T
                assert np.array_equal(got, np.concatenate([want, want], axis=1))
                hits = [np.zeros(k, np.int64) for k in numel]
                for li, t, length, chunk, aligned, head in tiles:
                    assert 1 <= length <= stretches * 64 * V and li + length <= numel[t]
                    hits[t][li : li + length] += 1
                    start, size = hv.hvdx_ring_chunk(counts[bucket_of[t]], n, chunk)
                    p = offset[t] + li
                    assert start <= p and p + length <= start + size
                    assert head < V and (aligned or head == 0)
                    if aligned:
                        assert all((ptrs[r * len(numel) + t] + (li + head) * te) % 16 == 0 for r in range(n))
                assert all((h == 1).all() for h in hits)
                if layout != "unalike":  # in wide tiles only what comes before a 16-byte boundary is not aligned
                    assert all(aligned or stretches > 1 and length < V for _, _, length, _, aligned, _ in tiles)
                if stretches > 1:  # whose wavefronts would each have a head
                    assert not any(head for *_, head in tiles)
                seen.add(stretches)
    assert seen == {1, 4}


def test_table_argument_errors():
    ok = dict(tensors=[1 << 32, 1 << 33], numel=[5], offset=[0], bucket_of=[0], bucket_count=[5],
              tensor_dtype=hv.FLOAT32, buf_dtype=hv.FLOAT32, nranks=2)
    hv.hvdx_fuse_cycle_table(**ok)
    for bad, status in (({"tensors": [1 << 32, 0]}, hv.ERR_INVALID), ({"tensors": [1 << 32, 2]}, hv.ERR_INVALID),
                        ({"offset": [1]}, hv.ERR_INVALID), ({"bucket_of": [1]}, hv.ERR_INVALID),
                        ({"numel": [-1]}, hv.ERR_INVALID), ({"nranks": 0}, hv.ERR_INVALID),
                        ({"tensor_dtype": 9}, hv.ERR_INVALID), ({"bucket_count": [-1]}, hv.ERR_INVALID),
                        ({"tensor_dtype": hv.FLOAT16}, hv.ERR_UNSUPPORTED)):
        with pytest.raises(hv.HvdxError) as e:
            hv.hvdx_fuse_cycle_table(**{**ok, **bad})
        assert e.value.status == status, bad
    huge = dict(tensors=[1 << 32] * 34, numel=[1 << 59] * 17, offset=[0] * 17, bucket_of=list(range(17)),
                bucket_count=[1 << 59] * 17)
    with pytest.raises(hv.HvdxError) as e:  # more elements than their sum holds
        hv.hvdx_fuse_cycle_table(**{**ok, **huge})
    assert e.value.status == hv.ERR_INVALID
    for args in ((0, 1, 4, 4, 9, hv.FLOAT32, hv.FLOAT32, 2, hv.SUM, False),
                 (256, 1, 4, 4, 9, hv.FLOAT32, hv.FLOAT32, 129, hv.SUM, False),
                 (256, 1, 4, 4, 9, hv.FLOAT32, 7, 2, hv.SUM, False), (256, 1, 4, 4, 9, hv.FLOAT32, hv.FLOAT32, 2, 5, False),
                 (264, 1, 4, 4, 9, hv.FLOAT32, hv.FLOAT32, 2, hv.SUM, False),
                 (256, 1, 4, 2, 9, hv.FLOAT32, hv.FLOAT32, 2, hv.SUM, False),
                 (256, 1, -1, 4, 9, hv.FLOAT32, hv.FLOAT32, 2, hv.SUM, False)):
        with pytest.raises(hv.HvdxError) as e:
            hv.hvdx_fuse_cycle(*args)
        assert e.value.status == hv.ERR_INVALID
    hv.hvdx_fuse_cycle(0, 0, 0, 1, 0, hv.FLOAT32, hv.FLOAT32, 2, hv.SUM, False)  # nothing to do
