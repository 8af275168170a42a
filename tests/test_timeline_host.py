"""Timeline host logic: the per-rank chunk labels follow the ring schedule, and the
C entry points refuse misuse without touching the GPU."""
import pytest

import paper_1802_05799_amd as hv
from oracle import ring
from paper_1802_05799_amd.timeline import chunks_of_step


def test_chunk_labels_follow_the_oracle_schedule():
    for n in (2, 3, 5, 8, 17):
        for s in range(n - 1):
            for r in range(n):
                sent, recv = chunks_of_step(hv._lib.KERNEL_REDUCE_SCATTER, s, r, n)
                assert ring.rs_sender(sent, s, n) == r and ring.rs_receiver(sent, s, n) == (r + 1) % n
                assert ring.rs_receiver(recv, s, n) == r and ring.rs_sender(recv, s, n) == (r - 1) % n
                sent, recv = chunks_of_step(hv._lib.KERNEL_ALLGATHER, s, r, n)
                assert ring.ag_sender(sent, s, n) == r and ring.ag_receiver(sent, s, n) == (r + 1) % n
                assert ring.ag_receiver(recv, s, n) == r and ring.ag_sender(recv, s, n) == (r - 1) % n


def test_timeline_refuses_misuse():
    with pytest.raises(hv.HvdxError):
        hv.hvdx_timeline_end(4)  # nothing recording
    with pytest.raises(hv.HvdxError):
        hv.hvdx_timeline_begin(0)
    with pytest.raises(hv.HvdxError):
        hv.hvdx_timeline_begin(-5)


def test_broadcast_labels_follow_the_oracle_chain():
    import numpy as np

    from oracle import broadcast
    from paper_1802_05799_amd.timeline import broadcast_step_args

    for n in (2, 3, 5):
        for root in range(n):
            x = np.zeros((n, 16 * n), np.uint8)
            for r in range(n):
                x[r] = r + 1
            chunks = broadcast.chunk_bytes(16 * n, n)
            prev = x.copy()
            seen = []
            broadcast.chain_broadcast(x, root, observe=lambda s, b: seen.append(b.copy()))
            for s, cur in enumerate(seen):
                for r in range(n):
                    args = broadcast_step_args(s, r, root, n)
                    changed = [j for j, (lo, hi) in enumerate(chunks) if not np.array_equal(cur[r, lo:hi], prev[r, lo:hi])]
                    if changed:
                        assert args.get("recv chunk") == changed[0] and len(changed) == 1
                prev = cur


def test_whole_broadcast_labels_cover_the_chain():
    """A broadcast in one launch (step -1): every rank's track names the chunks it sends and
    receives and in which steps, the union of its steps' labels."""
    from paper_1802_05799_amd.timeline import broadcast_step_args

    for n in (2, 3, 5, 8):
        for root in range(n):
            for r in range(n):
                whole = broadcast_step_args(-1, r, root, n)
                steps = [broadcast_step_args(s, r, root, n) for s in range(2 * n - 2)]
                for way, end in (("send", "to"), ("recv", "from")):
                    at = [(s, a[f"{way} chunk"]) for s, a in enumerate(steps) if f"{way} chunk" in a]
                    if not at:
                        assert end not in whole and f"{way} chunks" not in whole
                        continue
                    assert whole[end] == next(a[end] for a in steps if end in a)
                    assert [j for _, j in at] == list(range(n)) and whole[f"{way} chunks"] == f"0-{n - 1}"
                    assert whole[f"{way} steps"] == f"{at[0][0]}-{at[-1][0]}"
                assert whole  # every rank of a chain of two or more sends or receives


def test_one_launch_ring_labels_name_every_steps_chunks():
    """A ring in one launch: a rank's track still says which chunk it sends and receives in
    every step, as the first steps' chunks from which each further step counts down."""
    from paper_1802_05799_amd.timeline import whole_ring_args

    assert whole_ring_args(0, 1) == {}  # one rank sends nothing
    for n in (2, 3, 5, 8, 17):
        for r in range(n):
            args = whole_ring_args(r, n)
            assert args["to"] == (r + 1) % n and args["from"] == (r - 1) % n
            for phase, kind in (("adding", hv._lib.KERNEL_REDUCE_SCATTER), ("replacing", hv._lib.KERNEL_ALLGATHER)):
                assert args[f"{phase} steps"] == f"0-{n - 2}, each one chunk lower (mod {n})"
                sent, recv = args[f"{phase}: first chunk sent"], args[f"{phase}: first chunk received"]
                for s in range(n - 1):
                    assert ((sent - s) % n, (recv - s) % n) == chunks_of_step(kind, s, r, n)
