"""Performance cases of the data-parallel hot path, through its public entry points.

Three ways a program uses the library:

* "list": per-rank lists of gradient tensors, reduced in place by `FusedAllreduce` (plan
  built once, called every training step);
* "flat": one flat gradient buffer per rank, reduced in place through the C ABI
  (`hvdx_ring_allreduce`, or `hvdx_ring_allreduce_small` where the header recommends it);
* "broadcast": rank 0's parameter tensors copied to every rank by `TensorBroadcast`.

A rank's tensors are views into one flat storage: "aligned" starts each tensor on a
256-byte boundary, as an allocator does; "packed" lays them end to end, as views of one
flattened parameter buffer are (16-byte alignment is then a matter of luck).  A pass
returns every rank's whole storage, gaps included (nothing may write them).

A case's values: `shape` is one of the repository's models or "ragged" (sizes from
`shape_seed`, log-uniform, many small and a few large, `elements` in all); `dtype` "f32" or
"f16"; `compress` sends binary32 gradients as binary16; `threshold` is the fusion buffer's
size in bytes (0: every tensor is reduced by itself).
"""
import random

import torch

import paper_1802_05799_amd as hv
from workloads import configs

MIB = 1 << 20
_TORCH = {"f32": torch.float32, "f16": torch.float16}
_HVDX = {"f32": hv.FLOAT32, "f16": hv.FLOAT16}
_OP = {"average": hv.AVERAGE, "sum": hv.SUM}


def _list(name, shape, ranks, **kw):
    case = {"name": name, "use": "list", "shape": shape, "shape_seed": 0, "elements": 0, "ranks": ranks, "dtype": "f32",
            "compress": False, "op": "average", "threshold": 64 * MIB, "layout": "aligned"}
    case.update(kw)
    return case


def listed():
    return [
        # the smallest step: a toy model on four workers, where a call is all latency
        _list("tiny_n4", "tiny", 4),
        # a small model's 1.2 MB of ragged gradients, views of a flattened buffer, summed by three workers
        _list("ragged_small_n3_sum", "ragged", 3, shape_seed=1, elements=300_007, op="sum", layout="packed"),
        # a mid-sized one on six workers: the average is a true division, odd sizes, unaligned views
        _list("ragged_mid_n6", "ragged", 6, shape_seed=2, elements=5_000_011, layout="packed"),
        # the benchmark's ordinary workloads: ResNet-50 on 8 workers, Inception-V3 on 16
        _list("resnet50_n8", "resnet50", 8),
        _list("inceptionv3_n16", "inceptionv3", 16),
        # half-precision gradients, as mixed-precision training hands over
        _list("resnet50_f16_n8", "resnet50", 8, dtype="f16"),
        # Tensor Fusion switched off (the benchmark's ablation): 284 tensors, each on its own
        _list("inceptionv3_unfused_n16", "inceptionv3", 16, threshold=0),
        # the headline: VGG-16 on 32 workers, one tensor larger than the fusion buffer
        _list("vgg16_n32", "vgg16", 32),
        # the same gradients on 64 workers with fp16 compression, the largest case
        _list("vgg16_fp16_n64", "vgg16", 64, compress=True),
        # the C ABI on one flat buffer per rank, an odd count of elements
        {"name": "flat_ring_n8", "use": "flat", "elements": 25_557_033, "ranks": 8, "dtype": "f32", "compress": False,
         "op": "average"},
        # the start of training: every parameter of ResNet-50 from rank 0 to 8 workers
        {"name": "broadcast_resnet50_n8", "use": "broadcast", "shape": "resnet50", "shape_seed": 0, "elements": 0,
         "ranks": 8, "dtype": "f32", "layout": "aligned"},
        # ... and of a small model, where the chain's launches count
        {"name": "broadcast_small_n6", "use": "broadcast", "shape": "ragged", "shape_seed": 3, "elements": 100_003,
         "ranks": 6, "dtype": "f32", "layout": "packed"},
    ]


_MOST = 138_357_544 * 32  # elements of all ranks: no drawn case is larger than the headline


def draw(rng):
    use = rng.choice(["list", "list", "list", "list", "flat", "broadcast"])
    ranks = rng.choice([2, 3, 4, 5, 6, 7, 8, 8, 12, 16, 16, 24, 32, 48, 64])
    elements = int(10 ** rng.uniform(4.0, 8.0)) | 1
    while elements * ranks > _MOST:
        elements = elements // 2 | 1
    case = {"use": use, "elements": elements, "ranks": ranks, "dtype": rng.choice(["f32", "f32", "f32", "f16"])}
    if use != "broadcast":
        case["compress"] = case["dtype"] == "f32" and rng.random() < 0.25
        case["op"] = rng.choice(["average", "average", "sum"])
        if case["dtype"] == "f16" or case["compress"]:
            case["op"] = "average"  # binary16 sums of repeated passes would overflow
    if use != "flat":
        case["shape"] = rng.choice(["ragged", "ragged", "ragged", "resnet50", "inceptionv3", "vgg16"])
        if case["shape"] != "ragged":
            case["elements"] = 0
            if case["shape"] == "vgg16":
                case["ranks"] = min(ranks, 32)
        case["shape_seed"] = rng.randrange(1, 1 << 20)
        case["layout"] = rng.choice(["aligned", "packed"])
    if use == "list":
        case["threshold"] = rng.choice([0, MIB, 16 * MIB, 64 * MIB, 64 * MIB, 64 * MIB])
    return case


def _numel(case):
    if case["use"] == "flat":
        return [case["elements"]]
    if case["shape"] != "ragged":
        return configs.get(case["shape"]).numel()
    rng = random.Random(case["shape_seed"])
    left, out = case["elements"], []
    largest = max(8, left // 4)
    while left > 0:
        k = min(left, max(1, int(largest ** rng.random())))
        if len(out) >= 400:
            k = left
        out.append(k)
        left -= k
    return out


def _starts(case, numel):
    if case["use"] == "flat" or case["layout"] == "packed":
        step = 1
    else:
        step = 256 // _TORCH[case["dtype"]].itemsize
    starts, end = [], 0
    for k in numel:
        starts.append(end)
        end += -(-k // step) * step
    return starts, end


def _storage(case, seed, rank, size):
    """Rank `rank`'s values: gradients N(0, 0.01), the toy model's uniform in (-1, 1)."""
    x = torch.empty(size, dtype=_TORCH[case["dtype"]], device="cuda")
    g = torch.Generator(device="cuda").manual_seed(seed * 1009 + rank)
    if case.get("shape") == "tiny":
        return x.uniform_(-1.0, 1.0, generator=g)
    return x.normal_(0.0, 0.01, generator=g)


def prepare(case, seed):
    numel = _numel(case)
    starts, size = _starts(case, numel)
    n = case["ranks"]
    storage = [_storage(case, seed, r, size) for r in range(n)]
    state = {"use": case["use"], "storage": storage}
    if case["use"] == "flat":
        count, dtype, op = numel[0], _HVDX[case["dtype"]], _OP[case["op"]]
        compress = hv.COMPRESS_FP16 if case["compress"] else hv.COMPRESS_NONE
        ptrs = [x.data_ptr() for x in storage]
        if not compress and count * storage[0].element_size() <= hv.SMALL_BUCKET_BYTES:
            state["small"], state["args"] = True, (ptrs, n, count, dtype, op)
            return state
        need = hv.hvdx_ring_workspace_bytes(n, count, dtype, compress)
        state["workspace"] = torch.empty(max(need, 1), dtype=torch.uint8, device="cuda")
        state["small"] = False
        state["args"] = (ptrs, n, count, dtype, op, compress, state["workspace"].data_ptr() if need else 0, need)
        return state
    per_rank = [[x[s : s + k] for s, k in zip(starts, numel)] for x in storage]
    if case["use"] == "broadcast":
        state["call"] = hv.TensorBroadcast(per_rank)
    else:
        state["call"] = hv.FusedAllreduce(per_rank, op=case["op"], compress=case["compress"],
                                          threshold_bytes=case["threshold"])
    return state


def run(state):
    if state["use"] == "flat":
        stream = torch.cuda.current_stream().cuda_stream
        if state["small"]:
            hv.hvdx_ring_allreduce_small(*state["args"], stream)
        else:
            hv.hvdx_ring_allreduce(*state["args"], stream)
    else:
        state["call"]()
    return state["storage"]


def work(case):
    """Each rank's elements read once (the root's, for a broadcast) and every rank's written once."""
    numel, n = sum(_numel(case)), case["ranks"]
    size = _TORCH[case["dtype"]].itemsize
    if case["use"] == "broadcast":
        return {"bytes": n * numel * size, "flops": 0}
    return {"bytes": 2 * n * numel * size, "flops": n * numel}


def tolerance(case):
    """The sums are specified bit for bit: ring order from the chunk's first rank, each
    addition rounded in the buffer's type, one division.  A broadcast copies bytes."""
    return "exact"


_CHECKED = 4  # ranks compared with 64 bits: every rank ends with the same values


def exact(case, seed):
    numel = _numel(case)
    starts, size = _starts(case, numel)
    n = case["ranks"]
    keep = min(n, _CHECKED)
    first = [_storage(case, seed, r, size).double() for r in range(keep)]
    if case["use"] == "broadcast":
        total = first[0]
    else:
        total = torch.zeros(size, dtype=torch.float64, device="cuda")
        for r in range(n):
            total += first[r] if r < keep else _storage(case, seed, r, size).double()
        if case["op"] == "average":
            total /= n
    inside = torch.zeros(size, dtype=torch.bool, device="cuda")
    for s, k in zip(starts, numel):
        inside[s : s + k] = True
    return [torch.where(inside, total, x) for x in first] + [None] * (n - keep)
