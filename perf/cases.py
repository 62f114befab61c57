"""Workloads of the gradient-synchronization path, as a training program drives it.

A case is one pass through the public entry points: the ready marks of one iteration and the
finalizing call, one gradient-accumulation micro-step, a whole accumulate-then-synchronize
iteration, or the context-free call.  The parameter lists are the repository's own (the eight
small tensors, ResNet-50, BERT-large, whole or their first tensors) or generated ones with the
same make-up (weights of very different sizes, each followed by a bias); replica counts, element
types, bucket caps, pipelines and options span what the library accepts and is used with.

Keys of a case (all optional but "kind", "dtype", "R"):
  kind      "sync" | "accumulate" | "static"
  model     "tiny" | "resnet50" | "bert_large", with first = number of leading tensors (0 = all);
            or "generated" with tensors, elems (total), shape_seed
  dtype     0 binary32, 1 binary16, 2 bfloat16
  R         replicas
  cap       bucket cap in bytes
  pipeline  "fused" | "staged" (the library's default)
  marks     "each" = one call per gradient as a backward pass makes them, "many" = all in one call
  write_all every replica's tensors receive the average
  out32     16-bit gradients, binary32 averages in tensors of their own
  local     share of (replica, parameter) pairs that took part, or 0 = all of them
  unused    share of the parameters that are never marked
  micro     accumulation micro-steps in front of the synchronization
  dense     tensors packed without gaps (views into one flat buffer per replica) instead of at
            256-byte boundaries
  shift     replica r's buffer starts shift * (r mod 4) bytes later (ranks that place their flat
            buffers independently)
"""
import random

import numpy as np
import torch

import paper_2006_15704_amd as ddp
import workloads
from paper_2006_15704_amd import harness

MIB = 1 << 20
TORCH = {0: torch.float32, 1: torch.float16, 2: torch.bfloat16}
SIGMA = 1e-2


def listed():
    return [
        # the smallest synchronization a program makes: eight small tensors, two replicas, the
        # default pipeline, one ready mark per call
        {"name": "tiny_staged", "kind": "sync", "model": "tiny", "first": 0, "dtype": 0, "R": 2,
         "cap": 16384, "pipeline": "staged", "marks": "each"},
        # a small model synchronized by a caller that may not allocate
        {"name": "static_small", "kind": "static", "model": "resnet50", "first": 48, "dtype": 0, "R": 4,
         "cap": 1 * MIB},
        # the benchmark's shapes at its defaults: gradients are marked as a backward pass makes them
        {"name": "resnet50_r8", "kind": "sync", "model": "resnet50", "first": 0, "dtype": 0, "R": 8,
         "cap": 25 * MIB, "pipeline": "fused", "marks": "each"},
        {"name": "bert_large_r8", "kind": "sync", "model": "bert_large", "first": 0, "dtype": 0, "R": 8,
         "cap": 25 * MIB, "pipeline": "fused", "marks": "each"},
        # a program that changes no option: the staged pipeline, all marks after the backward pass
        {"name": "resnet50_staged", "kind": "sync", "model": "resnet50", "first": 0, "dtype": 0, "R": 8,
         "cap": 25 * MIB, "pipeline": "staged", "marks": "many"},
        # the small-bucket end of the bucket-size sweep: many short launches
        {"name": "resnet50_fp16_r16_cap1", "kind": "sync", "model": "resnet50", "first": 0, "dtype": 1, "R": 16,
         "cap": 1 * MIB, "pipeline": "fused", "marks": "each"},
        # gradients sent in bfloat16, averages kept in binary32
        {"name": "bert_bf16_out32", "kind": "sync", "model": "bert_large", "first": 0, "dtype": 2, "R": 8,
         "cap": 25 * MIB, "pipeline": "fused", "marks": "each", "out32": True},
        # replicas whose forward passes took different branches: per-replica participation
        {"name": "resnet50_partial", "kind": "sync", "model": "resnet50", "first": 0, "dtype": 0, "R": 8,
         "cap": 25 * MIB, "pipeline": "fused", "marks": "each", "local": 0.7},
        # one accumulation micro-step by itself (gradient accumulation in bfloat16)
        {"name": "accumulate_bf16", "kind": "accumulate", "model": "resnet50", "first": 0, "dtype": 2, "R": 8,
         "cap": 25 * MIB},
        # four accumulated micro-steps, then one synchronization over 32 replicas in which a tenth
        # of the parameters took no part (the first two layers of the BERT-large list)
        {"name": "no_sync_r32", "kind": "sync", "model": "bert_large", "first": 37, "dtype": 0, "R": 32,
         "cap": 25 * MIB, "pipeline": "fused", "marks": "many", "unused": 0.1, "micro": 4},
        # odd sizes packed without gaps, the ranks' flat buffers placed independently
        {"name": "ragged_r8", "kind": "sync", "model": "generated", "tensors": 90, "elems": 30000001, "shape_seed": 5,
         "dtype": 0, "R": 8, "cap": 25 * MIB, "pipeline": "fused", "marks": "many", "dense": True, "shift": 4},
        # every rank's tensors receive the average
        {"name": "write_all_bf16_r4", "kind": "sync", "model": "bert_large", "first": 101, "dtype": 2, "R": 4,
         "cap": 25 * MIB, "pipeline": "fused", "marks": "many", "write_all": True},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["sync"] * 8 + ["accumulate", "static"])
    dtype = rng.choice([0, 0, 1, 2])
    es = 4 if dtype == 0 else 2
    case = {"kind": kind, "dtype": dtype, "R": rng.choice([2, 3, 4, 5, 8, 8, 8, 12, 16, 16, 24, 32, 64]),
            "model": "generated", "shape_seed": rng.randrange(1 << 20)}
    if kind == "static":
        # the call's limit: (R + 1) x the gradients within its 32 MiB
        case["elems"] = _log_uniform(rng, 20000, 24 * MIB // (es * (case["R"] + 1)))
        case["tensors"] = rng.randrange(2, 60)
        case["cap"] = _log_uniform(rng, 16384, 4 * MIB)
        return case
    case["elems"] = _log_uniform(rng, 20000, 6 * 10 ** 9 // (es * (case["R"] + 1)))
    case["tensors"] = rng.randrange(4, 240)
    case["cap"] = _log_uniform(rng, 256 * 1024, 100 * MIB)
    if rng.random() < 0.3:
        case["dense"] = True
        if rng.random() < 0.5:
            case["shift"] = rng.choice([es, 8])
    if kind == "accumulate":
        return case
    case["pipeline"] = rng.choice(["fused", "fused", "staged"])
    case["marks"] = rng.choice(["each", "each", "many"])
    extra = rng.choice(["", "", "", "write_all", "out32", "local", "unused", "micro"])
    if extra == "out32":
        if dtype != 0 and case["pipeline"] == "fused":
            case["out32"] = True
    elif extra == "write_all":
        case["write_all"] = True
    elif extra == "local":
        case["local"] = rng.choice([0.5, 0.8, 0.95])
        case["marks"] = "each"
    elif extra == "unused":
        case["unused"] = 0.1
    elif extra == "micro":
        case["micro"] = rng.choice([1, 2, 4])
    return case


def _numel(case):
    if case["model"] != "generated":
        numel = workloads.numel_of(workloads.WORKLOAD_SHAPES[case["model"]]())
        return numel[:case["first"]] if case.get("first") else numel
    # weights whose sizes spread over three decades, each followed by a small vector
    rng = random.Random(case["shape_seed"])
    size = [10.0 ** rng.uniform(0.0, 3.0) if i % 2 == 0 else 0.02 * 10.0 ** rng.uniform(0.0, 1.5)
            for i in range(case["tensors"])]
    scale = case["elems"] / sum(size)
    return [max(1, int(s * scale)) for s in size]


class _State:
    def __init__(self):
        self.session = None

    def __del__(self):
        if self.session is not None:
            self.session.close()
            self.session = None


_streams = []      # the program's reduction and backward stream: made once, shared by its contexts


def _stream_pair():
    if not _streams:
        g = harness.DeviceGrads([256], [0], 2, fill=0)
        with harness.Session(g, MIB, ddp.DDP_PIPELINE_FUSED) as s:
            _streams.extend((s.reduce_stream, s.backward_stream))
    return tuple(_streams)


def _typed(grads, r, dtype):
    """Replica r's whole buffer as elements of its type."""
    buf = grads.bufs[r]
    es = harness.ESIZE[dtype]
    return buf[:buf.numel() // es * es].view(TORCH[dtype])


def _gradients(case, numel, seed, salt, R=None, dtype=None, fill=None):
    dtype = case["dtype"] if dtype is None else dtype
    R = case["R"] if R is None else R
    es = harness.ESIZE[dtype]
    shift = case.get("shift", 0) * es // harness.ESIZE[case["dtype"]]
    grads = harness.DeviceGrads(numel, [dtype] * len(numel), R, align=es if case.get("dense") else 256,
                                replica_skew=[shift * (r % 4) for r in range(R)] if shift else None, fill=fill)
    if fill is None:
        gen = torch.Generator("cuda")
        for r in range(R):
            gen.manual_seed((seed * 1000003 + salt * 4099 + r) % (1 << 62))
            grads.bufs[r].fill_(0)
            _typed(grads, r, dtype).normal_(0.0, SIGMA, generator=gen)
    return grads


def _participation(case, n, seed):
    """(parameters in ready order, [n][R] flags or None): drawn from the seed."""
    rng = np.random.default_rng([seed, 77])
    order = list(range(n - 1, -1, -1))
    flags = None
    if case.get("unused"):
        absent = set(int(i) for i in rng.choice(n, size=max(1, int(n * case["unused"])), replace=False))
        order = [i for i in order if i not in absent]
    if case.get("local"):
        flags = (rng.random((n, case["R"])) < case["local"]).astype(np.uint8)
    return order, flags


def prepare(case, seed):
    numel = _numel(case)
    n, R, dtype = len(numel), case["R"], case["dtype"]
    st = _State()
    st.case, st.numel = case, numel
    st.grads = _gradients(case, numel, seed, 1)
    st.order, st.flags = _participation(case, n, seed)
    if st.flags is not None:
        st.flag_rows = [[int(u) for u in row] for row in st.flags]
    st.micro = None
    if case["kind"] == "accumulate" or case.get("micro"):
        st.micro = _gradients(case, numel, seed, 2)
        present = set(st.order)
        st.micro_ptrs = [p if k % n in present else None for k, p in enumerate(st.micro.ptrs())]
    st.outputs = None
    if case["kind"] == "static":
        st.ptrs = st.grads.ptrs()
        st.stream = _stream_pair()[1]
        st.results = _results(st)
        return st
    if case.get("out32"):
        st.outputs = _gradients(case, numel, seed, 3, R=1, dtype=0, fill=0)
    pipeline = ddp.DDP_PIPELINE_STAGED if case.get("pipeline") == "staged" else ddp.DDP_PIPELINE_FUSED
    st.session = harness.Session(st.grads, case["cap"], pipeline, write_all=bool(case.get("write_all")),
                                 streams=_stream_pair(), outputs=st.outputs)
    if case.get("local"):
        ddp.ddp_set_option(st.session.ctx, ddp.DDP_OPT_FIND_UNUSED, 1)
    st.results = _results(st)
    return st


def _results(st):
    case = st.case
    if st.outputs is not None:
        return [_typed(st.outputs, 0, 0)]
    if case["kind"] == "accumulate" or case.get("micro") or case.get("write_all"):
        return [_typed(st.grads, r, case["dtype"]) for r in range(case["R"])]
    return [_typed(st.grads, 0, case["dtype"])]


def run(st):
    case = st.case
    if case["kind"] == "static":
        ddp.ddp_sync_static(case["R"], 0, st.stream.cuda_stream, st.numel, st.grads.dtype, st.ptrs, case["cap"])
        return st.results
    ctx = st.session.ctx
    if case["kind"] == "accumulate":
        ddp.ddp_no_sync_accumulate(ctx, st.micro_ptrs)
        return st.results
    for _ in range(case.get("micro", 0)):
        ddp.ddp_no_sync_accumulate(ctx, st.micro_ptrs)
    if st.flags is not None:
        for p in st.order:
            ddp.ddp_mark_ready_local(ctx, p, st.flag_rows[p])
    elif case["marks"] == "each":
        for p in st.order:
            ddp.ddp_mark_ready(ctx, p)
    else:
        ddp.ddp_mark_ready_many(ctx, st.order)
    ddp.ddp_finalize_backward(ctx)
    return st.results


def work(case):
    es = harness.ESIZE[case["dtype"]]
    elems, R = sum(_numel(case)), case["R"]
    if case["kind"] == "accumulate":
        return {"bytes": 3 * R * es * elems, "flops": R * elems}
    part = 1.0 - case.get("unused", 0.0)
    micro = case.get("micro", 0)
    read = part * (case.get("local") or 1.0) * R * es
    write = 4 if case.get("out32") else es * (R if case.get("write_all") else 1)
    return {"bytes": elems * (read + write + micro * part * 3 * R * es), "flops": elems * R * (1 + micro)}


def tolerance(case):
    # binary32: one rounding per addition over up to 64 terms; 16-bit results: one rounding to
    # storage (and one per accumulation step), about 1.7e-3 of a bfloat16 and 2.1e-4 of a binary16
    if case["dtype"] == 0 or case.get("out32"):
        return {"rel": 1e-6, "max": 1e-4}
    return {"rel": 8e-3, "max": 5e-2} if case["dtype"] == 2 else {"rel": 1e-3, "max": 1e-2}


def exact(case, seed):
    """The same results in 64 bits, tensor by tensor with plain torch."""
    numel = _numel(case)
    n, R, dtype = len(numel), case["R"], case["dtype"]
    es = harness.ESIZE[dtype]
    grads = _gradients(case, numel, seed, 1)
    order, flags = _participation(case, n, seed)
    present = set(order)
    micro = _gradients(case, numel, seed, 2) if case["kind"] == "accumulate" or case.get("micro") else None
    steps = 1 if case["kind"] == "accumulate" else case.get("micro", 0)

    def tensor(g, r, i):
        o = g.offsets[i] + g.replica_skew[r]
        return g.bufs[r][o:o + g.nbytes(i)].view(torch.uint8).clone().view(TORCH[dtype]).double()

    out32 = case.get("out32")
    if out32:
        into = _gradients(case, numel, seed, 3, R=1, dtype=0, fill=0)
        result = [_typed(into, 0, 0).double()]
    else:
        into = grads
        every = micro is not None or case.get("write_all")
        result = [_typed(grads, r, dtype).double() for r in range(R if every else 1)]

    def put(r, i, value):
        size = 4 if out32 else es
        o = (into.offsets[i] + into.replica_skew[r]) // size
        result[r][o:o + numel[i]] = value

    for i in range(n):
        if case["kind"] == "accumulate":
            for r in range(R):
                put(r, i, tensor(grads, r, i) + tensor(micro, r, i))
            continue
        users = [r for r in range(R) if i in present and (flags is None or flags[i][r])]
        total = torch.zeros(numel[i], dtype=torch.float64, device="cuda")
        for r in users:
            x = tensor(grads, r, i)
            if steps:
                x = x + steps * tensor(micro, r, i)
                put(r, i, x)
            total += x
        if not users and case.get("local"):
            continue                      # nobody used it: its gradients stay as they are
        for r in range(R if case.get("write_all") else 1):
            put(r, i, total / R)
    return result
