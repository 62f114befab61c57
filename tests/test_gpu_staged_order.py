"""GPU parity of launch ordering, the staged pipeline's above all, by device flags and by events: gradients start as NaN
and are produced by the synthetic backward stream after a delay, so a launch that ran ahead of its
gate, or one that was skipped and not repaired, shows in the flat buckets and in the results.  A
gate wait of 0 makes every gate give up without waiting (every kernel still ends normally)."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

FP32, FP16, BF16 = 0, 1, 2
STAGED = 0


def lib():
    import paper_2006_15704_amd as d
    from paper_2006_15704_amd import harness
    return d, harness


def flag_ordered_session(d, harness, grads, cap, pipeline):
    import torch
    streams = None
    for _ in range(8):           # a pair of streams on separate hardware queues, if there is one
        s = harness.Session(grads, cap, pipeline, streams=streams)
        if d.ddp_get_option(s.ctx, d.DDP_OPT_FLAG_ORDER):
            return s
        s.close()
        streams = (torch.cuda.Stream(), torch.cuda.Stream())
    pytest.skip("no pair of streams on separate hardware queues was found")


@pytest.mark.parametrize("dtype", [FP32, FP16, BF16])
@pytest.mark.parametrize("gate_wait_us", [100000, 0])
@pytest.mark.parametrize("tail_on_backward", [1, 0])
@pytest.mark.parametrize("R", [3, 17])         # 17: copied and reduced in two passes
def test_staged_launches_wait_for_the_backward_stream(dtype, gate_wait_us, tail_on_backward, R):
    staged_launches_wait(dtype, gate_wait_us, tail_on_backward, by_flag=True, R=R)


@pytest.mark.parametrize("dtype", [FP32, FP16, BF16])
@pytest.mark.parametrize("streams", [1, 2])
@pytest.mark.parametrize("tail_on_backward", [1, 0])
def test_staged_launches_ordered_by_events_wait_for_the_backward_stream(dtype, streams, tail_on_backward):
    staged_launches_wait(dtype, 100000, tail_on_backward, by_flag=False, streams=streams)


def staged_launches_wait(dtype, gate_wait_us, tail_on_backward, by_flag, streams=2, R=3):
    d, harness = lib()
    import torch
    numel = [5, 3000, 3 * 4096 + 7, 8192, 1, 777, 2 * 8192, 4000, 60, 5000]
    n, cap = len(numel), 32 << 10
    es = 4 if dtype == FP32 else 2
    dtypes = [dtype] * n
    grads = harness.DeviceGrads(numel, dtypes, R, fill=0xFF)
    keep = harness.DeviceGrads(numel, dtypes, 2, fill=0)
    srcs, reps, wants = [], [], []
    for it in range(2):
        reps.append([workloads.gaussian_replica(680 + it, r, 0, numel, 1.0, dtype) for r in range(R)])
        srcs.append(harness.DeviceGrads(numel, dtypes, R))
        for r in range(R):
            srcs[it].upload_replica(r, reps[it][r])
        wants.append(oracle.synchronize(numel, dtypes, cap, reps[it]))
    with (flag_ordered_session(d, harness, grads, cap, STAGED) if by_flag
          else harness.Session(grads, cap, STAGED)) as s:
        d.ddp_set_option(s.ctx, d.DDP_OPT_COALESCE, 0)
        d.ddp_set_option(s.ctx, d.DDP_OPT_REDUCE_STREAMS, streams)
        d.ddp_set_option(s.ctx, d.DDP_OPT_FLAG_ORDER, -1 if by_flag else 0)
        d.ddp_set_option(s.ctx, d.DDP_OPT_TAIL_ON_BACKWARD, tail_on_backward)
        d.ddp_set_option(s.ctx, d.DDP_OPT_GATE_WAIT_US, gate_wait_us)
        assert d.ddp_get_option(s.ctx, d.DDP_OPT_FLAG_ORDER) == int(by_flag)
        order = list(range(n - 1, -1, -1))
        for it in range(2):      # two iterations enqueued without host synchronization in between
            d.ddp_synth_backward(s.ctx, order, [150_000] * n, srcs[it].ptrs(), True)
            d.ddp_finalize_backward(s.ctx)
            assert d.ddp_get_launch_log(s.ctx, 1) == wants[it][2]
            with torch.cuda.stream(s.backward_stream):
                keep.bufs[it].copy_(grads.bufs[0], non_blocking=True)
        d.ddp_synchronize(s.ctx)
        torch.cuda.synchronize()
        repaired = d.ddp_get_option(s.ctx, d.DDP_STAT_REPAIRED_LAUNCHES)
        assert repaired == 0 if gate_wait_us else repaired >= 2
        bucket_of, offset = d.ddp_get_assignment(s.ctx, n)
        flat = [[s.bucket_bytes(b, r).tobytes() for r in range(-1, R)] for b in range(s.n_buckets)]
        for p in range(n):       # the buckets hold the second iteration's gradients and average
            at = slice(int(offset[p]) * es, (int(offset[p]) + numel[p]) * es)
            assert flat[bucket_of[p]][0][at] == wants[1][0][p].tobytes(), f"averaged bucket, parameter {p}"
            for r in range(R):
                assert flat[bucket_of[p]][r + 1][at] == np.asarray(reps[1][r][p]).tobytes(), f"replica {r} parameter {p}"
    for it in range(2):
        for p in range(n):
            assert keep.download(it, p).tobytes() == wants[it][0][p].tobytes(), f"iteration {it} parameter {p}"


@pytest.mark.parametrize("pipeline", [STAGED, 1])
@pytest.mark.parametrize("n", [1, 4, 5])        # up to four buckets stay on the backward stream by default
@pytest.mark.parametrize("elems", [3000, 140000])      # ... if they move less than 4 MiB together
def test_small_models_wait_for_the_backward_stream(pipeline, n, elems):
    d, harness = lib()
    numel, R = [elems + i for i in range(n)], 2
    reps = [workloads.gaussian_replica(690, r, 0, numel, 1.0, FP32) for r in range(R)]
    want, _, wlog = oracle.synchronize(numel, [FP32] * n, 0, reps)
    grads = harness.DeviceGrads(numel, [FP32] * n, R, fill=0xFF)
    src = harness.DeviceGrads(numel, [FP32] * n, R, fill=0)
    for r in range(R):
        src.upload_replica(r, reps[r])
    with harness.Session(grads, 0, pipeline) as s:
        for it in range(2):      # NaN until the delayed backward pass has produced them (the first time)
            d.ddp_synth_backward(s.ctx, list(range(n - 1, -1, -1)), [100_000] * n, src.ptrs(), True)
            d.ddp_finalize_backward(s.ctx)
            assert d.ddp_get_launch_log(s.ctx, 1) == wlog
        d.ddp_synchronize(s.ctx)
    for i in range(n):
        assert grads.download(0, i).tobytes() == want[i].tobytes(), f"parameter {i}"


def repaired_launches(d, harness, n, R, pipeline, options=()):
    """Launches that went through a gate when `n` tensors, a bucket each, become ready one by one
    under a delayed backward pass: with a gate wait of 0 each such launch is redone by the repair
    launch, and launches on the backward stream have no gate."""
    numel = [3000 + i for i in range(n)]
    reps = [workloads.gaussian_replica(691, r, 0, numel, 1.0, FP32) for r in range(R)]
    want, _, wlog = oracle.synchronize(numel, [FP32] * n, 0, reps)
    grads = harness.DeviceGrads(numel, [FP32] * n, R, fill=0xFF)
    src = harness.DeviceGrads(numel, [FP32] * n, R, fill=0)
    for r in range(R):
        src.upload_replica(r, reps[r])
    with flag_ordered_session(d, harness, grads, 0, pipeline) as s:
        d.ddp_set_option(s.ctx, d.DDP_OPT_GATE_WAIT_US, 0)
        for option, value in options:
            d.ddp_set_option(s.ctx, option, value)
        d.ddp_synth_backward(s.ctx, list(range(n - 1, -1, -1)), [150_000] * n, src.ptrs(), True)
        d.ddp_finalize_backward(s.ctx)
        assert d.ddp_get_launch_log(s.ctx, 1) == wlog
        repaired = d.ddp_get_option(s.ctx, d.DDP_STAT_REPAIRED_LAUNCHES)
    for i in range(n):
        assert grads.download(0, i).tobytes() == want[i].tobytes(), f"parameter {i}"
    return repaired


@pytest.mark.parametrize("pipeline", [STAGED, 1])
def test_small_models_leave_the_backward_stream_when_told_to(pipeline):
    """DDP_OPT_TAIL_ON_BACKWARD 0: every bucket goes to a reduction stream, whatever the model's size."""
    d, harness = lib()
    assert repaired_launches(d, harness, 4, 2, pipeline) == 0
    assert repaired_launches(d, harness, 4, 2, pipeline, [(d.DDP_OPT_TAIL_ON_BACKWARD, 0)]) >= 3


@pytest.mark.parametrize("pipeline", [STAGED, 1])
@pytest.mark.parametrize("n,R,stays", [(4, 5, True), (3, 8, True), (4, 6, False), (3, 9, False),
                                       (2, 16, True), (2, 17, False), (1, 64, True), (5, 2, False)])
def test_small_models_with_many_replicas_use_the_reduction_streams(pipeline, n, R, stays):
    """A launch on the backward stream holds the backward pass up for its own time, which grows with
    R: beyond R * (buckets - 1) = 16 the launches overlap with the backward pass instead."""
    d, harness = lib()
    repaired = repaired_launches(d, harness, n, R, pipeline)
    assert repaired == 0 if stays else repaired >= n - 1


@pytest.mark.parametrize("pipeline", [STAGED, 1])
@pytest.mark.parametrize("marks", ["each", "closing"])
@pytest.mark.parametrize("flag_order", [-1, 0])
def test_long_launches_wait_for_the_backward_stream(pipeline, marks, flag_order):
    """Launches of more than 160 MiB: chained on two reduction streams while gradients are still being
    produced, and spread over the backward stream and its partner by a call that completes the
    iteration behind a delayed backward pass.  Gradients start as NaN; the sums run in ascending
    order, so torch gives the same bits."""
    d, harness = lib()
    import torch
    R, n = 8, 5
    elems = [(10 << 18) + 3 * i for i in range(n)]     # 10 MiB each: 170 MiB a staged launch, 90 MiB a fused one
    if pipeline != STAGED:
        elems = [2 * x for x in elems]
    grads = harness.DeviceGrads(elems, [FP32] * n, R, fill=0xFF)
    src = harness.DeviceGrads(elems, [FP32] * n, R, fill=0)
    gen = torch.Generator("cuda")
    for r in range(R):
        gen.manual_seed(700 + r)
        for i in range(n):
            src.view(r, i).view(torch.float32).normal_(generator=gen)
    torch.cuda.synchronize()
    with (flag_ordered_session(d, harness, grads, 0, pipeline) if flag_order
          else harness.Session(grads, 0, pipeline)) as s:
        d.ddp_set_option(s.ctx, d.DDP_OPT_COALESCE, 0)
        d.ddp_set_option(s.ctx, d.DDP_OPT_FLAG_ORDER, flag_order)
        order = list(range(n - 1, -1, -1))
        for _ in range(2):       # two iterations enqueued without host synchronization in between
            d.ddp_synth_backward(s.ctx, order, [100_000] * n, src.ptrs(), marks == "each")
            if marks == "closing":
                d.ddp_mark_ready_many(s.ctx, order)
            d.ddp_finalize_backward(s.ctx)
        d.ddp_synchronize(s.ctx)
        assert d.ddp_get_option(s.ctx, d.DDP_STAT_REPAIRED_LAUNCHES) == 0
    for i in range(n):
        want = src.view(0, i).view(torch.float32).clone()
        for r in range(1, R):
            want += src.view(r, i).view(torch.float32)
        want /= R
        assert torch.equal(grads.view(0, i).view(torch.float32).view(torch.int32), want.view(torch.int32)), f"parameter {i}"
