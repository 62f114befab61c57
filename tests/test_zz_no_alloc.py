"""The allocation-free entry point (ddp_sync_static) against the context path it
is a variant of -- ddp_mark_ready_many + ddp_finalize_backward on a staged
context -- and against the CPU oracle, bit for bit, on two calls in a row (the
second with a smaller input, so that what the first call left in the static
scratch array must not leak into it).  Replicas whose tensors lie apart
the call reduces in place; tensors that share memory go
through the flat buckets in the array."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

FP32, FP16, BF16 = 0, 1, 2


def lib():
    import paper_2006_15704_amd as d
    from paper_2006_15704_amd import harness
    return d, harness


def ragged_list(seed, n, max_elems):
    rng = np.random.default_rng(seed)
    numel = [int(x) for x in rng.integers(1, max_elems, size=n)]
    numel[1] = 3            # partial vectors, unaligned offsets inside the flat bucket
    numel[n // 2] = 0       # an empty gradient
    numel[-1] = 8192 * 3 + 5
    return numel


def inputs(config, numel, R, sigma, dtype):
    return [workloads.gaussian_replica(config, r, 0, numel, sigma, dtype) for r in range(R)]


def via_context(d, harness, numel, dtypes, reps, cap):
    R = len(reps)
    grads = harness.DeviceGrads(numel, dtypes, R, fill=0xFF)
    for r in range(R):
        grads.upload_replica(r, reps[r])
    with harness.Session(grads, cap, d.DDP_PIPELINE_STAGED) as s:
        s.sync()
        nb = s.n_buckets
    return nb, [[grads.download(r, i) for i in range(len(numel))] for r in range(R)]


def via_static(d, harness, torch, numel, dtypes, reps, cap, stream):
    R = len(reps)
    grads = harness.DeviceGrads(numel, dtypes, R, fill=0xFF)
    for r in range(R):
        grads.upload_replica(r, reps[r])
    torch.cuda.synchronize()
    free_before = torch.cuda.mem_get_info()[0]
    nb = d.ddp_sync_static(R, 0, stream.cuda_stream, numel, dtypes, grads.ptrs(), cap)
    stream.synchronize()
    free_after = torch.cuda.mem_get_info()[0]
    assert free_after == free_before, "the call changed the amount of free device memory"
    return nb, [[grads.download(r, i) for i in range(len(numel))] for r in range(R)]


def check_case(d, harness, torch, stream, config, numel, dtype, R, sigma, cap, what):
    dtypes = [dtype] * len(numel)
    reps = inputs(config, numel, R, sigma, dtype)
    want, asg, _ = oracle.synchronize(numel, dtypes, cap, reps)
    nb_c, out_c = via_context(d, harness, numel, dtypes, reps, cap)
    nb_s, out_s = via_static(d, harness, torch, numel, dtypes, reps, cap, stream)
    assert nb_s == nb_c == len(asg.buckets), what
    for i in range(len(numel)):
        assert out_s[0][i].tobytes() == out_c[0][i].tobytes(), f"{what}: parameter {i} differs from the context path"
        assert out_s[0][i].tobytes() == want[i].tobytes(), f"{what}: parameter {i} differs from the oracle"
        for r in range(1, R):       # the other replicas' tensors are inputs only
            assert out_s[r][i].tobytes() == reps[r][i].tobytes(), f"{what}: replica {r} parameter {i} was modified"


def used_stream(d, harness, torch):
    # The runtime loads the library's code object -- the static array is part of its image -- when
    # the process first uses it, and a stream gets its queue when it is first used; neither is an
    # allocation of the call.  Touch them once so that the free-memory comparison around the calls
    # sees the calls alone.
    stream = torch.cuda.Stream()
    warm = harness.DeviceGrads([4], [FP32], 1, fill=0)
    d.ddp_sync_static(1, 0, stream.cuda_stream, [4], [FP32], warm.ptrs(), 0)
    stream.synchronize()
    return stream


def test_static_entry_point_matches_context_path_twice_in_a_row():
    d, harness = lib()
    import torch
    stream = used_stream(d, harness, torch)
    # first call: 40 ragged fp32 tensors, R = 4, several buckets, close to 5 MiB of flat buckets
    numel_a = ragged_list(11, 40, 12000)
    check_case(d, harness, torch, stream, 21, numel_a, FP32, 4, 1e-2, 64 << 10, "first call")
    # second call, smaller and of another element type: the tiny list in fp16, R = 2
    numel_b = workloads.numel_of(workloads.tiny_shapes())
    check_case(d, harness, torch, stream, 22, numel_b, FP16, 2, 1.0, 16384, "second call")
    # third: bf16 with a replica count that is not a power of two (true division)
    check_case(d, harness, torch, stream, 23, ragged_list(12, 9, 3000), BF16, 3, 1e-3, 0, "third call")


@pytest.mark.parametrize("dtype", [FP32, FP16, BF16])
@pytest.mark.parametrize("R", [24, 25, 64])       # the last that is reduced in place, and flat buckets
def test_static_entry_point_with_many_replicas_on_shrinking_lists(dtype, R):
    """Two calls in a row, the second with fewer and shorter tensors of odd lengths in buckets of other
    sizes: padding and slots that the first one filled lie inside the second one's buckets."""
    d, harness = lib()
    import torch
    stream = used_stream(d, harness, torch)
    rng = np.random.default_rng(100 + R)
    for call, (n, most, cap) in enumerate(((14, 4000, 16 << 10), (9, 500, 1 << 10), (3, 60, 0))):
        numel = [int(x) | 1 for x in rng.integers(1, most, size=n)]
        check_case(d, harness, torch, stream, 30 + call, numel, dtype, R, 1e-2, cap, f"R {R} call {call}")


@pytest.mark.parametrize("dtype", [FP32, FP16, BF16])
def test_static_entry_point_with_shared_memory_on_shrinking_lists(dtype):
    """Likewise for few replicas where one tensor stands under two parameters."""
    d, harness = lib()
    import torch
    stream = torch.cuda.Stream()
    R = 3
    for call, (numel, cap) in enumerate((([4001, 77, 9001, 4001], 16 << 10), ([301, 5, 301], 1 << 10), ([7, 7], 0))):
        n = len(numel)
        reps = inputs(35 + call, numel, R, 1.0, dtype)
        for r in range(R):
            reps[r][n - 1] = reps[r][0].copy()
        want, _, _ = oracle.synchronize(numel, [dtype] * n, cap, reps)
        grads = harness.DeviceGrads(numel, [dtype] * n, R, fill=0xFF)
        for r in range(R):
            grads.upload_replica(r, reps[r])
        ptrs = grads.ptrs()
        for r in range(R):
            ptrs[n * r + n - 1] = ptrs[n * r]
        torch.cuda.synchronize()
        d.ddp_sync_static(R, 0, stream.cuda_stream, numel, [dtype] * n, ptrs, cap)
        stream.synchronize()
        for i in range(n - 1):
            assert grads.download(0, i).tobytes() == want[i].tobytes(), f"call {call} parameter {i}"
            for r in range(1, R):
                assert grads.download(r, i).tobytes() == reps[r][i].tobytes()


def test_static_entry_point_refuses_what_does_not_fit():
    d, harness = lib()
    import torch
    stream = torch.cuda.Stream()
    R = 8
    numel = [1 << 20]                       # 4 MiB x (R + 1) = 36 MiB > 32 MiB
    grads = harness.DeviceGrads(numel, [FP32], R, fill=0)
    before = [grads.download(r, 0).tobytes() for r in range(R)]
    with pytest.raises(d.DdpError) as e:
        d.ddp_sync_static(R, 0, stream.cuda_stream, numel, [FP32], grads.ptrs(), 25 << 20)
    assert e.value.code == d.DDP_ERR_UNSUPPORTED
    assert "static scratch buffer" in str(e.value)
    stream.synchronize()
    assert [grads.download(r, 0).tobytes() for r in range(R)] == before      # nothing was enqueued
    for bad in (lambda: d.ddp_sync_static(0, 0, 0, [4], [0], [], 0),
                lambda: d.ddp_sync_static(1, 0, 0, [4], [7], [grads.ptr(0, 0)], 0),
                lambda: d.ddp_sync_static(1, 0, 0, [4], [0], [None], 0),
                lambda: d.ddp_sync_static(1, 0, 0, [4], [0], [grads.ptr(0, 0) + 2], 0)):
        with pytest.raises(d.DdpError) as e:
            bad()
        assert e.value.code == d.DDP_ERR_ARG
    # the largest single tensor that fits with R = 1: two slabs of just under 16 MiB
    numel = [(16 << 20) // 4 - 4096]
    g1 = harness.DeviceGrads(numel, [FP32], 1, fill=0)
    x = workloads.gaussian_grad(24, 0, 0, 0, numel[0], 1.0, FP32)
    g1.upload(0, 0, x)
    assert d.ddp_sync_static(1, 0, stream.cuda_stream, numel, [FP32], g1.ptrs(), 0) == 1
    stream.synchronize()
    assert g1.download(0, 0).tobytes() == x.tobytes()      # R = 1: the average of one replica is itself


def test_static_entry_point_with_tensors_that_share_memory():
    """Where replica 0's tensors share bytes with other tensors of the list, every input is read
    before any average is written, as the flat buckets do it."""
    d, harness = lib()
    import torch
    stream = torch.cuda.Stream()
    numel, R = [5000, 5000, 77, 5000], 3
    reps = inputs(25, numel, R, 1.0, FP32)
    for r in range(R):
        reps[r][3] = reps[r][0].copy()             # one tensor under two parameters
    want, _, _ = oracle.synchronize(numel, [FP32] * 4, 16384, reps)
    grads = harness.DeviceGrads(numel, [FP32] * 4, R, fill=0xFF)
    for r in range(R):
        grads.upload_replica(r, reps[r])
    ptrs = grads.ptrs()
    for r in range(R):
        ptrs[4 * r + 3] = ptrs[4 * r]
    assert d.ddp_sync_static(R, 0, stream.cuda_stream, numel, [FP32] * 4, ptrs, 16384) >= 1
    stream.synchronize()
    for i in range(3):
        assert grads.download(0, i).tobytes() == want[i].tobytes(), f"parameter {i}"
    # replicas whose tensors lie between each other's (one region for all of them)
    both = harness.DeviceGrads([x for x in numel for _ in range(R)], [FP32] * 4 * R, 1, fill=0xFF)
    for i in range(4):
        for r in range(R):
            both.upload(0, R * i + r, reps[r][i])
    ptrs = [both.ptr(0, R * i + r) for r in range(R) for i in range(4)]
    d.ddp_sync_static(R, 0, stream.cuda_stream, numel, [FP32] * 4, ptrs, 16384)
    stream.synchronize()
    for i in range(4):
        assert both.download(0, R * i).tobytes() == want[i].tobytes(), f"parameter {i}"
        for r in range(1, R):
            assert both.download(0, R * i + r).tobytes() == reps[r][i].tobytes()


@pytest.mark.parametrize("order", ["ascending", "descending", "shuffled"])
@pytest.mark.parametrize("n", [5, 2000, 2001])       # longer unordered lists are not searched for shared memory
@pytest.mark.parametrize("shared", [False, True])
def test_static_entry_point_with_tensors_in_any_order_of_addresses(order, n, shared):
    d, harness = lib()
    import torch
    stream = torch.cuda.Stream()
    rng = np.random.default_rng(50 + n)
    R, cap = 2, 1 << 20
    at = {"ascending": list(range(n)), "descending": list(range(n - 1, -1, -1)),
          "shuffled": [int(p) for p in rng.permutation(n)]}[order]      # parameter i is the at[i]-th in memory
    stored = [int(x) for x in rng.integers(1, 20, size=n)]
    if shared:
        at[n - 1] = at[0]
    numel = [stored[k] for k in at]
    reps = inputs(51, stored, R, 1.0, FP32)
    listed = [[reps[r][k] for k in at] for r in range(R)]
    want, _, _ = oracle.synchronize(numel, [FP32] * n, cap, listed)
    grads = harness.DeviceGrads(stored, [FP32] * n, R, align=4, fill=0xFF)
    for r in range(R):
        grads.bufs[r].copy_(torch.from_numpy(np.concatenate([np.concatenate(reps[r]).view(np.uint8),
                                                             np.full(128, 0xFF, np.uint8)])))
    torch.cuda.synchronize()
    d.ddp_sync_static(R, 0, stream.cuda_stream, numel, [FP32] * n, [grads.ptr(r, k) for r in range(R) for k in at], cap)
    stream.synchronize()
    result = [grads.bufs[r].cpu().numpy() for r in range(R)]
    for i in range(n):
        o, b = grads.offsets[at[i]], grads.nbytes(at[i])
        assert result[0][o:o + b].tobytes() == want[i].tobytes(), f"parameter {i}"
        assert result[1][o:o + b].tobytes() == listed[1][i].tobytes()


# Tables that travel in the launch's arguments: n (R + 1) words, or 2 n + R where the replicas lie alike; sizes on both sides of
# the 128, 256 and 448 words that an instance of the kernel holds, of slices, and of 64 segments.
@pytest.mark.parametrize("alike,R,n", [(False, 1, 64), (False, 1, 65), (False, 3, 64), (False, 3, 65), (False, 7, 56), (False, 7, 57),
                                       (False, 64, 6), (False, 64, 7), (False, 1, 224), (True, 2, 63), (True, 2, 64), (True, 16, 120),
                                       (True, 17, 120), (True, 64, 192), (True, 64, 193), (True, 8, 220), (True, 8, 221), (True, 5, 1)])
@pytest.mark.parametrize("large", [False, True])
def test_static_entry_point_with_tables_in_every_form(alike, R, n, large):
    d, harness = lib()
    import torch
    stream = torch.cuda.Stream()
    rng = np.random.default_rng(1000 * R + n + large)
    numel = [int(x) for x in rng.integers(1, 40, size=n)]
    dtypes = [int(t) for t in np.sort(rng.integers(0, 3, size=n))]
    if n > 4:
        numel[2] = numel[n - 1] = 0               # tensors without elements, also at the end
    if large:
        numel[0], numel[n // 2] = 100003 if R < 40 else 30011, 3 * 4096
    cap = 4096
    reps = [[workloads.gaussian_grad(70, r, 0, p, numel[p], 1.0, dtypes[p]) for p in range(n)] for r in range(R)]
    want, _, _ = oracle.synchronize(numel, dtypes, cap, reps)
    gaps = rng.integers(0, 5, size=(1 if alike else R, n)) * 4
    grads = [harness.DeviceGrads(numel, dtypes, 1, align=4, skew=[int(x) for x in gaps[0 if alike else r]],
                                 replica_skew=[4 * (r % 4)], fill=0xFF) for r in range(R)]
    for r in range(R):
        raw = np.full(grads[r].bufs[0].numel(), 0xFF, dtype=np.uint8)
        for i in range(n):
            o = grads[r].offsets[i] + grads[r].replica_skew[0]
            raw[o:o + grads[r].nbytes(i)] = reps[r][i].view(np.uint8)
        grads[r].bufs[0].copy_(torch.from_numpy(raw))
    ptrs = [grads[r].ptr(0, i) if numel[i] else None for r in range(R) for i in range(n)]
    torch.cuda.synchronize()
    for _ in range(1 if R > 1 else 2):                    # (R = 1: the average is the tensor itself)
        d.ddp_sync_static(R, 0, stream.cuda_stream, numel, dtypes, ptrs, cap)
    stream.synchronize()
    for r in range(R):
        raw = grads[r].bufs[0].cpu().numpy()
        for i in range(n):
            o = grads[r].offsets[i] + grads[r].replica_skew[0]
            x = want[i] if r == 0 else reps[r][i]
            assert raw[o:o + grads[r].nbytes(i)].tobytes() == x.tobytes(), f"replica {r} parameter {i}"
