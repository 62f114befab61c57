"""GPU parity of short launches (a thread block per 1 KiB slice of a tile) and of the ends of segments in
launches of whole tiles.  DDP_OPT_NONTEMPORAL 0 keeps every launch on tiles, so both kernels are run on the
same lists: segments of one element more or less than slices and tiles, replica counts around the four waves
and sixteen rows a block works with.  All sums run in the oracle's order: bit for bit."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

FP32, FP16, BF16 = 0, 1, 2
ES = {FP32: 4, FP16: 2, BF16: 2}
STAGED, FUSED = 0, 1
SLICE, TILE = 1024, 8192


def lib():
    import paper_2006_15704_amd as d
    from paper_2006_15704_amd import harness
    return d, harness


def edge_sizes(es):
    k, v = SLICE // es, 16 // es
    return [k - 1, k, k + 1, 8 * k - 1, 8 * k, 8 * k + 1, 1, v - 1, v, v + 1, 2 * v - 1, 10 * k + 3, 0, k + v]


def outside_is_untouched(grads, r, byte):
    raw = grads.bufs[r].cpu().numpy()
    inside = np.zeros(raw.size, dtype=bool)
    for i in range(grads.n):
        o = grads.offsets[i] + grads.replica_skew[r]
        inside[o:o + grads.nbytes(i)] = True
    return (raw[~inside] == byte).all()


@pytest.mark.parametrize("nontemporal", [1, 0])
@pytest.mark.parametrize("dtype", [FP32, FP16, BF16])
@pytest.mark.parametrize("R", [1, 2, 5, 15, 16, 17, 33, 64])
def test_slices_and_tiles(dtype, R, nontemporal):
    d, harness = lib()
    es = ES[dtype]
    numel = edge_sizes(es)
    n, cap = len(numel), 3 * TILE
    rng = np.random.default_rng(900 + R)
    reps = [workloads.gaussian_replica(900 + R, r, 0, numel, 1e-2, dtype) for r in range(R)]
    for r in range(R):           # zeros of both signs, and bits that arithmetic would not preserve
        for x in reps[r]:
            x.view(np.uint32 if dtype == FP32 else np.uint16)[::7] = (r % 2) << (8 * es - 1)
        reps[r][0].view(np.uint32 if dtype == FP32 else np.uint16)[-1:] = 0x7F800001 if dtype == FP32 else 0x7F81
    everyone = [(p, [1] * R) for p in range(n - 1, -1, -1)]
    some = (rng.random((n, R)) < 0.6).astype(np.uint8)
    some[3] = 0
    some[11, 1:] = 0
    for pipeline in (FUSED, STAGED):
        for marks, write_all, keep in ((everyone, False, False), (everyone, True, False),
                                       ([(p, some[p].tolist()) for p, _ in everyone], True, True)):
            with np.errstate(invalid="ignore"):
                want, _, wlog, _ = oracle.synchronize_local(numel, [dtype] * n, cap, reps, marks, find_unused=keep)
            grads = harness.DeviceGrads(numel, [dtype] * n, R, skew=[es * (3 * i % 8) for i in range(n)],
                                        replica_skew=[es * (5 * r % (16 // es)) for r in range(R)], fill=0xFF)
            for r in range(R):
                grads.upload_replica(r, reps[r])
            with harness.Session(grads, cap, pipeline, write_all) as s:
                d.ddp_set_option(s.ctx, d.DDP_OPT_NONTEMPORAL, nontemporal)
                d.ddp_set_option(s.ctx, d.DDP_OPT_FIND_UNUSED, int(keep))
                for p, used in marks:
                    if all(used):
                        d.ddp_mark_ready(s.ctx, p)
                    else:
                        d.ddp_mark_ready_local(s.ctx, p, used)
                d.ddp_finalize_backward(s.ctx)
                d.ddp_synchronize(s.ctx)
                assert d.ddp_get_launch_log(s.ctx, 1) == wlog
                if pipeline == STAGED:
                    bucket_of, offset = d.ddp_get_assignment(s.ctx, n)
                    flat = {b: [s.bucket_bytes(b, r).tobytes() for r in range(R)] for b in range(s.n_buckets)}
                    used_of = dict(marks)
                    for p in range(n):
                        for r in range(R):
                            got = flat[bucket_of[p]][r][offset[p] * es:(offset[p] + numel[p]) * es]
                            expect = reps[r][p].tobytes() if used_of[p][r] else bytes(numel[p] * es)
                            assert got == expect, f"flat bucket, replica {r} parameter {p}"
            for r in range(R):
                for p in range(n):
                    expect = want[r][p] if r == 0 or write_all else reps[r][p]
                    got = grads.download(r, p)
                    nan = np.isnan(oracle.to_f32(expect, dtype))
                    assert (np.isnan(oracle.to_f32(got, dtype)) == nan).all()
                    assert got[~nan].tobytes() == np.asarray(expect)[~nan].tobytes(), f"pipeline {pipeline} replica {r} parameter {p}"
                assert outside_is_untouched(grads, r, 0xFF), f"replica {r}: bytes between the tensors were written"


@pytest.mark.parametrize("nontemporal", [1, 0])
@pytest.mark.parametrize("transport", [FP16, BF16])
@pytest.mark.parametrize("R,out_skew", [(3, 0), (16, 4), (64, 12)])
def test_binary32_outputs(transport, R, out_skew, nontemporal):
    d, harness = lib()
    numel = edge_sizes(2)
    n, cap = len(numel), 3 * TILE
    sent = [workloads.gaussian_replica(920, r, 0, numel, 1e-2, transport) for r in range(R)]
    want, _, _ = oracle.synchronize_transport(numel, [transport] * n, cap, sent)
    grads = harness.DeviceGrads(numel, [transport] * n, R, replica_skew=[2 * (3 * r % 8) for r in range(R)], fill=0xFF)
    for r in range(R):
        grads.upload_replica(r, sent[r])
    outs = harness.DeviceGrads(numel, [FP32] * n, 1, skew=[out_skew] * n, fill=0x55)
    with harness.Session(grads, cap, FUSED, outputs=outs) as s:
        d.ddp_set_option(s.ctx, d.DDP_OPT_NONTEMPORAL, nontemporal)
        s.sync()
    for i in range(n):
        assert outs.download(0, i).tobytes() == want[i].tobytes(), f"parameter {i}"
    assert outside_is_untouched(outs, 0, 0x55)
    for r in range(R):
        for i in range(n):
            assert grads.download(r, i).tobytes() == sent[r][i].tobytes(), "the transport copies are inputs only"


@pytest.mark.parametrize("pipeline,dtype,R,tiles", [(FUSED, FP32, 4, 128), (FUSED, FP32, 16, 128), (FUSED, BF16, 9, 192),
                                                    (FUSED, FP16, 64, 128), (STAGED, BF16, 3, 128), (STAGED, FP32, 8, 256),
                                                    (STAGED, FP16, 17, 256), (STAGED, FP32, 64, 128)])
def test_launches_on_both_sides_of_the_limit(pipeline, dtype, R, tiles):
    """The longest launch that takes slices, and one tile more.  The sum runs in ascending order and
    is rounded once, so torch gives the same bits."""
    d, harness = lib()
    import torch
    es, t = ES[dtype], {FP32: torch.float32, FP16: torch.float16, BF16: torch.bfloat16}[dtype]
    for extra in (0, 1):
        k = TILE // es
        numel = [(tiles + extra - 2) * k - 7, k + 2]          # the second one reaches two elements into its second tile
        grads = harness.DeviceGrads(numel, [dtype] * 2, R, skew=[0, 3 * es], fill=0xFF)
        gen = torch.Generator("cuda")
        each = []
        for r in range(R):
            gen.manual_seed(940 + r)
            for i in range(2):
                grads.view(r, i).copy_(torch.randn(numel[i], generator=gen, device="cuda").to(t).view(torch.uint8))
            # (copies: a view at an odd offset cannot be seen as its type)
            each.append([grads.view(r, i).clone().view(t).float() for i in range(2)])
        torch.cuda.synchronize()
        with harness.Session(grads, 1 << 40, pipeline) as s:
            s.sync()
        for i in range(2):
            total = each[0][i].clone()
            for r in range(1, R):
                total = total + each[r][i]
            # (divided on the CPU: by a number, torch multiplies with the reciprocal on the GPU)
            want = (total.cpu() / torch.full((1,), float(R))).to(t)
            assert grads.download(0, i).tobytes() == want.view(torch.uint8).numpy().tobytes(), f"{tiles + extra} tiles, parameter {i}"


@pytest.mark.parametrize("long_launch", [0, 1])
@pytest.mark.parametrize("dtype", [FP32, FP16, BF16])
@pytest.mark.parametrize("R", [1, 2, 3, 5, 6, 10, 11, 15, 16, 17, 24, 64])
def test_whole_tiles_with_tables_in_every_form(dtype, R, long_launch):
    """Launches above the limit for slices, whole tiles and ends: how the tables of a long one (600 MiB) are read depends on the number
    of replicas, on the output's type and on how many replicas are written.  The reference sums and divides in binary32 in the same order."""
    import torch
    d, harness = lib()
    es = ES[dtype]
    ttype = {FP32: torch.float32, FP16: torch.float16, BF16: torch.bfloat16}[dtype]
    t = TILE // es
    numel = [(77000 // (R + 1) if long_launch else 130) * t + 5, 1, 70 * t - 3, t, 90 * t + 1, 33]
    n = len(numel)
    grads = harness.DeviceGrads(numel, [dtype] * n, R, skew=[es * (3 * i % 8) for i in range(n)],
                                replica_skew=[es * (5 * r % (16 // es)) for r in range(R)], fill=0)
    gen = torch.Generator("cuda")
    gen.manual_seed(R)
    inputs = [[torch.randn(k, generator=gen, device="cuda").to(ttype) for k in numel] for _ in range(R)]
    want = []
    for i in range(n):
        s = inputs[0][i].float()
        for r in range(1, R):
            s = s + inputs[r][i].float()
        want.append(s / torch.full_like(s, float(R)))
    for write_all, binary32 in ((False, False), (True, False), (False, True)):
        if binary32 and dtype == FP32:
            continue
        for r in range(R):
            for i in range(n):
                grads.view(r, i).copy_(inputs[r][i].view(torch.uint8))
        outputs = harness.DeviceGrads(numel, [FP32] * n, 1, fill=0xFF) if binary32 else None
        with harness.Session(grads, 1 << 40, FUSED, write_all, outputs=outputs) as s:
            s.sync()
        for r in range(R if write_all else 1):
            for i in range(n):
                expect = want[i] if binary32 else want[i].to(ttype)
                got = (outputs if binary32 else grads).view(r, i)
                assert torch.equal(got, expect.view(torch.uint8)), f"replica {r} parameter {i} write_all {write_all}"


def slice_line(R, es, staged):
    """Tiles up to which every launch takes slices; eight slices a tile are what a list of slices may hold."""
    return 128 if R <= 4 or R > 32 else 256 if staged else 192 if es == 2 else 128


@pytest.mark.parametrize("dtype", [FP32, BF16])
@pytest.mark.parametrize("R,pipeline", [(5, STAGED), (16, FUSED), (16, STAGED), (24, FUSED), (25, STAGED)])
@pytest.mark.parametrize("slices", ["of one tile more than the line", "as many as may be listed", "one more"])
def test_lists_of_tensors_much_smaller_than_a_tile(dtype, R, pipeline, slices):
    """A tile for each tensor, most of it empty: up to so many slices that hold something, and one more, which takes tiles."""
    d, harness = lib()
    line = slice_line(R, ES[dtype], pipeline == STAGED)
    n = line + 1 if slices == "of one tile more than the line" else 8 * line - 2 + (slices == "one more")
    numel = [1 + (7 * i) % 23 for i in range(n)]             # a slice each, but for one that holds three
    numel[n // 3] = 2 * SLICE // ES[dtype] + 3
    reps = [workloads.gaussian_replica(960, r, 0, numel, 1e-2, dtype) for r in range(R)]
    want, _, _ = oracle.synchronize(numel, [dtype] * n, 1 << 30, reps)
    grads = harness.DeviceGrads(numel, [dtype] * n, R, align=ES[dtype], replica_skew=[ES[dtype] * (r % 3) for r in range(R)], fill=0x5A)
    upload_packed(grads, reps)
    with harness.Session(grads, 1 << 30, pipeline) as s:
        s.sync()
    check_packed(grads, want, reps)


def torch_from(raw):
    import torch
    return torch.from_numpy(raw)


@pytest.mark.parametrize("dtype,R,tiles", [(FP32, 8, 128), (FP32, 8, 129), (FP32, 9, 192), (FP32, 9, 193), (FP32, 24, 192), (FP32, 24, 193), (FP32, 25, 129),
                                           (BF16, 9, 240), (BF16, 9, 241), (BF16, 16, 240), (BF16, 16, 241), (BF16, 17, 192), (BF16, 17, 193)])
def test_context_free_lists_of_small_tensors(dtype, R, tiles):
    """Slices without a list of them: on both sides of the numbers of tiles up to which they are taken, with tables in arguments
    and in memory."""
    d, harness = lib()
    import torch
    numel = [1 + (7 * i) % 23 for i in range(tiles)]
    numel[tiles // 3] = 2 * SLICE // ES[dtype] + 3
    reps = [workloads.gaussian_replica(980, r, 0, numel, 1e-2, dtype) for r in range(R)]
    want, _, _ = oracle.synchronize(numel, [dtype] * tiles, 1 << 30, reps)
    grads = harness.DeviceGrads(numel, [dtype] * tiles, R, align=ES[dtype], replica_skew=[ES[dtype] * (r % 3) for r in range(R)], fill=0x5A)
    upload_packed(grads, reps)
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    assert d.ddp_sync_static(R, 0, stream.cuda_stream, numel, [dtype] * tiles, grads.ptrs(), 1 << 30) == 1
    stream.synchronize()
    check_packed(grads, want, reps)


@pytest.mark.parametrize("dtype,R,tiles", [(FP32, 8, 384), (FP32, 8, 385), (BF16, 5, 340), (BF16, 5, 341), (BF16, 24, 340), (BF16, 24, 341)])
def test_small_tensors_of_a_model_without_a_list_of_slices(dtype, R, tiles):
    """More than 16 MiB a replica: the bucket of small tensors takes slices of its tiles, staged, up to so many of those."""
    d, harness = lib()
    numel = [(17 << 20) // ES[dtype]] + [1 + (7 * i) % 23 for i in range(tiles)]
    n = tiles + 1
    reps = [[np.full(numel[0], 0, dtype=harness.NP_STORAGE[dtype])] + workloads.gaussian_replica(990, r, 0, numel[1:], 1e-2, dtype) for r in range(R)]
    cap = sum(numel[1:]) * ES[dtype]
    want, _, _ = oracle.synchronize(numel, [dtype] * n, cap, reps)
    grads = harness.DeviceGrads(numel, [dtype] * n, R, align=ES[dtype], replica_skew=[ES[dtype] * (r % 3) for r in range(R)], fill=0x5A)
    upload_packed(grads, reps)
    with harness.Session(grads, cap, STAGED) as s:
        assert s.n_buckets == 2
        d.ddp_set_option(s.ctx, d.DDP_OPT_COALESCE, 0)
        s.sync()
    check_packed(grads, want, reps)


def upload_packed(grads, reps):
    for r in range(grads.R):
        raw = np.full(grads.bufs[r].numel(), 0x5A, dtype=np.uint8)
        o = grads.offsets[0] + grads.replica_skew[r]
        data = np.concatenate([x.view(np.uint8) for x in reps[r]])
        raw[o:o + data.size] = data
        grads.bufs[r].copy_(torch_from(raw))


def check_packed(grads, want, reps):
    for r in range(grads.R):
        raw = grads.bufs[r].cpu().numpy()
        o = grads.offsets[0] + grads.replica_skew[r]
        data = np.concatenate([x.view(np.uint8) for x in (want if r == 0 else reps[r])])
        assert raw[o:o + data.size].tobytes() == data.tobytes(), f"replica {r}"
        assert outside_is_untouched(grads, r, 0x5A)
