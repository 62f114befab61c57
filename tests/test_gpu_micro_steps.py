"""Micro-steps in a row: the pointer tables travel through a few pinned buffers that are used in turn, also while
the GPU is behind.  Every step takes other tensors, some of them absent, so that a table that was overwritten
before it was read would show."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R,n", [(1, 1), (3, 5), (64, 33), (64, 140)])      # (the last: two tables instead of four)
@pytest.mark.parametrize("delay_us", [0, 300])
def test_tables_of_many_micro_steps(R, n, delay_us):
    import torch
    import paper_2006_15704_amd as d
    from paper_2006_15704_amd import harness
    steps = 11
    numel = [1 + 37 * i for i in range(n)]
    rng = np.random.default_rng(800 + R)
    grads = harness.DeviceGrads(numel, [0] * n, R, fill=0)
    micro = [harness.DeviceGrads(numel, [0] * n, R) for _ in range(steps)]
    want = np.zeros((R, n), dtype=np.float32)
    tables = []
    for k, m in enumerate(micro):
        present = rng.random((R, n)) < 0.8
        for r in range(R):
            m.bufs[r][:m.slab_bytes // 4 * 4].view(torch.float32).fill_(float(1 << k))      # every subset of steps has a sum of its own
        want += present * np.float32(1 << k)
        tables.append([m.ptr(r, i) if present[r, i] else None for r in range(R) for i in range(n)])
    torch.cuda.synchronize()
    with harness.Session(grads, 1 << 20, 1) as s:
        for ptrs in tables:
            if delay_us:
                d.ddp_synth_backward(s.ctx, [0], [delay_us * 1000], mark=False)
            d.ddp_no_sync_accumulate(s.ctx, ptrs)
        d.ddp_synchronize(s.ctx)
    for r in range(R):
        for i in range(n):
            assert (grads.download(r, i) == want[r, i]).all(), f"replica {r} parameter {i}"


# Lists that travel in the launch's arguments as they are (R n pointers), as R bases and n distances where the replicas
# lie alike, and as a table: sizes on both sides of the 64, 192 and 448 words that an instance of the kernel holds.
@pytest.mark.parametrize("R,n", [(1, 1), (2, 32), (2, 33), (3, 64), (2, 224), (2, 225), (8, 56), (8, 57), (4, 188), (4, 189),
                                 (8, 440), (8, 441), (1, 447), (1, 448), (64, 7), (64, 8), (64, 384)])
@pytest.mark.parametrize("layout", ["alike", "one tensor apart", "replicas absent", "parameters absent", "first absent"])
def test_every_form_of_a_list_of_pointers(R, n, layout):
    import torch
    import paper_2006_15704_amd as d
    from paper_2006_15704_amd import harness
    numel = [1 + (13 * i) % 29 for i in range(n)]
    dtypes = [i % 3 for i in range(n)]
    rng = np.random.default_rng(900 + R * n)
    present = np.ones((R, n), dtype=bool)
    if layout == "replicas absent":
        present = rng.random((R, n)) < 0.7
    elif layout == "parameters absent":
        present[:, rng.random(n) < 0.3] = False
    elif layout == "first absent":
        present[:, 0] = False
    grads = harness.DeviceGrads(numel, dtypes, R, fill=0)
    micro = harness.DeviceGrads(numel, dtypes, R, align=4, replica_skew=[64 * (r % 2) for r in range(R)], fill=0)
    value = (np.arange(R)[:, None] * 7 + np.arange(n)[None, :] * 3) % 50 + 1      # whole numbers, exact in every type
    ptrs = [micro.ptr(r, i) if present[r, i] else None for r in range(R) for i in range(n)]
    torch_type = (torch.float32, torch.float16, torch.bfloat16)
    host = [np.zeros(micro.slab_bytes + 64, dtype=np.uint8) for _ in range(R)]
    for r in range(R):
        for i in range(n):
            x = torch.full((numel[i],), float(value[r, i]), dtype=torch_type[dtypes[i]]).view(torch.uint8).numpy()
            o = micro.offsets[i] + micro.replica_skew[r]
            host[r][o:o + x.size] = x
        micro.bufs[r].copy_(torch.from_numpy(host[r]))
    if layout == "one tensor apart":
        o = micro.offsets[n - 1] + micro.replica_skew[R - 1]
        size = micro.nbytes(n - 1)
        apart = torch.zeros(size + 64, dtype=torch.uint8, device="cuda")
        apart[:size].copy_(micro.bufs[R - 1][o:o + size])
        ptrs[-1] = apart.data_ptr()
    torch.cuda.synchronize()
    with harness.Session(grads, 1 << 20, 1) as s:
        for _ in range(2):
            d.ddp_no_sync_accumulate(s.ctx, ptrs)
        d.ddp_synchronize(s.ctx)
        used = d.ddp_get_used_map(s.ctx, n, 0)
    for r in range(R):
        raw = grads.bufs[r].cpu().numpy()
        for i in range(n):
            o = grads.offsets[i]
            got = torch.from_numpy(raw[o:o + grads.nbytes(i)].copy()).view(torch_type[dtypes[i]]).float().numpy()
            assert (got == (2 * value[r, i] if present[r, i] else 0)).all(), f"replica {r} parameter {i}"
    assert [bool(u) for u in used] == [bool(x) for x in present.any(axis=0)]
