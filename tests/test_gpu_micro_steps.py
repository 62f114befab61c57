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
