"""The clock stamps of a timed plan's diff where only its last 4096 workgroups
write the end: below, at and above that many workgroups (64 KiB each in 16 KiB
pages), the stamped time lies between what the caches' peak rate allows (20 TB/s
over both copies) and the events around the launch."""
import pytest

from tests.gpu_util import log

pytestmark = pytest.mark.gpu

KiB, MiB = 1 << 10, 1 << 20


@pytest.mark.parametrize("mib", [1, 256, 257, 768])
def test_stamped_time_is_that_of_the_launch(mib):
    import torch
    import paper_1808_00117_amd as crum
    from paper_1808_00117_amd.api import Snapshotter

    P, n = 16 * KiB, mib * MiB
    log(f"[stamps] {mib} MiB")
    s = Snapshotter(0)
    try:
        cur = torch.empty(n // 8, dtype=torch.int64, device="cuda").random_()
        shadow = cur.clone()
        room = crum.crum_image_bytes(1, n // P, 1, P)
        staging = torch.empty(room, dtype=torch.uint8, device="cuda")
        status = torch.zeros(64, dtype=torch.uint8, pin_memory=True)
        crum.crum_ctx_set_timing(s.ctx, crum.TIMING_DIFF)
        plan = crum.Plan(s.ctx, [([(cur.data_ptr(), shadow.data_ptr(), n, 1)], P, 0, 1)],
                         staging.data_ptr(), room, 0, 0)
        try:
            stream = torch.cuda.current_stream().cuda_stream
            for _ in range(3):
                torch.cuda.synchronize()
                crum.crum_ctx_timing_reset(s.ctx)
                a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
                a.record()
                assert plan.launch(stream, status.data_ptr()) == crum.CRUM_OK
                b.record()
                b.synchronize()
                count, ms = crum.crum_ctx_timing(s.ctx, 0)
                assert count == 1
                assert 2 * n / 20e12 * 1e3 <= ms <= a.elapsed_time(b), (ms, a.elapsed_time(b))
        finally:
            plan.destroy()
    finally:
        s.close()
