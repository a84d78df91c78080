"""The diff time that a timed plan reports, from the clocks its workgroups leave,
against events around the same diff in a snapshot: nothing new, and new pages
behind the known ones (whose workgroups end at once, last).  The launches are 160 us
and longer; events read a few microseconds more than the kernel's own time, and the
clocks cost it up to 6 %, so the shortest of eight of each agree within 15 %."""
import pytest

from tests.gpu_util import log

pytestmark = pytest.mark.gpu

MiB = 1 << 20


@pytest.mark.parametrize("P", [4096, 65536])
@pytest.mark.parametrize("known,new", [(512, 0), (1024, 0), (1024, 512)])
def test_clocks_and_events_agree(P, known, new):
    import torch
    import paper_1808_00117_amd as crum
    log(f"[clock] P={P} {known}+{new} MiB")
    cur = torch.empty(known * MiB // 8, dtype=torch.int64, device="cuda").random_()
    shadow = cur.clone()
    extra = torch.empty(max(new, 1) * MiB, dtype=torch.uint8, device="cuda")
    table = [(cur.data_ptr(), shadow.data_ptr(), known * MiB, 1)]
    if new:
        table.append((extra.data_ptr(), 0, new * MiB, 2))
    room = crum.crum_image_prefix_bytes(len(table), (known + new) * MiB // P) + 4096
    staging = torch.empty(room, dtype=torch.uint8, device="cuda")
    status = torch.zeros(64, dtype=torch.uint8, pin_memory=True)
    stream = torch.cuda.current_stream().cuda_stream
    ctx = crum.crum_ctx_create(0)
    plan = None
    try:
        crum.crum_ctx_set_timing(ctx, crum.TIMING_DIFF)
        crum.crum_ctx_set_param(ctx, crum.CRUM_PARAM_CHUNK_BYTES, 1 << 40)
        crum.crum_ctx_set_param(ctx, crum.CRUM_PARAM_EAGER, 0)
        plan = crum.Plan(ctx, [(table, P, 0, 1)], staging.data_ptr(), room, 0, 0)

        def snapshot():
            return crum.crum_snapshot(ctx, table, P, 0, 1, staging.data_ptr(), room, 0, 0, stream,
                                      status.data_ptr())

        def best(call):
            times = []
            for _ in range(10):
                torch.cuda.synchronize()
                crum.crum_ctx_timing_reset(ctx)
                assert call() == crum.CRUM_OK
                torch.cuda.synchronize()
                count, ms = crum.crum_ctx_timing(ctx, 0)
                assert count == 1
                times.append(ms)
            return min(times[2:])
        events, clocks = best(snapshot), best(lambda: plan.launch(stream, status.data_ptr()))
        assert 0.85 * events <= clocks <= 1.15 * events, (clocks, events)
    finally:
        if plan is not None:
            plan.destroy()
        crum.crum_ctx_destroy(ctx)
