"""Calls prepared while an earlier call of the same context is still queued: a
snapshot without a host image returns before the device has run, and the next
call writes the same pinned buffers.  Behind other work on the stream, a device
image (with room for it and without) and then, with no wait between, a call whose
tables are kernel arguments (16 regions and fewer) or uploaded; every image is
the oracle's."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import image_capacity, log, upload
from tests.test_gpu_small_calls import table

pytestmark = pytest.mark.gpu

KiB = 1 << 10
P = 4 * KiB


class Call:
    """A table of n regions, its oracle image and the buffers of one call."""

    def __init__(self, n_regions, n_pages, seed, seq, host, room=True):
        import torch
        from paper_1808_00117_amd.api import regions_of
        regs = table(n_regions, n_pages, P, seed)
        st, self.image, _ = oracle.snapshot(regs, P, seq=seq)
        self.n_dirty, self.seq, self.room = st.n_dirty, seq, room
        self.dev = upload(regs)
        self.regions = regions_of(self.dev)
        # room for every page, or one byte short of the image
        self.size = image_capacity(self.dev, P) if room else self.image.size - 1
        self.staging = torch.zeros(self.size, dtype=torch.uint8, device="cuda")
        self.h = torch.full((self.size,), 0xAB, dtype=torch.uint8,
                            pin_memory=True) if host else None
        self.status = torch.zeros(64, dtype=torch.uint8, pin_memory=True)

    def enqueue(self, entry, ctx):
        import torch
        h = self.h.data_ptr() if self.h is not None else 0
        assert entry(ctx, self.regions, P, 0, self.seq, self.staging.data_ptr(), self.size, h,
                     self.size, torch.cuda.current_stream().cuda_stream,
                     self.status.data_ptr()) == 0

    def check(self):
        import paper_1808_00117_amd as crum
        st = crum.read_status(self.status.data_ptr())
        assert st.code == (0 if self.room else crum.CRUM_ENOSPC)
        assert st.n_dirty == self.n_dirty and st.image_bytes == self.image.size
        n = self.image.size
        if self.room:
            assert np.array_equal(self.staging[:n].cpu().numpy(), self.image)
        if self.h is not None:
            h = self.h.numpy()
            assert np.array_equal(h[:n], self.image) and (h[n:] == 0xAB).all()


@pytest.mark.parametrize("entry", ["crum_snapshot_noalloc", "crum_snapshot"])
@pytest.mark.parametrize("first_regions,room", [(5, True), (5, False), (16, True), (20, True)])
@pytest.mark.parametrize("n_regions", [3, 16, 17, 18, 40])
def test_pending_device_image_then_host_image(entry, first_regions, room, n_regions):
    import torch
    import paper_1808_00117_amd as crum
    log(f"[pending] {entry} {first_regions} regions room={room}, then {n_regions}")
    call = getattr(crum, entry)
    ctx = crum.crum_ctx_create(0)
    try:
        first = Call(first_regions, 1500, 3 * first_regions, 1, host=False, room=room)
        calls = [first, Call(n_regions, 700, n_regions, 2, host=True),
                 Call(n_regions + 1, 300, 50 + n_regions, 3, host=False),
                 Call(n_regions, 400, 100 + n_regions, 4, host=True)]
        assert len({c.n_dirty for c in calls}) == len(calls)
        warm = Call(n_regions, 1600, 7, 5, host=True)  # scratch and buffers at their size
        warm.enqueue(call, ctx)
        torch.cuda.synchronize()
        warm.check()
        busy = torch.empty(1 << 30, dtype=torch.uint8, device="cuda")
        for _ in range(16):  # a few milliseconds
            busy.fill_(1)
        for c in calls:
            c.enqueue(call, ctx)
        torch.cuda.synchronize()
        for c in calls:
            c.check()
    finally:
        crum.crum_ctx_destroy(ctx)
