"""Snapshots on a stream that is being captured are refused, with a host image (whose
drain is sized by a wait) and without (where the call would not wait): no call is
left in the graph, and the context's next calls give the oracle's image."""
import ctypes

import numpy as np
import pytest

import oracle
from tests.gpu_util import image_capacity, log, upload
from tests.test_gpu_small_calls import table

pytestmark = pytest.mark.gpu

P = 4096


@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("n_regions", [2, 20])
@pytest.mark.parametrize("host", [False, True])
@pytest.mark.parametrize("used", [False, True])
@pytest.mark.parametrize("entry", ["crum_snapshot", "crum_snapshot_noalloc"])
def test_a_call_under_capture_is_refused(entry, used, host, n_regions, mode):
    import torch
    import paper_1808_00117_amd as crum
    from paper_1808_00117_amd import hip as H
    from paper_1808_00117_amd.api import regions_of
    log(f"[capture] {entry} used={used} host={host} {n_regions} regions mode {mode}")
    regs = table(n_regions, 300, P, n_regions)
    _, img, _ = oracle.snapshot(regs, P, seq=3)
    dev = upload(regs)
    cap = image_capacity(dev, P)
    staging = torch.zeros(cap, dtype=torch.uint8, device="cuda")
    image = torch.zeros(cap, dtype=torch.uint8, pin_memory=True)
    status = torch.zeros(64, dtype=torch.uint8, pin_memory=True)
    hip = H.hip()
    stream, graph = ctypes.c_void_p(), ctypes.c_void_p()
    assert hip.hipStreamCreateWithFlags(ctypes.byref(stream), 1) == 0
    ctx = crum.crum_ctx_create(0)
    try:
        def call(h):
            return getattr(crum, entry)(ctx, regions_of(dev), P, 0, 3, staging.data_ptr(), cap,
                                        image.data_ptr() if h else 0, cap if h else 0,
                                        stream.value, status.data_ptr())
        torch.cuda.synchronize()
        if used:
            assert call(True) == crum.CRUM_OK
            assert hip.hipStreamSynchronize(stream) == 0
        assert hip.hipStreamBeginCapture(stream, mode) == 0
        rc = call(host)
        assert hip.hipStreamEndCapture(stream, ctypes.byref(graph)) == 0  # still whole
        hip.hipGraphDestroy(graph)
        assert rc == crum.CRUM_EHIP
        for h in (True, False):
            staging.zero_(), image.zero_()
            torch.cuda.synchronize()
            assert call(h) == crum.CRUM_OK and hip.hipStreamSynchronize(stream) == 0
            got = image.numpy() if h else staging.cpu().numpy()
            assert np.array_equal(got[:img.size], img)
    finally:
        crum.crum_ctx_destroy(ctx)
        hip.hipStreamDestroy(stream)
