"""Small calls at the edges of their dispatch, against the oracle: region tables
that are kernel arguments or uploaded (16 and 17 regions), bitmaps formed in the
scan or before it (128 and 129 words, 64 and 65 regions), every order of
crum_snapshot and the allocation-free entry point, in status memory that the
device maps and images with and without room."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import log, upload
from tests.test_gpu_parity import check_parity, snap, snap_direct, snap_small_chunks  # noqa: F401

pytestmark = pytest.mark.gpu

KiB = 1 << 10


def table(n_regions, n_pages, P, seed):
    rng = np.random.default_rng(seed)
    cuts = np.sort(rng.choice(np.arange(1, n_pages), n_regions - 1, replace=False)) \
        if n_regions > 1 else np.zeros(0, np.int64)
    counts = np.diff(np.concatenate([[0], cuts, [n_pages]])).astype(int)
    out = []
    for i, n in enumerate(counts):
        cur = rng.integers(0, 256, n * P, dtype=np.uint8)
        sh = cur.copy()
        hit = np.flatnonzero(rng.random(n) < 0.2)
        sh[hit * P + rng.integers(0, P, hit.size)] ^= 0x21
        # the last page always, and now and then no shadow
        sh[n * P - 1] ^= 1
        out.append((cur, None if n < 40 and i % 5 == 4 else sh, 60 + i))
    return out


@pytest.mark.parametrize("n_pages", [65, 64 * 127 + 1, 64 * 128, 64 * 128 + 1])
@pytest.mark.parametrize("n_regions", [1, 16, 17, 64, 65])
def test_edges(snap, snap_small_chunks, snap_direct, n_regions, n_pages):  # noqa: F811
    import torch
    import paper_1808_00117_amd as crum

    P = 4 * KiB
    log(f"[small] {n_regions} regions, {n_pages} pages")
    regs = table(n_regions, n_pages, P, n_regions * 7919 + n_pages)
    dev, img = check_parity(snap, regs, P, others=(snap_small_chunks, snap_direct))
    # the allocation-free entry point: with room, and one byte short of it
    from paper_1808_00117_amd.api import regions_of
    for room in (img.size, img.size - 1):
        staging = torch.zeros(img.size, dtype=torch.uint8, device="cuda")
        h = torch.zeros(img.size, dtype=torch.uint8, pin_memory=True)
        st = torch.zeros(64, dtype=torch.uint8, pin_memory=True)
        rc = crum.crum_snapshot_noalloc(snap.ctx, regions_of(dev), P, 0, 3, staging.data_ptr(),
                                        room, h.data_ptr(), room,
                                        torch.cuda.current_stream().cuda_stream, st.data_ptr())
        torch.cuda.synchronize()
        got = crum.read_status(st.data_ptr())
        assert rc == 0 and got.image_bytes == img.size
        if room == img.size:
            assert got.code == 0 and np.array_equal(h.numpy(), img)
        else:
            assert got.code == crum.CRUM_ENOSPC and not h.any()
            at = 64 + 32 * n_regions
            words = 8 * ((n_pages + 63) // 64)
            assert np.array_equal(staging[at:at + words].cpu().numpy(), img[at:at + words])


def test_only_regions_without_shadow(snap):  # noqa: F811
    """No diff at all; on the device only, and with an update that has no shadow to write."""
    log("[small] no shadow")
    regs = [(c, None, r) for c, _, r in table(3, 300, 16 * KiB, 9)]
    check_parity(snap, regs, 16 * KiB, flags=1)
    st_o, img_o, _ = oracle.snapshot(regs, 16 * KiB, seq=4)
    dev = upload(regs)
    from tests.gpu_util import gpu_snapshot
    rc, st, _, staging = gpu_snapshot(snap, dev, 16 * KiB, seq=4, drain=False)
    assert rc == 0 and st.code == 0 and st.n_dirty == 300
    assert np.array_equal(staging[:st.image_bytes].cpu().numpy(), img_o)
