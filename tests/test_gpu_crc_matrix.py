"""Page CRCs from the matrix cores against the oracle: every bit position of a
4 KiB batch by itself, and batches of zeros, of ones (the largest sums) and of
random bytes at the smallest and largest pages and pieces, packed and verified."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import gpu_snapshot, log, upload

pytestmark = pytest.mark.gpu

KiB = 1 << 10


def check(cur, P, piece_shift):
    import torch
    import paper_1808_00117_amd as crum
    from paper_1808_00117_amd.api import Snapshotter

    s = Snapshotter(0)
    try:
        crum.crum_ctx_set_param(s.ctx, crum.CRUM_PARAM_PIECE_SHIFT, piece_shift)
        regs = [(cur, None, 9)]
        st_o, img_o, _ = oracle.snapshot(regs, P, seq=1)
        dev = upload(regs)
        rc, st, img, staging = gpu_snapshot(s, dev, P, seq=1)
        assert rc == 0 and st.code == 0
        assert np.array_equal(img, img_o)
        target = torch.empty(cur.size, dtype=torch.uint8, device="cuda")
        h = torch.from_numpy(img).pin_memory()
        rc, st = s.restore([(target, None, 9)], h, img.size, staging, flags=crum.CRUM_VERIFY)
        assert rc == 0 and st.code == 0
        assert torch.equal(target, dev[0][0])
        # the last bit of the last page flipped: found, in its slot
        at = st_o.image_bytes - ((4 * st_o.n_dirty + 7) & ~7) - 1
        h[at] ^= 0x80
        rc, st = s.restore([(target, None, 9)], h, img.size, staging, flags=crum.CRUM_VERIFY)
        assert rc == 0 and st.code == crum.CRUM_ECRC and st.first_bad == st_o.n_dirty - 1
    finally:
        s.close()


def test_every_bit_of_a_batch():
    P = 4 * KiB
    cur = np.zeros((8 * P, P), np.uint8)
    bit = np.arange(8 * P)
    cur[bit, bit >> 3] = 1 << (bit & 7)
    log("[crc] one bit per page")
    check(cur.reshape(-1), P, 14)


@pytest.mark.parametrize("fill", ["zeros", "ones", "random"])
@pytest.mark.parametrize("P,piece_shift", [(4 * KiB, 12), (8 * KiB, 16), (16 * KiB, 12),
                                           (64 * KiB, 14), (64 * KiB, 16), (256 * KiB, 16)])
def test_pages_and_pieces(P, piece_shift, fill):
    log(f"[crc] P={P} piece_shift={piece_shift} {fill}")
    n = 5
    cur = {"zeros": np.zeros(n * P, np.uint8), "ones": np.full(n * P, 255, np.uint8),
           "random": np.random.default_rng(P + piece_shift).integers(0, 256, n * P,
                                                                     dtype=np.uint8)}[fill]
    check(cur, P, piece_shift)


@pytest.mark.parametrize("n_pages", [1024 * 3 + 1, 262144 + 77, 3 * 262144 // 2])
def test_checksums_of_long_messages(n_pages):
    """crcs_crc and meta_crc of CRC arrays and prefixes of one to hundreds of
    4 KiB batches (shares followed by more than 255 batches)."""
    import torch
    import paper_1808_00117_amd as crum
    from paper_1808_00117_amd.api import Snapshotter

    P = 4 * KiB
    log(f"[crc] {n_pages} pages")
    s = Snapshotter(0)
    try:
        cur = torch.empty(n_pages * P // 8, dtype=torch.int64, device="cuda").random_()
        size = crum.crum_image_bytes(1, n_pages, n_pages, P)
        staging = torch.empty(size, dtype=torch.uint8, device="cuda")
        rc, st = s.snapshot([(cur, None, 3)], P, staging, seq=2)
        assert rc == 0 and st.code == 0 and st.n_dirty == n_pages
        prefix_end = 64 + 32 + 8 * ((n_pages + 63) // 64)
        prefix = staging[:prefix_end].cpu().numpy()
        at = crum.crum_image_prefix_bytes(1, n_pages) + n_pages * P
        crcs = staging[at:at + 4 * n_pages].cpu().numpy()
        meta, crcs_crc = prefix[56:64].copy().view(np.uint32)
        assert crcs_crc == oracle.crc32c(crcs)
        prefix[56:60] = 0
        assert meta == oracle.crc32c(prefix)
        rc, st = s.restore([(cur, None, 3)], None, size, staging, flags=crum.CRUM_VERIFY)
        assert rc == 0 and st.code == 0
    finally:
        s.close()
