"""Verified restores of images around the sizes where the order of the two
passes changes (256 and 512 MiB of pages): every byte of the table and its
shadow, and a bad page in either part of the verify found before anything is
written.  The first sizes keep the order, the next are verified in one launch
and the last in two, with pages of one and of several pieces."""
import pytest

from tests.gpu_util import log

pytestmark = pytest.mark.gpu

KiB, MiB = 1 << 10, 1 << 20


@pytest.mark.parametrize("mib", [256, 512, 1024])
@pytest.mark.parametrize("P,more", [(4 * KiB, 0), (4 * KiB, 1), (64 * KiB, 1), (256 * KiB, 1),
                                    (2 * MiB, 3)])
def test_restore_of_large_images(mib, P, more):
    import torch
    import paper_1808_00117_amd as crum
    from paper_1808_00117_amd.api import Snapshotter

    D = mib * MiB // P + more
    log(f"[order] P={P} {D} pages")
    s = Snapshotter(0)
    try:
        n1 = D // 3
        cur = [torch.empty(n * P // 8, dtype=torch.int64, device="cuda").random_()
               for n in (n1, D - n1)]
        shadow = torch.zeros_like(cur[0])
        size = crum.crum_image_bytes(2, D, D, P)
        staging = torch.empty(size, dtype=torch.uint8, device="cuda")
        rc, st = s.snapshot([(c, None, 1 + i) for i, c in enumerate(cur)], P, staging, seq=2)
        assert rc == 0 and st.code == 0 and st.n_dirty == D
        new = [torch.full_like(c, -1) for c in cur]
        table = [(new[0], shadow, 1), (new[1], None, 2)]
        flags = crum.CRUM_VERIFY | crum.CRUM_UPDATE_SHADOW
        data = crum.crum_image_prefix_bytes(2, D)
        for bad in (0, D - 256 * MiB // P - 1, D - 1):
            if bad < 0:
                continue
            at = data + bad * P + P - 5
            staging[at] ^= 4
            rc, st = s.restore(table, None, size, staging, flags=flags)
            assert rc == 0 and st.code == crum.CRUM_ECRC and st.first_bad == bad
            assert all(bool((t == -1).all()) for t in new) and not bool(shadow.any())
            staging[at] ^= 4
        rc, st = s.restore(table, None, size, staging, flags=flags)
        assert rc == 0 and st.code == 0
        assert all(torch.equal(a, b) for a, b in zip(new, cur)) and torch.equal(shadow, cur[0])
    finally:
        s.close()
