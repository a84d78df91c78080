"""A restore from an image in device memory reads the header and the region table
back to the host, by a kernel or by a copy: tables at the size where that changes
(192 KiB, 6142 regions) and far from it, restored, and refused for one wrong
length."""
import pytest

from tests.gpu_util import log

pytestmark = pytest.mark.gpu

P = 4096


@pytest.mark.parametrize("n_regions", [1, 300, 6142, 6143, 9000])
def test_rollback_of_many_regions(n_regions):
    import torch
    import paper_1808_00117_amd as crum
    from paper_1808_00117_amd.api import Snapshotter
    log(f"[tables] {n_regions} regions")
    s = Snapshotter(0)
    try:
        cur = torch.empty(n_regions * P // 8, dtype=torch.int64, device="cuda").random_()
        new = torch.zeros_like(cur)
        table = [[(t.data_ptr() + i * P, 0, P, i) for i in range(n_regions)] for t in (cur, new)]
        size = crum.crum_image_bytes(n_regions, n_regions, n_regions, P)
        staging = torch.empty(size, dtype=torch.uint8, device="cuda")
        rc, st = s.snapshot(table[0], P, staging)
        assert rc == 0 and st.code == 0 and st.n_dirty == n_regions
        wrong = table[1][:-1] + [table[1][-1][:2] + (0, n_regions - 1)]
        rc, st = s.restore(wrong, None, size, staging, flags=crum.CRUM_VERIFY)
        assert rc == st.code == crum.CRUM_EMISMATCH and not bool(new.any())
        rc, st = s.restore(table[1], None, size, staging, flags=crum.CRUM_VERIFY)
        assert rc == 0 and st.code == 0 and torch.equal(new, cur)
    finally:
        s.close()
