"""The largest and the smallest refused inputs of crum_snapshot_noalloc: what its
fixed scratch holds is one sum over the table's shape, and a call is refused
exactly when that passes CRUM_NOALLOC_SCRATCH_BYTES.  Tables without shadows and
room for the image's prefix only: no page is read."""
import pytest

from tests.gpu_util import log

pytestmark = pytest.mark.gpu

P, LIMIT, GRAIN = 4096, 64 << 20, 256


def scratch(n_regions, pages):
    up = lambda n: -(-n // GRAIN) * GRAIN  # noqa: E731
    words = -(-pages // 64)
    # region table, request and results; one flag a page; bitmap, prefix sums, slot
    # list, CRCs; no piece CRCs; the chunk's count
    return (up(64 * n_regions) + 2 * GRAIN + up(pages) + up(8 * words) + up(4 * words) +
            2 * up(256 * words) + GRAIN + GRAIN)


@pytest.mark.parametrize("n_regions", [1, 4, 8, 17, 2048])
def test_the_limit_is_where_it_is(n_regions):
    import torch
    import paper_1808_00117_amd as crum
    pages = 64 * max(w for w in range(113000, 115000) if scratch(n_regions, 64 * w) <= LIMIT)
    log(f"[noalloc limit] {n_regions} regions: {pages} pages")
    cur = torch.empty((pages + 64) * P, dtype=torch.uint8, device="cuda")
    prefix = crum.crum_image_prefix_bytes(n_regions, pages + 64)
    staging = torch.empty(prefix, dtype=torch.uint8, device="cuda")
    status = torch.zeros(64, dtype=torch.uint8, pin_memory=True)
    ctx = crum.crum_ctx_create(0)
    try:
        def call(n):
            share = [n // n_regions] * (n_regions - 1)
            share.append(n - sum(share))
            regs, at = [], cur.data_ptr()
            for i, k in enumerate(share):
                regs.append((at, 0, k * P, i))
                at += k * P
            rc = crum.crum_snapshot_noalloc(ctx, regs, P, 0, 1, staging.data_ptr(), prefix, 0, 0,
                                            torch.cuda.current_stream().cuda_stream,
                                            status.data_ptr())
            torch.cuda.synchronize()
            return rc
        assert call(pages + 64) == -9  # CRUM_ELIMIT
        assert call(pages) == crum.CRUM_OK
        st = crum.read_status(status.data_ptr())
        assert st.code == crum.CRUM_ENOSPC and st.n_dirty == st.total_pages == pages
    finally:
        crum.crum_ctx_destroy(ctx)
