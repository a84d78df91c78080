"""Pages of many diff units and pieces against the oracle: the flags of a wide
page at unaligned places (smaller pages of another request before it in a
plan), a change in its first, last or a middle unit only, and 2 to 256 pieces
combined, in one launch with pages of a single piece."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import log
from tests.test_gpu_batched import run_plan

pytestmark = pytest.mark.gpu

KiB, MiB = 1 << 10, 1 << 20


def region(rng, n, P, where, rid):
    cur = rng.integers(0, 256, n * P, dtype=np.uint8)
    sh = cur.copy()
    for pg in range(0, n, 2):
        sh[pg * P + {"first": 0, "last": P - 1, "middle": P // 2 + 5}[where]] ^= 0x5A
    return cur, sh, rid


@pytest.mark.parametrize("piece_shift", [12, 14, 16])
@pytest.mark.parametrize("where", ["first", "middle", "last"])
def test_wide_pages_behind_small_ones(piece_shift, where):
    import paper_1808_00117_amd as crum
    from paper_1808_00117_amd.api import Snapshotter

    log(f"[wide] piece_shift={piece_shift} {where}")
    rng = np.random.default_rng(piece_shift)
    sizes = [(1, 4 * KiB), (5, 64 * KiB), (2, 4 * KiB), (3, 1 * MiB), (3, 8 * KiB),
             (9, 16 * KiB), (5, 32 * KiB), (6, 256 * KiB)]
    reqs = [([region(rng, n, P, where, 10 * q)], P, q) for q, (n, P) in enumerate(sizes)]
    reqs.append(([(rng.integers(0, 256, 2 * MiB, dtype=np.uint8), None, 99)], 1 * MiB, 50))
    s = Snapshotter(0)
    try:
        crum.crum_ctx_set_param(s.ctx, crum.CRUM_PARAM_PIECE_SHIFT, piece_shift)
        _, results, _ = run_plan(s, reqs)
    finally:
        s.close()
    sts, imgs = results[0]
    for q, (regs, P, seq) in enumerate(reqs):
        st_o, img_o, _ = oracle.snapshot(regs, P, seq=seq)
        assert sts[q][0] == 0 and np.array_equal(imgs[q], img_o), (q, P)
