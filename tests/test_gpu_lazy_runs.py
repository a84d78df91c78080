"""On-demand restores whose windows hold many runs: more than one launch's list of
runs, runs read in place beside copied ones, and a bad page among them, after
which nothing of its run or of a later one is written."""
import numpy as np
import pytest

from tests.gpu_util import log
from tests.test_gpu_lazy import Session, env, make_case  # noqa: F401

pytestmark = pytest.mark.gpu

KiB = 1 << 10
P = 64 * KiB
SMALL, LARGE = 37, 40  # regions of three pages, and pages of the copied run
COUNTS = [3] * SMALL + [LARGE] + [3] * 3


def start(env, flags, bad_slot=None):
    """A session over an image with every page, the middle page of every small
    region fetched: what is left are runs of one or two pages and a copied one."""
    crum, ctx, status = env
    regs, img = make_case(COUNTS, P, 2.0, seed=5)
    if bad_slot is not None:
        img = img.copy()
        data_off = int(np.frombuffer(img[48:56].tobytes(), np.uint64)[0])
        img[data_off + bad_slot * P + 77] ^= 4
    s = Session(crum, ctx, status, regs, img, P, flags, 0)
    for r, n in enumerate(COUNTS):
        if n == 3:
            s.lz.touch(r, P, 1, s.stream.cuda_stream)
    s.stream.synchronize()
    return s, regs


def pages(t):
    return t.cpu().numpy().reshape(-1, P)


@pytest.mark.parametrize("flags", [0, 2])
def test_many_runs(env, flags):
    log(f"[lazy] many runs flags={flags}")
    s, regs = start(env, flags)
    s.lz.finish(s.stream.cuda_stream, s.status.data_ptr())
    s.stream.synchronize()
    assert s.st().code == 0 and s.lz.stats()["pages_fetched"] == sum(COUNTS)
    for t, (new, _, _) in zip(s.targets, regs):
        assert np.array_equal(t.cpu().numpy(), new)
    s.lz.close()


# pages to the left: in the first list, at its last run, in the second, in the
# copied run (its last page), behind it
@pytest.mark.parametrize("bad", [(0, 0), (14, 2), (30, 0), (SMALL, LARGE - 1), (SMALL + 2, 2)])
def test_bad_page_among_runs(env, bad):
    region, page = bad
    first = np.concatenate([[0], np.cumsum(COUNTS)])
    slot = int(first[region]) + page
    log(f"[lazy] bad page {bad}, slot {slot}")
    s, regs = start(env, 2, slot)
    s.lz.finish(s.stream.cuda_stream, s.status.data_ptr())
    s.stream.synchronize()
    st = s.st()
    assert st.code == -3 and st.first_bad == slot
    # the bad run starts behind the last page that was fetched before
    fetched = {int(first[r]) + 1 for r, n in enumerate(COUNTS) if n == 3}
    run = slot
    while run > 0 and run - 1 not in fetched:
        run -= 1
    for r, (t, (new, old, _)) in enumerate(zip(s.targets, regs)):
        got, new, old = pages(t), new.reshape(-1, P), old.reshape(-1, P)
        for i in range(COUNTS[r]):
            k = int(first[r]) + i
            want = new if k in fetched or k < run else old
            assert np.array_equal(got[i], want[i]), (r, i)
    # a later call writes nothing, also before the bad page
    before = [t.clone() for t in s.targets]
    s.lz.touch(0, 0, 3 * P, s.stream.cuda_stream, s.status.data_ptr())
    s.stream.synchronize()
    assert s.st().code == -3
    assert all((a == b).all().item() for a, b in zip(before, s.targets))
    s.lz.close()


def test_nothing_is_written_after_an_earlier_call_failed(env):
    log("[lazy] a call after a bad page")
    s, regs = start(env, 2, int(sum(COUNTS[:20])))
    s.lz.touch(20, 0, 1, s.stream.cuda_stream, s.status.data_ptr())
    s.stream.synchronize()
    assert s.st().code == -3
    before = [t.clone() for t in s.targets]
    s.lz.touch(3, 0, 1, s.stream.cuda_stream, s.status.data_ptr())  # a lower slot, a good page
    s.lz.finish(s.stream.cuda_stream, s.status.data_ptr())
    s.stream.synchronize()
    assert s.st().code == -3 and s.st().first_bad == sum(COUNTS[:20])
    assert all((a == b).all().item() for a, b in zip(before, s.targets))
    s.lz.close()
