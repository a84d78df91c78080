"""The diff kernel's grid for a unit count, a group and a limit (host code)."""
import json
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_diff_grid(tmp_path):
    exe = str(tmp_path / "diff_grid")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror",
                        "-I" + os.path.join(ROOT, "paper_1808_00117_amd", "csrc"),
                        os.path.join(ROOT, "tests", "c", "diff_grid_test.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "diff grid: ok" in r.stdout, r.stdout + r.stderr


def test_committed_shapes_do_not_limit_the_grid():
    """The committed classes were tuned when 2048 workgroups were the default, which no
    trial of theirs beat by more than its spread; as a value it is a limit."""
    from paper_1808_00117_amd import autotune
    for classes in json.load(open(autotune.DEFAULT_CACHE)).values():
        for name, entry in classes.items():
            assert "diff_blocks" not in entry["params"], name


@pytest.mark.gpu
def test_the_default_and_what_was_the_default_are_two_values():
    import torch
    import paper_1808_00117_amd as crum
    from paper_1808_00117_amd import autotune
    assert torch.cuda.is_available()  # torch's HIP runtime is loaded first
    ctx = crum.crum_ctx_create(0)
    try:
        default = crum.crum_ctx_get_param(ctx, crum.CRUM_PARAM_DIFF_BLOCKS)
        assert default == 1 << 20
        shapes = autotune.current(ctx)
        autotune.apply(ctx, shapes)  # setting what was read changes nothing
        assert autotune.current(ctx) == shapes
        crum.crum_ctx_set_param(ctx, crum.CRUM_PARAM_DIFF_BLOCKS, 2048)
        assert crum.crum_ctx_get_param(ctx, crum.CRUM_PARAM_DIFF_BLOCKS) == 2048
        with pytest.raises(ValueError):
            crum.crum_ctx_set_param(ctx, crum.CRUM_PARAM_DIFF_BLOCKS, (1 << 20) + 1)
    finally:
        crum.crum_ctx_destroy(ctx)


@pytest.mark.gpu
@pytest.mark.parametrize("P,n_new", [(4096, 8300), (4096, 20001), (16384, 8300)])
def test_tables_that_are_mostly_new(P, n_new):
    """Most pages without a shadow, more units than the limited grid of 8 workgroups per
    compute unit takes in one stride, and shadowed regions before, between and behind
    them: a snapshot, the allocation-free one and a plan give the oracle's image."""
    import numpy as np
    import torch
    import oracle
    import paper_1808_00117_amd as crum
    from paper_1808_00117_amd.api import regions_of
    from tests.gpu_util import image_capacity, log, upload
    log(f"[new] P={P} {n_new} pages")
    rng = np.random.default_rng(n_new)
    regs = []
    for i, n in enumerate((130, n_new, 77, n_new // 2, 300)):
        cur = rng.integers(0, 256, n * P, dtype=np.uint8)
        sh = cur.copy()
        sh[rng.choice(n, n // 5, replace=False) * P + 9] ^= 3
        regs.append((cur, None if i % 2 else sh, i))
    _, img, _ = oracle.snapshot(regs, P, seq=6)
    dev = upload(regs)
    cap = image_capacity(dev, P)
    ctx = crum.crum_ctx_create(0)
    try:
        status = torch.zeros(64, dtype=torch.uint8, pin_memory=True)
        stream = torch.cuda.current_stream().cuda_stream
        table = regions_of(dev)

        def launch(name, staging):
            if name == "plan":
                plan = crum.Plan(ctx, [(table, P, 0, 6)], staging.data_ptr(), cap, 0, 0)
                rc = plan.launch(stream, status.data_ptr())
                torch.cuda.synchronize()
                plan.destroy()
                return rc
            rc = getattr(crum, name)(ctx, table, P, 0, 6, staging.data_ptr(), cap, 0, 0, stream,
                                     status.data_ptr())
            torch.cuda.synchronize()
            return rc
        for name in ("crum_snapshot", "crum_snapshot_noalloc", "plan"):
            staging = torch.zeros(cap, dtype=torch.uint8, device="cuda")
            assert launch(name, staging) == crum.CRUM_OK
            assert np.array_equal(staging[:img.size].cpu().numpy(), img), name
    finally:
        crum.crum_ctx_destroy(ctx)
