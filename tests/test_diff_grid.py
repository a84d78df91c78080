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
