"""The shape tuner's choice, on a context that is a table: a parameter that no kernel
looks at is never chosen, however fast its run was; one with an effect is, when its
gain passes the spread."""
from paper_1808_00117_amd import autotune


def test_a_parameter_without_effect_is_never_chosen(monkeypatch):
    ctx = {"pack_depth": 4, "crc_variant": 6, "pack_prefetch": 0, "pack_blocks": 1024}
    start = dict(ctx)
    monkeypatch.setattr(autotune, "current", lambda c: dict(c))
    monkeypatch.setattr(autotune, "apply", lambda c, params: c.update(params))

    def run():
        noise = 0.5 * sum(ctx[k] != start[k] for k in autotune.NO_EFFECT)
        return (0.8 if ctx["pack_blocks"] == 2048 else 1.0) - noise
    space = {"crc_variant": [0, 3], "pack_depth": [8, 16], "pack_prefetch": [1],
             "pack_blocks": [512, 2048]}
    best, trials, stats = autotune.search(ctx, run, space, repeats=1)
    assert best == dict(start, pack_blocks=2048) == ctx
    assert len(trials) == 8 and stats["best_s"] == 0.8
    assert autotune.NO_EFFECT <= set(autotune.PARAMS)
