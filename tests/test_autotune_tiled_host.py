"""The autotuner on problems whose transforms are tiles: the shapes of the
level-by-level kernels are not timed there (timings replaced by a stand-in)."""

from types import SimpleNamespace

import pytest

from synthetic import get_config


def context(name, **layer0):
    cfg = get_config(name)
    cfg["layers"][0].update(layer0)
    return SimpleNamespace(cfg=cfg, device=0)


@pytest.mark.parametrize("ctx,shaped", [
    (context("maory_like"), False), (context("vlt_like"), False), (context("tiny"), False),
    (context("maory_like", n=64, levels=6), False),  # six levels, every side 64 or more
    (context("tiny", n=16, levels=3), True), (context("small", levels=2), True),
    (context("vlt_like", n=2048, levels=5), True), (context("tiny", n=64, levels=6), True),
])
def test_rule(lib, ctx, shaped):
    from paper_2202_11945_amd import autotune
    assert autotune.level_by_level([ctx]) == shaped
    assert autotune.level_by_level([context("maory_like"), ctx]) == shaped


@pytest.mark.parametrize("layer0,plans", [({}, 4), ({"n": 16, "levels": 2}, 11)])
def test_only_plans_that_differ_are_timed(lib, monkeypatch, layer0, plans):
    from paper_2202_11945_amd import autotune
    monkeypatch.setattr(autotune, "signature", lambda ctxs, iters: "key")
    seen = []

    def time_plan(ctxs, iters, tuning, steps=10, warmup=3):
        seen.append(tuple(sorted(tuning.items())))
        return 1000.0

    monkeypatch.setattr(autotune, "time_plan", time_plan)
    rec = autotune.tune([context("maory_like", **layer0)] * 2, 4, use_cache=False)
    # 4 and 8 rows, split tiles, two streams; level by level also three sides,
    # the fused levels of the 256 x 256 layer at two of them, and quarters
    assert len(seen) == len(set(seen)) == plans
    assert set(rec["us"]) == {"%d/%d" % (r, p) for r in (32, 64, 128) for p in autotune.PT_ROWS}
    assert (rec["dwt_resident"], rec["pt_rows"], rec["pt_split"], rec["glob_fuse"], rec["res_split"]) == (128, 4, 0, 0, 0)
