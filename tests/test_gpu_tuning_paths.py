"""The launch shapes that a tuning asks for are the ones that run: the stages'
workgroups tell which kernels a plan has, and the frames agree with those of
the other shapes (bitwise where the header says so) or with the oracle."""

import numpy as np
import pytest

from synthetic import get_config
from test_gpu_batch_rules import frames, same
from test_gpu_parity import synth_slopes, to_dev
from test_gpu_transforms import layered

pytestmark = pytest.mark.gpu

STAGE = {"IDWT_RES": 0, "IDWT_GLOB": 1, "P_T": 4, "FDWT_GLOB": 5, "FDWT_RES": 6}


def workgroups(batch, stage):
    return batch.time_stage(STAGE[stage], reps=1)[1]


def pt_tiles(cfg, rows):
    return sum(-(-l["n"] // rows) * -(-l["n"] // 64) for l in cfg["layers"])


# narrow and wide pairs (the 37 m system has up to six corners per node), and a fitting step
@pytest.mark.parametrize("name", ["maory_like", "paper_maory", "small_fit"])
def test_unsplit_propagation_tiles_on_request(gpu_lib, systems, name):
    print("\n[gpu-tune] unsplit tiles", name, flush=True)
    cfg = get_config(name)
    ctx = gpu_lib.Context(cfg, device=0)
    s = [to_dev(synth_slopes(systems(name), 0))]
    out = {}
    # node rows of a tile: 16 and 32 where rows are asked for, 4 split ones by default and on request
    for key, tuning, rows in (("rows 4", {"pt_rows": 4}, 16), ("rows 8", {"pt_rows": 8}, 32), ("default", None, 4),
                              ("split", {"pt_split": 1}, 4), ("split 4", {"pt_rows": 4, "pt_split": 1}, 4)):
        batch = gpu_lib.Batch([ctx], tuning=tuning)
        out[key] = frames(batch, s, cfg["iters"])[0]
        assert workgroups(batch, "P_T") == pt_tiles(cfg, rows), key
        batch.close()
    for key, got in out.items():
        assert same(got, out["default"]), key
    assert np.isfinite(out["default"][1].cpu().numpy()).all()
    ctx.close()


# whole layers of 64 x 64 (vlt_like), tiles, three levels
@pytest.mark.parametrize("name", ["vlt_like", "mid", "small"])
def test_shapes_of_the_level_by_level_kernels_choose_nothing_elsewhere(gpu_lib, systems, name):
    print("\n[gpu-tune] tiled", name, flush=True)
    cfg = get_config(name)
    ctx = gpu_lib.Context(cfg, device=0)
    s = [to_dev(synth_slopes(systems(name), 0))]
    seen = []
    for tuning in (None, 32, {"dwt_resident": 32, "glob_fuse": 1}, {"dwt_resident": 64, "res_split": 4}):
        batch = gpu_lib.Batch([ctx], tuning=tuning)
        seen.append((frames(batch, s, cfg["iters"])[0], [workgroups(batch, k) for k in STAGE if k != "P_T"]))
        batch.close()
    for got, wgs in seen[1:]:
        assert same(got, seen[0][0]) and wgs == seen[0][1]
    ctx.close()


# the autotuner's rule against the library's: a resident side of 32 changes
# the transforms' workgroups where some layer above it is level by level
@pytest.mark.parametrize("grids", [[(32, 3), (64, 5)], [(64, 6), (128, 3)], [(32, 3), (64, 6)], [(64, 4)], [(128, 2)],
                                   [(16, 3), (64, 3)], [(1024, 5)], [(2048, 6)], [(128, 7)]])
def test_the_autotuners_rule_is_the_librarys(gpu_lib, grids):
    from paper_2202_11945_amd import autotune
    print("\n[gpu-tune] rule", grids, flush=True)
    ctx = gpu_lib.Context(layered(grids), device=0)
    wgs = []
    for res in (128, 32):
        batch = gpu_lib.Batch([ctx], tuning=res)
        frames(batch, [to_dev(np.zeros(ctx.n_slopes))], 1)
        wgs.append([workgroups(batch, k) for k in STAGE if k != "P_T"])
        batch.close()
    assert (wgs[0] != wgs[1]) == autotune.level_by_level([ctx])
    ctx.close()
