"""The level-by-level transforms, which a problem keeps whose layers the tiles
do not take (here one of side 16 and one of two global levels): M x, a frame
from zero, a warm one and one from the true residual, plain and augmented,
for every launch shape, against the oracle; the stages' workgroups tell that
the shape asked for ran."""

import numpy as np
import pytest

from oracle.operators import System
from oracle.solver import State, frame
from parity import check_blocks
from synthetic import get_config, random_vector
from test_gpu_parity import FRAME_ETOL, LAYER_TOL, OP_TOL, synth_slopes, to_dev, to_host
from test_gpu_tuning_paths import workgroups

pytestmark = pytest.mark.gpu

GRIDS = [(16, 3), (64, 4), (256, 3)]


def config(**overrides):
    cfg = get_config("small", **overrides)
    for l, (n, levels) in zip(cfg["layers"], GRIDS):
        l["n"], l["levels"] = n, levels
    return cfg


_oracle = {}


def oracle(augment=0):
    if augment not in _oracle:
        _oracle[augment] = System(config(augment=augment))
    return _oracle[augment]


# workgroups of the resident inverse levels, of its global and of the forward's global levels:
# 32 x 32 tiles of every level above the resident side, or of two of them at once
SHAPES = [
    (None, 3, 64, 64),
    ({"dwt_resident": 64}, 3, 16 + 64, 64 + 16),
    ({"dwt_resident": 32}, 3, 4 + 4 + 16 + 64, 64 + 16 + 4 + 4),
    ({"res_split": 4}, 12, 64, 64),
    ({"dwt_resident": 64, "res_split": 4}, 12, 16 + 64, 64 + 16),
    ({"dwt_resident": 64, "glob_fuse": 1}, 3, 64, 64),
    ({"dwt_resident": 32, "glob_fuse": 1}, 3, 4 + 4 + 64, 64 + 4 + 4),
    ({"dwt_resident": 64, "glob_fuse": 1, "res_split": 4}, 12, 64, 64),
]


@pytest.mark.parametrize("tuning,resident,inverse,forward", SHAPES)
@pytest.mark.parametrize("augment", [0, 2])
def test_frames(gpu_lib, tuning, resident, inverse, forward, augment):
    import torch
    print("\n[gpu-level]", tuning, "augment", augment, flush=True)
    S = oracle(augment)
    ctx = gpu_lib.Context(config(augment=augment), device=0, tuning=tuning)
    n, o = S.geom.n_coeff, S.geom.layer_off
    if augment == 0:
        x = random_vector(n, 930)
        check_blocks(to_host(ctx.apply_M(to_dev(x))), S.apply_M(x), o, OP_TOL, "M x layer")
    batch = gpu_lib.Batch([ctx], tuning=tuning)
    refresh = augment == 0
    if refresh:
        batch.set_refresh(2)
    st, lay = torch.zeros(ctx.n_state, device="cuda"), torch.empty(n, device="cuda")
    for k in range(3):
        before = to_host(st)
        s = synth_slopes(S, k)
        batch.reconstruct([to_dev(s)], [st], [lay], iters=4, use_graph=bool(k))
        got = State.unpack(to_host(st), n, n, augment)
        ref, phi = frame(S, State.unpack(before, n, n, augment), s.astype(np.float64), iters=4,
                         refresh=refresh and k == 2)
        tag = "frame %d" % k
        check_blocks(to_host(lay), phi, o, LAYER_TOL, tag + " layers", FRAME_ETOL)
        check_blocks(got.c, ref.c, o, LAYER_TOL, tag + " c", FRAME_ETOL)
        check_blocks(got.r, ref.r, o, LAYER_TOL, tag + " r", FRAME_ETOL, scale=ref.b)
    assert [workgroups(batch, k) for k in ("IDWT_RES", "IDWT_GLOB", "FDWT_GLOB")] == [resident, inverse, forward]
    batch.close()
    ctx.close()


@pytest.mark.parametrize("side", [0, 4])
def test_converged_solve(gpu_lib, side):
    # the search direction with the coarse-level correction, formed ahead of
    # the level-by-level inverse transform; bound as in the solves of the tiles
    from oracle.gradients import exact_solve
    cfg = config()
    cfg["layers"][2]["n"], cfg["layers"][2]["levels"] = 32, 2
    S = System(cfg)
    ctx = gpu_lib.Context(cfg, device=0)
    ctx.set_solve_coarse(side)
    g = random_vector(S.geom.n_coeff, 931).astype(np.float32)
    print("\n[gpu-level] solve, coarse side", side, flush=True)
    x, _, r = ctx.solve_map(g_layers=to_dev(g), rtol=1e-10, max_iters=40000)
    ref = exact_solve(S, S.W_invT(g.astype(np.float64)))
    assert r <= 1e-10
    assert np.linalg.norm(to_host(x) - ref) / np.linalg.norm(ref) <= 1e-6
    ctx.close()
