"""The transforms at the edges of their tiles: layers of one and of many
tiles, of every number of levels that the one-launch inverse transform takes
and of some that it leaves to the level-by-level kernels, against the FP64
oracle (1e-5 per operator, tests/parity.py); frames and transforms with
buffers of any 4-byte alignment and in place, bitwise."""

import numpy as np
import pytest

from oracle.operators import System
from parity import check_blocks
from synthetic import get_config, random_vector
from test_gpu_parity import OP_TOL, to_dev, to_host

pytestmark = pytest.mark.gpu


def layered(grids):
    """The tiny system with layers of the given (side, levels)."""
    cfg = get_config("tiny")
    cfg["layers"] = [{"h": 500.0 * k, "n": n, "levels": lv, "cn2": 1.0 / len(grids)} for k, (n, lv) in enumerate(grids)]
    return cfg


# copies: enough problems of a batch for the larger tile (320 tiles of 64)
@pytest.mark.parametrize("grids,copies", [
    ([(32, 3), (32, 4), (32, 5), (64, 5), (128, 5), (256, 5)], 1),   # tiles of 32, one to 64 of them
    ([(64, 3), (128, 4), (512, 5)], 1),                              # forward tiles of 64 from 64 of them on
    ([(64, 3), (1024, 7)], 1),
    ([(64, 3), (64, 6), (128, 6), (256, 5)], 15),                    # tiles of 64
    ([(512, 4), (512, 6)], 3),
    ([(16, 3), (64, 2), (64, 6), (128, 5), (256, 2)], 2),            # level by level
])
def test_transforms_at_tile_edges(gpu_lib, grids, copies):
    print("\n[gpu-dwt]", grids, "x", copies, flush=True)
    cfg = layered(grids)
    S = System(cfg)
    ctx = gpu_lib.Context(cfg, device=0)
    batch = gpu_lib.Batch([ctx] * copies)
    x = [random_vector(S.geom.n_coeff, 900, k) for k in range(copies)]
    phi = batch.apply_Winv([to_dev(v) for v in x])
    c = batch.apply_WinvT([to_dev(v) for v in x])
    for k in {0, copies - 1}:
        check_blocks(to_host(phi[k]), S.W_inv(x[k]), S.geom.layer_off, OP_TOL, "W^-1 layer")
        check_blocks(to_host(c[k]), S.W_invT(x[k]), S.geom.layer_off, OP_TOL, "W^-T layer")
    check_blocks(to_host(ctx.apply_M(to_dev(x[0]))), S.apply_M(x[0]), S.geom.layer_off, OP_TOL, "M x layer")
    batch.close()
    ctx.close()


@pytest.mark.parametrize("loop", ["open", "closed"])
def test_outputs_of_any_alignment(gpu_lib, systems, loop):
    # layers and commands written to addresses 4 bytes past a multiple of 16
    import torch
    S = systems("small", loop=loop, gain=0.5)
    ctx = gpu_lib.Context(get_config("small", loop=loop, gain=0.5), device=0)
    s = to_dev(S.apply_A(random_vector(S.geom.n_coeff, 901)).astype(np.float32))
    out = []
    for shift in (0, 1):
        st = torch.zeros(ctx.n_state, device="cuda")
        bufs = [torch.zeros(ctx.n_coeff + shift, device="cuda")[shift:] for _ in range(3)]
        for _ in range(2):
            ctx.reconstruct(s, st, bufs[0], bufs[1], iters=3)
        ctx.apply_Winv(st[:ctx.n_coeff].clone(), bufs[2])
        torch.cuda.synchronize()
        out.append([st] + bufs)
    for a, b in zip(*out):
        assert torch.equal(a, b)
    ctx.close()


@pytest.mark.parametrize("grids", [[(32, 3), (64, 4)], [(64, 3), (256, 5)], [(16, 2), (64, 3)]])
def test_transforms_in_place_and_unaligned(gpu_lib, grids):
    import torch
    cfg = layered(grids)
    ctx = gpu_lib.Context(cfg, device=0)
    batch = gpu_lib.Batch([ctx] * 2)
    n = ctx.n_coeff
    x = [to_dev(random_vector(n, 902, k)) for k in range(2)]
    for apply in (batch.apply_Winv, batch.apply_WinvT):
        ref = apply(x)
        own = [v.clone() for v in x]
        apply(own, own)                      # in place
        cross = [v.clone() for v in x]
        apply(cross, cross[::-1])            # each problem into the other's input
        odd = [torch.cat([v[:1], v])[1:] for v in x]
        odd_out = [torch.empty(n + 1, device="cuda")[1:] for _ in x]
        apply(odd, odd_out)                  # 4 bytes past a multiple of 16
        torch.cuda.synchronize()
        for k in range(2):
            assert torch.equal(own[k], ref[k]) and torch.equal(cross[1 - k], ref[k]) and torch.equal(odd_out[k], ref[k])
    batch.close()
    ctx.close()
