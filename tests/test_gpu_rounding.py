"""One rounding per operation, whichever kernels a plan takes: a layer's
inverse transform and the control update give the same bits in the tiled
kernels and in the level-by-level ones."""

import numpy as np
import pytest

from synthetic import random_vector
from test_gpu_parity import to_dev
from test_gpu_transforms import layered

pytestmark = pytest.mark.gpu


# levels of output side above 128 below the finest one, and none
@pytest.mark.parametrize("n,levels", [(64, 5), (256, 5), (512, 3), (512, 5), (1024, 5)])
def test_inverse_transform_rounds_by_the_level_side(gpu_lib, n, levels):
    # a layer of side 16 keeps its problem on the level-by-level kernels
    import torch
    print("\n[gpu-dwt]", n, levels, flush=True)
    tiled = gpu_lib.Context(layered([(n, levels)]), device=0)
    by_level = gpu_lib.Context(layered([(n, levels), (16, 2)]), device=0)
    x = to_dev(random_vector(by_level.n_coeff, 910))
    a = tiled.apply_Winv(x[:n * n].clone())
    b = by_level.apply_Winv(x)[:n * n]
    assert torch.equal(a, b)
    tiled.close()
    by_level.close()


def fma32(a, b, c):
    """a b + c of FP32 arrays, rounded once: the FP64 sum's last bit is set
    when the sum is inexact, so that rounding it to FP32 cannot round twice."""
    p, c = a.astype(np.float64) * b.astype(np.float64), c.astype(np.float64)
    s = p + c
    t = s - p
    err = (p - (s - t)) + (c - t)
    bits = s.view(np.int64)
    toward = np.where((err > 0) == (s > 0), 1, -1)
    odd = np.where((err != 0) & (bits & 1 == 0), bits + np.where(toward > 0, 1, -1), bits)
    return odd.view(np.float64).astype(np.float32)


# one-launch tiles; resident and global levels of the level-by-level kernels
@pytest.mark.parametrize("grids", [[(32, 3), (64, 4)], [(64, 4), (256, 5)], [(16, 2), (64, 2), (256, 3)]])
@pytest.mark.parametrize("loop", ["open", "closed"])
def test_control_update_rounds_the_same_way_everywhere(gpu_lib, grids, loop):
    import torch
    print("\n[gpu-control]", grids, loop, flush=True)
    cfg = layered(grids)
    cfg["gain"], cfg["loop"] = 0.6, loop
    ctx = gpu_lib.Context(cfg, device=0)
    st = torch.zeros(ctx.n_state, device="cuda")
    lay, dm = torch.empty(ctx.n_coeff, device="cuda"), torch.empty(ctx.n_act, device="cuda")
    g = np.float32(cfg["gain"])
    for k in range(3):
        prev = st[3 * ctx.n_coeff:].cpu().numpy()
        ap, a = prev[:ctx.n_act], prev[ctx.n_act:2 * ctx.n_act]
        ctx.reconstruct(to_dev(0.01 * random_vector(ctx.n_slopes, 911, k)), st, lay, dm, iters=3)
        torch.cuda.synchronize()
        v = lay.cpu().numpy()
        gv = np.full_like(v, g)
        want = fma32(gv, v - ap, a) if loop == "closed" else fma32(gv, v, (1 - g) * a)
        for (n, _), off in zip(grids, np.cumsum([0] + [n * n for n, _ in grids])):
            if loop == "open" and n > 128:  # the rounded product is that of v there
                l = slice(off, off + n * n)
                want[l] = fma32(1 - gv[l], a[l], g * v[l])
        assert np.array_equal(dm.cpu().numpy(), want), k
        assert torch.equal(st[3 * ctx.n_coeff + ctx.n_act:3 * ctx.n_coeff + 2 * ctx.n_act], dm), k
    ctx.close()
