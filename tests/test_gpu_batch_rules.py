"""A problem's results do not depend on the batch that it is in: the kernels
and tile sides that a plan chooses by its number of tiles, or by the layers of
other problems, give every problem its single-context bits."""

import pytest

from synthetic import random_vector
from test_gpu_parity import to_dev
from test_gpu_transforms import layered

pytestmark = pytest.mark.gpu


def slopes_of(ctx, count):
    return [to_dev(0.01 * random_vector(ctx.n_slopes, 920, k)) for k in range(count)]


def new_state(ctx):
    import torch
    return torch.zeros(-(-ctx.n_state // 4) * 4, device="cuda")[:ctx.n_state]


def frames(batch, slopes, iters):
    """State and layers of every problem after two frames."""
    import torch
    st = [new_state(c) for c in batch.ctxs]
    ly = [torch.empty(c.n_coeff, device="cuda") for c in batch.ctxs]
    for _ in range(2):
        batch.reconstruct(slopes, st, ly, iters=iters)
    torch.cuda.synchronize()
    return list(zip(st, ly))


def alone(lib, ctx, slopes, iters):
    b = lib.Batch([ctx])
    out = [frames(b, [s], iters)[0] for s in slopes]
    b.close()
    return out


def same(a, b):
    import torch
    return all(torch.equal(x, y) for x, y in zip(a, b))


# 5 transform tiles of 64 a side per problem; the tile sides change at 64 and at 320 of them
@pytest.mark.parametrize("count,streams", [(12, 1), (13, 1), (63, 1), (64, 1), (14, 2)])
def test_frames_on_either_side_of_the_tile_rules(gpu_lib, count, streams):
    print("\n[gpu-batch]", count, "problems,", streams, "streams", flush=True)
    ctx = gpu_lib.Context(layered([(64, 4), (128, 5)]), device=0)
    s = slopes_of(ctx, 3)
    want = alone(gpu_lib, ctx, s, 20)
    batch = gpu_lib.Batch([ctx] * count, tuning={"streams": streams})
    got = frames(batch, [s[k % 3] for k in range(count)], 20)
    for k in range(count):
        assert same(got[k], want[k % 3]), k
    batch.close()
    ctx.close()


def test_solve_on_either_side_of_the_tile_rules(gpu_lib):
    # thousands of steps carry a difference in the last bit of an inner
    # product into the solution
    import torch
    ctx = gpu_lib.Context(layered([(64, 4), (128, 5)]), device=0)
    rhs = ctx.rhs(slopes_of(ctx, 1)[0])
    x, it, _ = ctx.solve(rhs, rtol=1e-9, max_iters=6000)
    batch = gpu_lib.Batch([ctx] * 13)
    print("\n[gpu-batch] solve,", it, "steps", flush=True)
    xs, itb, _ = batch.solve([rhs] * 13, rtol=1e-9, max_iters=6000)
    torch.cuda.synchronize()
    assert itb == it
    for v in xs:
        assert torch.equal(v, x)
    batch.close()
    ctx.close()


# problem, its mates: layers that the tiled transforms do not take (side 16),
# or that make another choice of tiles (side 32; a tail of another size; six levels)
MATES = [
    ([(64, 4), (128, 5)], [[(16, 2)]]),
    ([(512, 5), (64, 4)], [[(16, 2)], [(64, 2), (256, 2)]]),
    ([(64, 4), (64, 3)], [[(512, 5)]]),
    ([(256, 6), (64, 3)], [[(32, 3)], [(16, 3), (64, 2)]]),
    ([(256, 6)], [[(256, 5)]] * 20),
    ([(16, 3), (64, 2)], [[(16, 2), (128, 2)], [(64, 4)]]),
]


@pytest.mark.parametrize("own,mates", MATES)
def test_frames_beside_other_systems(gpu_lib, own, mates):
    print("\n[gpu-batch]", own, "beside", mates[:3], flush=True)
    ctx = gpu_lib.Context(layered(own), device=0)
    other = {repr(m): gpu_lib.Context(layered(m), device=0) for m in mates}
    s = slopes_of(ctx, 2)
    want = alone(gpu_lib, ctx, s, 8)
    ctxs = [ctx] + [other[repr(m)] for m in mates] + [ctx]
    batch = gpu_lib.Batch(ctxs)
    got = frames(batch, [s[0]] + [slopes_of(c, 1)[0] for c in ctxs[1:-1]] + [s[1]], 8)
    assert same(got[0], want[0]) and same(got[-1], want[1])
    x = to_dev(random_vector(ctx.n_coeff, 921))
    xs = [x] + [to_dev(random_vector(c.n_coeff, 922)) for c in ctxs[1:]]
    for apply, one in ((batch.apply_Winv, ctx.apply_Winv), (batch.apply_WinvT, ctx.apply_WinvT)):
        assert same([apply(xs)[0]], [one(x)])
    batch.close()
    for c in [ctx] + list(other.values()):
        c.close()


def test_solves_beside_other_systems(gpu_lib):
    # the coarse-level correction where one problem's inverse transform is
    # tiled and the other's level by level; 48 steps, fewer than either needs
    # to end a refinement sweep, so that both take all of them in any batch
    import torch
    a, b = (gpu_lib.Context(layered(g), device=0) for g in ([(64, 4), (128, 5)], [(16, 3), (128, 5)]))
    rhs = [c.rhs(slopes_of(c, 1)[0]) for c in (a, b)]
    one = [c.solve(r, rtol=0.0, max_iters=48) for c, r in zip((a, b), rhs)]
    batch = gpu_lib.Batch([a, b, a])
    print("\n[gpu-batch] solves of two systems", flush=True)
    xs, it, _ = batch.solve([rhs[0], rhs[1], rhs[0]], rtol=0.0, max_iters=48)
    torch.cuda.synchronize()
    assert it == one[0][1] == one[1][1] == 48
    assert torch.equal(xs[0], one[0][0]) and torch.equal(xs[1], one[1][0]) and torch.equal(xs[2], one[0][0])
    batch.close()
    a.close()
    b.close()
