"""The launch shapes chosen by the number of tiles (threads per tile of the
sensor adjoint and the inverse transform, transform tile side, sensors of the
propagation adjoint per workgroup): every problem of a batch of any size
gives its own single-context frame bitwise, since no shape changes the order
of a sum; the single frame is checked against the oracle in test_gpu_parity.
A problem of the small system has 5 sensor tiles and 6 small or 3 large
transform tiles; the lines lie at 256 and 1024 tiles and at 320 large ones."""

import numpy as np
import pytest

from synthetic import frozen_flow_frames, get_config, slope_noise

pytestmark = pytest.mark.gpu


def measured(S, k):
    true = next(frozen_flow_frames(S.cfg, 1, 11, first=k))
    s = S.apply_A(np.concatenate([p.astype(np.float64).ravel() for p in true]))
    return (s + slope_noise(S.geom.n_slopes, [w["sigma"] for w in S.cfg["wfs"]], 11, k)).astype(np.float32)


@pytest.mark.parametrize("count", [2, 42, 43, 52, 107, 206])
def test_batch_of_any_size_is_bitwise_the_single_frame(gpu_lib, systems, count):
    import torch
    S = systems("small")
    ctx = gpu_lib.Context(get_config("small"), device=0)
    slopes = [torch.from_numpy(measured(S, k)).cuda() for k in range(3)]
    want = []
    for s in slopes:
        st = torch.zeros(ctx.n_state, device="cuda")
        ly = torch.empty(ctx.n_coeff, device="cuda")
        ctx.reconstruct(s, st, ly, iters=3)
        want.append((st, ly))
    print("[gpu] batch of", count, flush=True)
    batch = gpu_lib.Batch([ctx] * count)
    sts = [torch.zeros(-(-ctx.n_state // 4) * 4, device="cuda")[:ctx.n_state] for _ in range(count)]
    lys = [torch.empty(ctx.n_coeff, device="cuda") for _ in range(count)]
    batch.reconstruct([slopes[k % 3] for k in range(count)], sts, lys, iters=3)
    torch.cuda.synchronize()
    for k in range(count):
        assert torch.equal(sts[k], want[k % 3][0]) and torch.equal(lys[k], want[k % 3][1]), k
    batch.close()
    ctx.close()
