"""The coarse-level correction of the converged solves where it is split over
workgroups: more problems of one system than a workgroup takes (8) beside
another system, and coarse blocks whose rows are no whole 16-byte runs
(side 2: 12 unknowns; side 16: 768).  Against the dense FP64 solution; a
residual ratio of 1e-10 leaves at most 1e-6 here, as in the single solve."""

import os
import sys

import numpy as np
import pytest

from oracle.gradients import exact_solve
from oracle.operators import System
from synthetic import random_vector

sys.path.insert(0, os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden"))
from make_gradients import frames_for  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("side", [2, 16])
def test_solves_of_ten_problems_and_a_second_system(gpu_lib, side):
    import torch
    cfg, cfg_true, _ = frames_for("grad_small", 1)
    S = [System(cfg), System(cfg_true)]
    ctx = [gpu_lib.Context(c, device=0) for c in (cfg, cfg_true)]
    which = [0] * 4 + [1] + [0] * 6
    batch = gpu_lib.Batch([ctx[w] for w in which])
    batch.set_solve_coarse(side)
    g = [random_vector(S[0].geom.n_coeff, 540, k).astype(np.float32) for k in range(len(which))]
    print("[gpu-grad] batch of 10 + 1 adjoint solves, coarse side", side, flush=True)
    x, it, r = batch.solve_map(g_layers=[torch.from_numpy(v).cuda() for v in g], rtol=1e-10, max_iters=40000)
    torch.cuda.synchronize()
    assert r <= 1e-10
    for k, w in enumerate(which):
        ref = exact_solve(S[w], S[w].W_invT(g[k].astype(np.float64)))
        err = np.linalg.norm(x[k].cpu().numpy() - ref) / np.linalg.norm(ref)
        assert err <= 1e-6, (k, err)
    batch.close()
    for c in ctx:
        c.close()
