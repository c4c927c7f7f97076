"""One rounding per operation, whichever kernels a plan takes: a layer's
inverse transform gives the same bits in the tiled kernels and in the
level-by-level ones."""

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
