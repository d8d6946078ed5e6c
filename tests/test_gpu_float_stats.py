"""GPU: the float statistics table, every record against NumPy (white box: one
record {double s, double r} per block origin, s the block's sum, r =
1/sqrt(N sum v^2 - s^2) or 0 for a flat block).  Voxels are whole numbers below
1024, so that every sum is exact in 64 bits in any order: s is compared for
equality, r within the rounding of one root and one division.  Edges with an
unrolled ring (5, 7, 9) and without, z extents around one and several rounds of
the ring, ragged 64 x 4 tiles."""

import sys

import numpy as np
import pytest

import paper_2308_10868_amd as nrr
from tests.gpu_util import to_dev
from tests.test_gpu_stats_table import box_sum

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b", [3, 5, 7, 9, 11, 13, 15])
@pytest.mark.parametrize("extra", [(0, 0, 0), (1, 2, 1), (63, 3, 5), (64, 4, 10), (70, 9, 41)])
def test_float_statistics_are_exact(b, extra):
    import torch

    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    nx, ny, nz = (b + e for e in extra)
    print("[gpu-case] float statistics", b, (nx, ny, nz), flush=True)
    sys.stdout.flush()
    rng = np.random.default_rng(b)
    v = rng.integers(-1023, 1024, size=(nz, ny, nx))
    v[:, : b + 1, : b + 1] = 77  # flat blocks
    ws = nrr.window_stats(to_dev(v.astype(np.float32)), b)
    torch.cuda.synchronize()
    shape = tuple(e + 1 for e in extra[::-1])
    rec = ws.cpu().numpy()[: int(np.prod(shape)) * 16].view(np.float64).reshape(shape + (2,))
    s, q = box_sum(v, b), box_sum(v * v, b)
    var = (b ** 3 * q - s * s).astype(np.float64)
    r = np.zeros(shape)
    r[var > 0] = 1.0 / np.sqrt(var[var > 0])
    assert np.array_equal(rec[..., 0], s)
    assert np.allclose(rec[..., 1], r, rtol=2.0 ** -50, atol=0)
