"""GPU: the directional confidence on both sides of its staging rules against
the oracle: block edges staged in LDS or not (by type), blocks that touch a
face, lie outside or end at the volume's last voxels, row lengths that leave
the last 4-voxel load short of the volume's end."""

import sys

import numpy as np
import pytest

import oracle
from tests.test_gpu_confidence import border_centres, check, gpu_conf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["u16", "f32"])
@pytest.mark.parametrize("b", [3, 5, 7, 9, 11, 13, 15])
def test_staged_confidence(b, dtype):
    import torch

    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    dims = (b + 5, b + 4, b + 3)
    print("[gpu-case] staged confidence", b, dtype, dims, flush=True)
    sys.stdout.flush()
    rng = np.random.default_rng(b)
    if dtype == "u16":
        ref = rng.integers(0, 4096, size=dims[::-1], dtype=np.uint16)
    else:
        ref = (rng.normal(size=dims[::-1]) * 100).astype(np.float32)
    h = (b - 1) // 2
    c = np.concatenate([border_centres(dims, b, rng, 40),
                        np.array([[d - 2 - h for d in dims]], np.int32)])
    conf = rng.random(len(c)).astype(np.float32)
    check(gpu_conf(ref, c, b, conf), oracle.structure_confidence(ref, c, b, conf), conf)
