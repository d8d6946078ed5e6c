"""GPU: selections of overlapping candidate grids against the oracle, bit for
bit: on both sides of the rule that takes candidate rows or tiles (stride 1;
edges 5 and 7 at strides 2 to 4), edges whose region no tile holds, row chunks
ragged at the end, one candidate per axis, full 16-bit values."""

import sys

import numpy as np
import pytest

import oracle
import paper_2308_10868_amd as nrr
from tests.gpu_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,b,stride", [
    ((67, 21, 19), 3, 1), ((66, 22, 17), 5, 2), ((71, 23, 20), 5, 3), ((90, 25, 21), 5, 4),
    ((69, 24, 18), 7, 1), ((75, 26, 19), 7, 2), ((131, 31, 23), 9, 8), ((80, 40, 33), 15, 2),
    ((97, 33, 31), 15, 14), ((9, 10, 11), 9, 8), ((64, 9, 9), 9, 5),
])
@pytest.mark.parametrize("top", [4096, 65536])
def test_overlapping_selection(dims, b, stride, top):
    import torch

    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    print("[gpu-case] overlapping selection", dims, b, stride, top, flush=True)
    sys.stdout.flush()
    rng = np.random.default_rng(b + stride)
    vol = rng.integers(0, top, size=dims[::-1]).astype(np.uint16)
    c = nrr.select_blocks(to_dev(vol), b, stride, 0.3)
    torch.cuda.synchronize()
    assert np.array_equal(c.cpu().numpy(), oracle.select(vol, b, stride, 0.3)[0])
