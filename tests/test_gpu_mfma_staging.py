"""GPU: the matrix-core search's staging at the sizes where it changes form.

The kernel holds the window's rows in registers up to a number of steps and
reads the rest twice (windows of more rows), reads chunks that would pass the
volume's last voxel 8 voxels early and shifts them (blocks at the far corner;
odd shifts only with odd row lengths), and masks the columns past the window
from the value range where the row length is odd.  Every case has blocks on
the far corner and in the interior and is held to the parity rule.
"""

import sys

import numpy as np
import pytest

import oracle
import paper_2308_10868_amd as nrr
from paper_2308_10868_amd import synth
from tests.gpu_util import check_match, to_dev, to_host

pytestmark = pytest.mark.gpu

# (block, window, slack of each axis beyond the full window): the windows
# around and above what the registers hold, and tiny ones; even and odd rows
CASES = [(3, 8, (1, 3, 0)), (3, 13, (0, 1, 2)), (5, 12, (3, 0, 1)), (5, 14, (0, 2, 1)),
         (7, 12, (1, 0, 2)), (7, 13, (2, 1, 0)), (7, 15, (3, 2, 0)), (9, 12, (0, 0, 0)),
         (9, 13, (1, 2, 0)), (3, 1, (0, 1, 0)), (9, 1, (0, 3, 1))]


@pytest.mark.parametrize("b,w,slack", CASES)
def test_staging_forms(b, w, slack):
    import torch

    dims = tuple(2 * w + b + s for s in slack)
    print("[gpu-case] staging", b, w, dims, flush=True)
    sys.stdout.flush()
    if nrr.match_plan(nrr.U16, dims, b, w)["form"] != "mfma":
        pytest.skip("the window does not fit the matrix-core form")
    p = synth.gen_random(1000 + 31 * b + w, dims, "u16", smooth=0.8)
    h = b // 2
    hi = [d - 1 - h for d in dims]
    centers = np.array([[h + w, h + w, h + w], hi, [hi[0] - 1, hi[1], hi[2]],
                        [hi[0] - 2, hi[1] - 1, hi[2]], [hi[0], hi[1], hi[2] - 1], [h, h, h],
                        [hi[0], h, hi[2]], [h, hi[1], hi[2]]], dtype=np.int32)
    ref, flt = to_dev(p.ref), to_dev(p.flt)
    disp, ncc, conf = nrr.block_match(ref, flt, torch.from_numpy(centers).cuda(), b, w)
    torch.cuda.synchronize()
    check_match(p.ref, p.flt, centers, b, w, to_host(disp), to_host(ncc), to_host(conf),
                (b, w, dims))


@pytest.mark.parametrize("b", [3, 5, 7, 9])
def test_wide_records_agree(b):
    """The diagnostic instantiation reads its records through clamped 64-bit
    addresses (the form of volumes with very large planes), the plain one
    through a buffer descriptor: the winners are the same bits."""
    import torch

    w, dims = 6, (2 * 6 + b + 9, 2 * 6 + b + 4, 2 * 6 + b + 5)
    print("[gpu-case] wide records", b, dims, flush=True)
    p = synth.gen_random(77 + b, dims, "u16", smooth=0.8)
    centers = oracle.select(p.ref, b, 3, 0.6)[0]
    ref, flt = to_dev(p.ref), to_dev(p.flt)
    cd = torch.from_numpy(np.ascontiguousarray(centers, dtype=np.int32)).cuda()
    got = nrr.block_match(ref, flt, cd, b, w)
    wide = nrr.block_match_surface(ref, flt, cd, b, w, "mfma")[:3]
    torch.cuda.synchronize()
    for a, c in zip(got, wide):
        assert np.array_equal(to_host(a), to_host(c))
