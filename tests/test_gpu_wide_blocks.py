"""GPU: the 8-bit matrix-core search of 12-bit blocks with edges 11 to 15
against the dot2 form (NRR_ARITH=dot2 asks for it): the same displacements and
the same bits of the correlation.  Windows from one displacement to several
tiles and phases, blocks at the volume's faces and outside it, and a window
that does not fit (both sides are the dot2 form then)."""

import sys

import numpy as np
import pytest

import paper_2308_10868_amd as nrr
from tests.gpu_util import to_dev, to_host
from tests.test_gpu_aniso_filter import pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["u16 smooth", "u16 noise", "u16 flat", "u16 extremes"])
@pytest.mark.parametrize("b,w", [(b, w) for b in (11, 13, 15) for w in (0, 1, 3, 6, 9, 12)])
def test_same_bits_as_the_dot2_form(monkeypatch, kind, b, w):
    import torch

    for v in ("NRR_ARITH", "NRR_TILE", "NRR_CZ"):
        monkeypatch.delenv(v, raising=False)
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    dims = tuple(b + min(2 * w, 14) + e for e in (9, 6, 3))
    print("[gpu-case] wide blocks", kind, b, w, dims, flush=True)
    sys.stdout.flush()
    ref, flt = pair(kind, dims, b + w)
    rng = np.random.default_rng(b * w)
    h = (b - 1) // 2
    c = [[int(rng.integers(h, d - h)) for d in dims] for _ in range(20)]
    c += [[h] * 3, [d - 1 - h for d in dims], [0, 0, dims[2] - 1], [h, dims[1] - 1 - h, h]]
    c = torch.from_numpy(np.array(c, dtype=np.int32)).cuda()
    r, f = to_dev(ref), to_dev(flt)
    got = [to_host(t) for t in nrr.block_match(r, f, c, b, w)]
    ws = nrr.window_stats(f, b, window=w)
    got2 = [to_host(t) for t in nrr.block_match(r, f, c, b, w, workspace=ws, prepared=True)]
    monkeypatch.setenv("NRR_ARITH", "dot2")
    want = [to_host(t) for t in nrr.block_match(r, f, c, b, w)]
    # the prepared statistics serve either search
    late = [to_host(t) for t in nrr.block_match(r, f, c, b, w, workspace=ws, prepared=True)]
    for a, a2, e, e2, name in zip(got, got2, want, late, ("disp", "ncc", "conf")):
        for x in (a, a2, e2):
            assert np.array_equal(x.view(np.int32), e.view(np.int32)), (kind, b, w, name)
