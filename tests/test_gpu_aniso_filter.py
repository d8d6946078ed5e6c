"""GPU: the per-axis search behind the matrix-core filter against the FMA form
(NRR_ANISO_TILE asks for it): the same bits, for 12-bit and float data, over
the filter's compiled shapes (z edges 3-9, small and large x and y edges) and
the sizes it leaves to the FMA form."""

import sys

import numpy as np
import pytest

import paper_2308_10868_amd as nrr
from paper_2308_10868_amd import synth
from tests.gpu_util import to_dev, to_host
from tests.test_gpu_f32_filter import volumes

pytestmark = pytest.mark.gpu

# block edges and half windows (x, y, z)
SIZES = [((7, 7, 3), (10, 10, 4)), ((3, 5, 3), (4, 6, 2)), ((9, 9, 3), (5, 4, 1)),
         ((5, 5, 5), (3, 3, 3)), ((7, 5, 5), (6, 0, 2)), ((9, 7, 5), (3, 5, 4)),
         ((7, 7, 7), (4, 4, 4)), ((9, 9, 7), (2, 3, 5)), ((9, 9, 9), (6, 5, 4)),
         ((1, 9, 9), (5, 2, 0)), ((9, 1, 3), (0, 0, 0)), ((9, 9, 9), (15, 15, 15)),
         ((3, 3, 1), (3, 3, 3)), ((11, 5, 3), (3, 3, 2)),
         # windows large enough for the filter, for each of its shapes
         ((5, 5, 3), (8, 7, 4)), ((9, 9, 3), (9, 7, 2)), ((5, 5, 5), (8, 8, 5)),
         ((7, 7, 5), (9, 8, 4)), ((9, 9, 5), (7, 9, 4)), ((7, 7, 7), (8, 8, 4)),
         ((9, 7, 7), (6, 8, 3))]


def pair(kind, dims, seed):
    if kind.startswith("f32"):
        return volumes(kind[4:], dims, seed)
    nx, ny, nz = dims
    rng = np.random.default_rng(seed)
    p = synth.gen_random(seed, dims, "u16", smooth=1.5)
    ref, flt = p.ref.copy(), p.flt.copy()
    if kind == "u16 noise":
        ref = rng.integers(0, 4096, size=ref.shape, dtype=np.uint16)
        flt = rng.integers(0, 4096, size=ref.shape, dtype=np.uint16)
    elif kind == "u16 flat":
        ref[:, :, : nx // 2] = 700
        flt[:, : ny // 2] = 900
    elif kind == "u16 extremes":
        ref = (rng.integers(0, 2, size=ref.shape) * 4095).astype(np.uint16)
        flt = (rng.integers(0, 2, size=ref.shape) * 4095).astype(np.uint16)
    return ref, flt


@pytest.mark.parametrize("kind", ["u16 smooth", "u16 noise", "u16 flat", "u16 extremes",
                                  "f32 smooth", "f32 noise", "f32 periodic", "f32 flat",
                                  "f32 decades", "f32 bad"])
@pytest.mark.parametrize("b,w", SIZES)
def test_same_bits_as_the_fma_form(monkeypatch, kind, b, w):
    import torch

    for v in ("NRR_ANISO_ARITH", "NRR_ANISO_TILE", "NRR_ANISO_CZ"):
        monkeypatch.delenv(v, raising=False)
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    dims = tuple(min(2 * q, 12) + e + 9 + i for i, (e, q) in enumerate(zip(b, w)))
    print("[gpu-case] per-axis filter", kind, b, w, dims, flush=True)
    sys.stdout.flush()
    ref, flt = pair(kind, dims, sum(b) + sum(w))
    rng = np.random.default_rng(3)
    h = [(e - 1) // 2 for e in b]
    c = [[int(rng.integers(k, d - k)) for k, d in zip(h, dims)] for _ in range(24)]
    c += [h, [d - 1 - k for k, d in zip(h, dims)], [0, 0, dims[2] - 1]]
    c = torch.from_numpy(np.array(c, dtype=np.int32)).cuda()
    r, f = to_dev(ref), to_dev(flt)
    got = [to_host(t) for t in nrr.block_match_aniso(r, f, c, b, w)]
    monkeypatch.setenv("NRR_ANISO_TILE", "8")
    want = [to_host(t) for t in nrr.block_match_aniso(r, f, c, b, w)]
    for a, e, name in zip(got, want, ("disp", "ncc", "conf")):
        assert np.array_equal(a.view(np.int32), e.view(np.int32)), (kind, b, w, name)


@pytest.mark.parametrize("b,w", [((7, 7, 3), (10, 10, 4)), ((7, 7, 3), (5, 4, 4)),
                                 ((9, 9, 5), (7, 9, 4))])
def test_zero_keys_of_either_sign(monkeypatch, b, w):
    """Float texture far below the common level: every key is a zero."""
    import torch
    from tests.test_gpu_f32_filter import level_pair

    for v in ("NRR_ANISO_ARITH", "NRR_ANISO_TILE", "NRR_ANISO_CZ"):
        monkeypatch.delenv(v, raising=False)
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    dims = tuple(2 * q + e + 6 for e, q in zip(b, w))
    print("[gpu-case] per-axis filter zero keys", b, w, dims, flush=True)
    sys.stdout.flush()
    ref, flt = level_pair(dims, sum(b))
    rng = np.random.default_rng(4)
    h = [(e - 1) // 2 for e in b]
    c = np.array([[int(rng.integers(k, d - k)) for k, d in zip(h, dims)] for _ in range(40)],
                 dtype=np.int32)
    r, f, c = to_dev(ref), to_dev(flt), torch.from_numpy(c).cuda()
    got = [to_host(t) for t in nrr.block_match_aniso(r, f, c, b, w)]
    monkeypatch.setenv("NRR_ANISO_TILE", "8")
    want = [to_host(t) for t in nrr.block_match_aniso(r, f, c, b, w)]
    for a, e, name in zip(got, want, ("disp", "ncc", "conf")):
        assert np.array_equal(a.view(np.int32), e.view(np.int32)), (b, w, name)


@pytest.mark.parametrize("dtype", ["u16", "f32"])
@pytest.mark.parametrize("noise", [0.0, 0.005, 0.02])
@pytest.mark.parametrize("b,w", [((7, 7, 3), (10, 10, 4)), ((5, 7, 3), (8, 12, 5)),
                                 ((5, 7, 5), (12, 4, 6)), ((9, 9, 5), (7, 9, 4)),
                                 ((7, 9, 7), (7, 9, 4)), ((9, 5, 9), (9, 8, 5))])
def test_broad_peaks(monkeypatch, b, w, noise, dtype):
    """Smooth blobs: many displacements within the filter's bound, ranked in
    turns, around the peak, one by one or by the FMA form."""
    import torch

    for v in ("NRR_ANISO_ARITH", "NRR_ANISO_TILE", "NRR_ANISO_CZ"):
        monkeypatch.delenv(v, raising=False)
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    print("[gpu-case] per-axis filter broad peaks", b, w, noise, dtype, flush=True)
    sys.stdout.flush()
    p = synth.gen_translation_f32(seed=sum(b) + sum(w), n=48, n_blobs=17, noise=noise)
    ref, flt = p.ref, p.flt
    if dtype == "u16":
        lo, hi = min(ref.min(), flt.min()), max(ref.max(), flt.max())
        ref, flt = [np.round((v - lo) * (4095 / (hi - lo))).astype(np.uint16) for v in (ref, flt)]
    rng = np.random.default_rng(5)
    h = [(e - 1) // 2 for e in b]
    c = np.array([[int(rng.integers(k, 48 - k)) for k in h] for _ in range(60)], dtype=np.int32)
    r, f, c = to_dev(ref), to_dev(flt), torch.from_numpy(c).cuda()
    got = [to_host(t) for t in nrr.block_match_aniso(r, f, c, b, w)]
    monkeypatch.setenv("NRR_ANISO_TILE", "8")
    want = [to_host(t) for t in nrr.block_match_aniso(r, f, c, b, w)]
    for a, e, name in zip(got, want, ("disp", "ncc", "conf")):
        assert np.array_equal(a.view(np.int32), e.view(np.int32)), (b, w, name)
