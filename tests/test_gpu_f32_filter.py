"""GPU: the float search behind the matrix-core filter against the FMA form.

The filter may only leave out displacements that cannot win, and re-ranks the
rest in the FMA form's own operations, so displacements, NCC and confidence
are the same bits as a pinned FMA shape's.  The inputs are those where a
bound or a fallback could go wrong: surfaces with many near-equal keys, exact
ties, flat blocks and windows, local levels far from the block's, magnitudes
near and past the limits of the scaling, and values that are not finite.
"""

import sys

import numpy as np
import pytest

import paper_2308_10868_amd as nrr
from paper_2308_10868_amd import synth
from tests.gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu


def volumes(kind, dims, seed):
    nx, ny, nz = dims
    rng = np.random.default_rng(seed)
    p = synth.gen_random(seed, dims, "f32", smooth=1.5)
    ref, flt = p.ref.copy(), p.flt.copy()
    if kind == "smooth":  # a shifted copy: broad peaks, many keys near the best
        base = synth.gen_random(seed, dims, "f32", smooth=4.0).ref
        ref, flt = base, np.roll(base, (1, -1, 2), (0, 1, 2)).astype(np.float32)
    elif kind == "noise":  # no true match: the best keys lie close together
        ref = rng.normal(size=(nz, ny, nx)).astype(np.float32)
        flt = rng.normal(size=(nz, ny, nx)).astype(np.float32)
    elif kind == "periodic":  # exact ties, the lowest shift index wins
        z, y, x = np.meshgrid(np.arange(nz), np.arange(ny), np.arange(nx), indexing="ij")
        ref = ((x % 4) + 2 * (y % 3) + 3 * (z % 2)).astype(np.float32)
        flt = ref.copy()
    elif kind == "flat":  # flat blocks, flat windows and a constant half
        ref[:, :, : nx // 2] = 0.25
        flt[:, : ny // 2] = 0.25
    elif kind == "levels":  # steps of the local level, each with little texture
        step = (np.arange(nx) // 7 % 3).astype(np.float32) * 1000.0
        ref, flt = (ref * 0.1 + step).astype(np.float32), (flt * 0.1 + step).astype(np.float32)
    elif kind == "decades":
        e = rng.integers(-4, 5, size=ref.shape)
        ref, flt = (ref * 10.0 ** e).astype(np.float32), (flt * 10.0 ** e).astype(np.float32)
    elif kind == "offset":  # a large common level: few bits left for the texture
        ref, flt = (ref + 30000.0).astype(np.float32), (flt + 30000.0).astype(np.float32)
    elif kind.startswith("scale"):
        s = np.float32(10.0) ** np.float32(int(kind[5:]))
        ref, flt = ref * s, flt * s
    elif kind == "bad":  # undefined results, but the same ones, and no fault
        flt.reshape(-1)[rng.integers(0, flt.size, 40)] = np.inf
        flt.reshape(-1)[rng.integers(0, flt.size, 40)] = np.nan
        ref.reshape(-1)[rng.integers(0, ref.size, 5)] = np.nan
    return np.ascontiguousarray(ref), np.ascontiguousarray(flt)


KINDS = ["random", "smooth", "noise", "periodic", "flat", "levels", "decades", "offset",
         "scale-25", "scale-17", "scale17", "scale25", "bad"]


@pytest.fixture(autouse=True)
def no_pins(monkeypatch):
    import torch

    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    for k in ("NRR_ARITH", "NRR_TILE", "NRR_CZ"):
        monkeypatch.delenv(k, raising=False)
    nrr.clear_tuning()
    yield
    nrr.clear_tuning()


def both(ref, flt, centers, b, w):
    import torch

    r, f, c = to_dev(ref), to_dev(flt), torch.from_numpy(centers).cuda()
    got = [to_host(t) for t in nrr.block_match(r, f, c, b, w)]
    shape = next(s for s in nrr.match_shapes(nrr.F32, b, w) if s["rx"] == 4)
    nrr.set_tuned_shape(nrr.F32, b, w, shape)
    want = [to_host(t) for t in nrr.block_match(r, f, c, b, w)]
    nrr.clear_tuning()
    return got, want


def centers_of(dims, b, seed, n=48):
    h = b // 2
    rng = np.random.default_rng(seed)
    lo, hi = [h] * 3, [d - 1 - h for d in dims]
    c = [[int(rng.integers(l, u + 1)) for l, u in zip(lo, hi)] for _ in range(n)]
    c += [lo, hi, [hi[0], lo[1], hi[2]], [lo[0], hi[1], lo[2]], [0, 0, 0],
          [dims[0] - 1, dims[1] // 2, dims[2] // 2]]  # the last two not inside
    return np.array(c, dtype=np.int32)


@pytest.mark.parametrize("b,w,dims", [(5, 4, (29, 26, 24)), (5, 8, (31, 29, 26)), (7, 5, (33, 30, 27)),
                                      (9, 6, (37, 34, 31))])
@pytest.mark.parametrize("kind", KINDS)
def test_same_bits_as_the_fma_form(kind, b, w, dims):
    print("[gpu-case] f32 filter", kind, b, w, dims, flush=True)
    sys.stdout.flush()
    ref, flt = volumes(kind, dims, 11 * b + w)
    got, want = both(ref, flt, centers_of(dims, b, b), b, w)
    for a, e, name in zip(got, want, ("disp", "ncc", "conf")):
        assert np.array_equal(a.view(np.int32), e.view(np.int32)), (kind, name)


# windows around and past the chunks a thread holds, one plane, and the sizes
# whose window no longer fits (the FMA form then serves by itself)
@pytest.mark.parametrize("b,w", [(5, 0), (5, 1), (5, 10), (5, 13), (5, 16), (7, 0), (7, 10),
                                 (7, 12), (7, 15), (9, 0), (9, 3), (9, 11), (9, 13)])
def test_window_sizes(b, w):
    dims = (2 * w + b + 3, 2 * w + b, 2 * w + b + 2)
    print("[gpu-case] f32 filter window", b, w, dims, flush=True)
    sys.stdout.flush()
    ref, flt = volumes("smooth", dims, 5 * b + w)
    got, want = both(ref, flt, centers_of(dims, b, w, 10), b, w)
    for a, e in zip(got, want):
        assert np.array_equal(a.view(np.int32), e.view(np.int32))


def level_pair(dims, seed, level=1e6, std=0.4):
    """Texture far below the common level: every record is flagged flat (its
    variance is below 1e-12 of its mean square), so every key is a zero, of
    either sign, and the lowest shift index wins."""
    rng = np.random.default_rng(seed)
    return [(level + std * rng.normal(size=dims[::-1])).astype(np.float32) for _ in range(2)]


@pytest.mark.parametrize("b,w", [(7, 1), (7, 2), (7, 3), (7, 6), (9, 4), (5, 7)])
def test_zero_keys_of_either_sign(b, w):
    dims = (2 * w + b + 8, 2 * w + b + 7, 2 * w + b + 5)
    print("[gpu-case] f32 filter zero keys", b, w, dims, flush=True)
    sys.stdout.flush()
    ref, flt = level_pair(dims, b + w)
    got, want = both(ref, flt, centers_of(dims, b, w), b, w)
    for a, e, name in zip(got, want, ("disp", "ncc", "conf")):
        assert np.array_equal(a.view(np.int32), e.view(np.int32)), (b, w, name)


@pytest.mark.parametrize("top", [56.0, 57.9, 58.5, 59.9, 60.4])
@pytest.mark.parametrize("b,w", [(7, 3), (9, 5)])
def test_sums_past_the_float_range(b, w, top):
    """Magnitudes whose FP32 cross terms overflow near a match: the FMA form's
    keys tie at infinity there."""
    dims = (2 * w + b + 8, 2 * w + b + 7, 2 * w + b + 5)
    print("[gpu-case] f32 filter large magnitudes", b, w, top, flush=True)
    sys.stdout.flush()
    base = synth.gen_random(b + w, dims, "f32", smooth=2.5).ref.astype(np.float64)
    base = np.tanh(4.0 * (base - base.mean()) / base.std())  # two levels, soft edges
    base = (base * 2.0 ** top).astype(np.float32)
    flt = np.ascontiguousarray(np.roll(base, (1, -1, 2), (0, 1, 2)))
    got, want = both(base, flt, centers_of(dims, b, w), b, w)
    for a, e, name in zip(got, want, ("disp", "ncc", "conf")):
        assert np.array_equal(a.view(np.int32), e.view(np.int32)), (b, w, top, name)


@pytest.mark.parametrize("noise", [0.0, 0.005, 0.02])
@pytest.mark.parametrize("b,w", [(5, 8), (5, 12), (7, 3), (7, 6), (7, 10), (9, 5), (9, 11)])
def test_broad_peaks(b, w, noise):
    """Smooth blobs: hundreds of displacements within the filter's bound, which
    are swept again, ranked around the peak, one by one or by the FMA form."""
    print("[gpu-case] f32 filter broad peaks", b, w, noise, flush=True)
    sys.stdout.flush()
    p = synth.gen_translation_f32(seed=b + w, n=48, n_blobs=17, noise=noise)
    got, want = both(p.ref, p.flt, centers_of((48, 48, 48), b, w), b, w)
    for a, e, name in zip(got, want, ("disp", "ncc", "conf")):
        assert np.array_equal(a.view(np.int32), e.view(np.int32)), (b, w, name)
