"""GPU: selection with a candidate mask and a connectivity pattern, against
the oracle (bit-exact: same centres, same order)."""

import json
import os
import sys

import numpy as np
import pytest

import oracle
import paper_2308_10868_amd as nrr
from paper_2308_10868_amd import synth
from tests.gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu
HERE = os.path.dirname(os.path.abspath(__file__))


def say(*a):
    print("[gpu-case]", *a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def torch_dev():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    nrr.load()
    return torch


def gpu_ex(vol, b, s, f, mask, conn):
    import torch

    c = nrr.select_blocks_ex(to_dev(vol), b, s, f, None if mask is None else to_dev(mask), conn)
    torch.cuda.synchronize()
    return to_host(c)


@pytest.mark.parametrize("conn", [0, 6, 18, 26])
@pytest.mark.parametrize("dtype", ["u16", "f32"])
def test_tiny_random_with_masks(torch_dev, conn, dtype):
    for seed in range(3):
        p = synth.gen_random(30 + seed, (19, 15, 13), dtype, smooth=1.0)
        rng = np.random.default_rng(seed)
        mask = (rng.random(p.ref.shape) < 0.7).astype(np.uint8) if seed != 0 else None
        for b, s, f in [(3, 2, 0.4), (3, 1, 0.2), (5, 3, 0.9), (3, 3, 1.0)]:
            say("select_ex", dtype, conn, seed, b, s, f)
            want, _ = oracle.select_ex(p.ref, b, s, f, mask, conn)
            got = gpu_ex(p.ref, b, s, f, mask, conn)
            assert np.array_equal(got, want), (dtype, conn, seed, b, s, f)


def test_golden_cases(torch_dev):
    from tests.test_oracle_select_ex import golden_volume

    for case in json.load(open(os.path.join(HERE, "golden", "select_connectivity.json")))["cases"]:
        vol, mask = golden_volume(case)
        got = gpu_ex(vol, 3, 3, case["fraction"], mask, case["connectivity"])
        gx = case["dims"][0] // 3
        want = np.array([[3 * (g % gx) + 1, 3 * (g // gx) + 1, 1] for g in case["taken"]],
                        dtype=np.int32).reshape(-1, 3)
        assert np.array_equal(got, want), case["why"]


@pytest.mark.parametrize("conn", [6, 26])
def test_mri_workload_with_region_mask(torch_dev, conn):
    p = synth.gen_mri_u16(seed=0)
    nz, ny, nx = p.ref.shape
    z, y, x = np.mgrid[0:nz, 0:ny, 0:nx]
    # an ellipsoidal region (a stand-in for the intracranial cavity)
    mask = (((x - nx / 2) / (0.42 * nx)) ** 2 + ((y - ny / 2) / (0.45 * ny)) ** 2 +
            ((z - nz / 2) / (0.48 * nz)) ** 2 <= 1.0).astype(np.uint8)
    say("select_ex mri", conn)
    want, _ = oracle.select_ex(p.ref, 7, 7, 0.25, mask, conn)
    got = gpu_ex(p.ref, 7, 7, 0.25, mask, conn)
    assert len(want) > 300  # a nontrivial set (26-connectivity leaves about 800)
    assert np.array_equal(got, want)


def test_plain_special_case_equals_select_blocks(torch_dev):
    p = synth.gen_translation_f32(seed=0)
    a = to_host(nrr.select_blocks(to_dev(p.ref), 7, 7, 0.2))
    b = gpu_ex(p.ref, 7, 7, 0.2, None, 0)
    assert np.array_equal(a, b)


# Grids above 24,576 candidates take the round-launch path.
@pytest.mark.parametrize("conn", [0, 6, 18, 26])
@pytest.mark.parametrize("dtype", ["u16", "f32"])
def test_large_grids_every_pattern(torch_dev, conn, dtype):
    p = synth.gen_random(50, (66, 60, 52), dtype, smooth=1.5)  # b 3, stride 1: 184,800
    rng = np.random.default_rng(7)
    for mask in (None, (rng.random(p.ref.shape) < 0.8).astype(np.uint8)):
        for b, s, f in [(3, 1, 0.3), (5, 2, 0.9)]:
            say("select_ex large", dtype, conn, mask is not None, b, s, f)
            want, _ = oracle.select_ex(p.ref, b, s, f, mask, conn)
            got = gpu_ex(p.ref, b, s, f, mask, conn)
            assert np.array_equal(got, want), (dtype, conn, b, s, f)


def test_large_grid_with_long_decision_chains(torch_dev):
    """Block variance rising along x and y (a checkerboard of growing
    amplitude): every candidate's decision waits for its neighbour's, so the
    chains run across the whole grid and through many tiles."""
    nz, ny, nx = 12, 90, 300
    z, y, x = np.mgrid[0:nz, 0:ny, 0:nx]
    vol = (((x + y + z) % 2) * (10 * x + 3 * y + 1)).astype(np.uint16)
    vol = np.minimum(vol, 4095).astype(np.uint16)
    for conn in (6, 26):
        say("select_ex chains", conn)
        want, _ = oracle.select_ex(vol, 3, 1, 1.0, None, conn)
        got = gpu_ex(vol, 3, 1, 1.0, None, conn)
        assert len(want) > 1000
        assert np.array_equal(got, want), conn


@pytest.mark.parametrize("conn", [6, 26])
def test_dense_grid_with_region_mask(torch_dev, conn):
    """The dense 512x512x256 workload's grid (9^3 blocks, stride 5: 510,050
    candidates), a region mask and a pattern, against the oracle."""
    import time

    import torch

    p = synth.gen_blobs_u16(seed=0)
    nz, ny, nx = p.ref.shape
    z, y, x = np.ogrid[0:nz, 0:ny, 0:nx]
    mask = (((x - nx / 2) / (0.42 * nx)) ** 2 + ((y - ny / 2) / (0.45 * ny)) ** 2 +
            ((z - nz / 2) / (0.48 * nz)) ** 2 <= 1.0).astype(np.uint8)
    say("select_ex dense", conn)
    want, _ = oracle.select_ex(p.ref, 9, 5, 0.7, mask, conn)
    ref, md = to_dev(p.ref), to_dev(mask)
    nrr.select_blocks_ex(ref, 9, 5, 0.7, md, conn)  # warm-up
    torch.cuda.synchronize()
    t = time.perf_counter()
    c = nrr.select_blocks_ex(ref, 9, 5, 0.7, md, conn)
    torch.cuda.synchronize()
    say("select_ex dense %d: %d taken, %.2f ms" % (conn, len(c), (time.perf_counter() - t) * 1e3))
    assert len(want) > 10000  # 6: about 77,000; 26: about 19,000
    assert np.array_equal(to_host(c), want)


# Per-axis block edges and strides with the variants.
@pytest.mark.parametrize("conn", [0, 6, 18, 26])
@pytest.mark.parametrize("dtype", ["u16", "f32"])
def test_aniso_variants_small(torch_dev, conn, dtype):
    import torch

    p = synth.gen_random(60, (23, 19, 15), dtype, smooth=1.0)
    rng = np.random.default_rng(8)
    for mask in (None, (rng.random(p.ref.shape) < 0.7).astype(np.uint8)):
        for b, s, f in [((3, 5, 1), (2, 3, 1), 0.5), ((5, 3, 3), (1, 2, 3), 0.9),
                        ((1, 3, 5), (2, 1, 2), 0.3), ((7, 3, 3), (3, 3, 1), 1.0)]:
            say("select_aniso_ex", dtype, conn, mask is not None, b, s, f)
            want, _ = oracle.select_aniso_ex(p.ref, b, s, f, mask, conn)
            c = nrr.select_blocks_aniso_ex(to_dev(p.ref), b, s, f,
                                           None if mask is None else to_dev(mask), conn)
            torch.cuda.synchronize()
            assert np.array_equal(to_host(c), want), (dtype, conn, b, s, f)


@pytest.mark.parametrize("conn", [6, 26])
def test_aniso_variants_mri_slices(torch_dev, conn):
    """The MRI pair with blocks thinner along the slice axis (7 x 7 x 3,
    stride 7 x 7 x 3: 53,136 candidates, the round-launch path) inside an
    ellipsoidal region."""
    import torch

    p = synth.gen_mri_u16(seed=0)
    nz, ny, nx = p.ref.shape
    z, y, x = np.ogrid[0:nz, 0:ny, 0:nx]
    mask = (((x - nx / 2) / (0.42 * nx)) ** 2 + ((y - ny / 2) / (0.45 * ny)) ** 2 +
            ((z - nz / 2) / (0.48 * nz)) ** 2 <= 1.0).astype(np.uint8)
    say("select_aniso_ex mri", conn)
    want, _ = oracle.select_aniso_ex(p.ref, (7, 7, 3), (7, 7, 3), 0.25, mask, conn)
    c = nrr.select_blocks_aniso_ex(to_dev(p.ref), (7, 7, 3), (7, 7, 3), 0.25, to_dev(mask), conn)
    torch.cuda.synchronize()
    assert len(want) > 1000
    assert np.array_equal(to_host(c), want)


@pytest.mark.parametrize("dtype", ["u16", "f32"])
def test_plain_selection_large_grid_with_ties(torch_dev, dtype):
    """Grids above 32,768 candidates take the multi-workgroup radix select,
    smaller ones the one-workgroup select with its keys in registers: half
    the volume is flat, so thousands of candidates share the key 0 and the
    K-th key falls among them (ties to the lower grid index)."""
    import torch

    p = synth.gen_random(70, (120, 100, 90), dtype, smooth=1.0)
    ref = p.ref.copy()
    ref[:, :, :60] = ref[0, 0, 0]  # flat half
    for b, s, f in [(3, 2, 0.7), (5, 1, 0.55), (3, 1, 0.05), (15, 8, 0.3)]:
        say("plain selection large", dtype, b, s, f)
        want, _ = oracle.select(ref, b, s, f)
        got = nrr.select_blocks(to_dev(ref), b, s, f)
        torch.cuda.synchronize()
        assert np.array_equal(to_host(got), want), (dtype, b, s, f)
    small = ref[:64, :64, :64].copy()  # b 3, stride 2: 29,791 candidates (one workgroup)
    for f in (0.6, 0.999):
        want, _ = oracle.select(small, 3, 2, f)
        got = nrr.select_blocks(to_dev(small), 3, 2, f)
        torch.cuda.synchronize()
        assert np.array_equal(to_host(got), want), (dtype, "29,791", f)


# Edges above 15, which the variants take (the plain selection does not):
# overlapping by tiles and by a wavefront per candidate, and apart.
@pytest.mark.parametrize("dims,b,s", [
    ((75, 40, 33), 17, 8), ((90, 41, 34), 17, 17), ((90, 41, 34), 17, 19), ((70, 60, 45), 33, 5),
    ((101, 69, 40), 33, 12), ((140, 70, 66), 33, 33), ((100, 83, 70), 67, 3),
    ((110, 90, 69), 67, 9), ((140, 69, 68), 67, 71),
])
@pytest.mark.parametrize("dtype", ["u16", "f32"])
def test_edges_above_fifteen(torch_dev, dtype, dims, b, s):
    p = synth.gen_random(b + s, dims, dtype)
    rng = np.random.default_rng(b)
    for mask, conn in [(None, 0), ((rng.random(p.ref.shape) < 0.8).astype(np.uint8), 6)]:
        say("select_ex edges above 15", dtype, dims, b, s, conn)
        want, _ = oracle.select_ex(p.ref, b, s, 0.5, mask, conn)
        got = gpu_ex(p.ref, b, s, 0.5, mask, conn)
        assert np.array_equal(got, want), (dtype, dims, b, s, conn)


# Grids one workgroup serves also run in the plain selection's workspace: the
# masks of ranked-above neighbours are then made in that workgroup.
@pytest.mark.parametrize("conn", [0, 6, 26])
@pytest.mark.parametrize("dims", [(84, 84, 81), (60, 50, 43), (48, 46, 90), (51, 45, 30)])
@pytest.mark.parametrize("axes", [False, True])
def test_in_the_plain_workspace(torch_dev, dims, conn, axes):
    import ctypes

    torch, lib = torch_dev, nrr.load()
    b, s = (3, 3) if dims[0] == 84 else (3, 2) if dims[0] == 60 else (5, 3)
    p = synth.gen_random(sum(dims), dims, "u16", smooth=1.0)
    mask = (np.random.default_rng(2).random(p.ref.shape) < 0.85).astype(np.uint8)
    n = int(np.prod(nrr.grid_shape(dims, b, s)))
    assert n <= 24576

    def up(v):
        return (v + 255) // 256 * 256

    plain = up(8 * n) + 256 + up(16 * ((n + 2047) // 2048))
    say("select_ex in the plain workspace", dims, b, s, conn, axes, n)
    ws = torch.full((plain + 4096,), 171, dtype=torch.uint8, device="cuda")
    c = torch.zeros((n, 3), dtype=torch.int32, device="cuda")
    k = torch.zeros(1, dtype=torch.int64, device="cuda")
    vol, m = to_dev(p.ref), to_dev(mask)
    d3 = (ctypes.c_int32 * 3)(*dims)
    b3, s3 = (ctypes.c_int32 * 3)(b, b, b), (ctypes.c_int32 * 3)(s, s, s)

    def ptr(t):
        return ctypes.c_void_p(t.data_ptr())

    if axes:
        call = lambda size: lib.nrr_select_blocks_aniso_ex(
            ptr(vol), nrr.U16, d3, b3, s3, 0.6, ptr(m), conn, ptr(c), n, ptr(k), ptr(ws), size,
            None)
    else:
        call = lambda size: lib.nrr_select_blocks_ex(
            ptr(vol), nrr.U16, d3, b, s, 0.6, ptr(m), conn, ptr(c), n, ptr(k), ptr(ws), size, None)
    assert call(plain) == 0, lib.nrr_last_error()
    torch.cuda.synchronize()
    want, _ = oracle.select_ex(p.ref, b, s, 0.6, mask, conn)
    assert int(k.item()) == len(want) and np.array_equal(to_host(c)[: len(want)], want)
    assert bool((ws[plain:] == 171).all())  # nothing written past the size given
    assert call(plain - 1) == 2  # still refused below it


@pytest.mark.parametrize("dims,b,s", [((3, 3, 3), 3, 3), ((18, 18, 21), 3, 3),      # 1, 252
                                      ((33, 33, 27), 3, 3), ((48, 48, 48), 3, 3),   # 1089, 4096
                                      ((51, 51, 45), 3, 3), ((84, 84, 81), 3, 3)])  # 4335, 21168
@pytest.mark.parametrize("conn", [0, 6, 26])
def test_everything_taken_and_one_less(torch_dev, dims, b, s, conn):
    """The count reaches what the pattern takes, passes it, and stays one below."""
    p = synth.gen_random(sum(dims) + conn, dims, "u16", smooth=0.7)
    rng = np.random.default_rng(conn)
    mask = (rng.random(p.ref.shape) < 0.9).astype(np.uint8)
    full, _ = oracle.select_ex(p.ref, b, s, 1.0, mask, conn)
    h = b // 2
    n_in = int(mask[h::s, h::s, h::s][:dims[2] // s, :dims[1] // s, :dims[0] // s].sum())
    for k in {len(full) - 1, len(full), n_in} - {0, -1}:  # (a fraction is above 0)
        f = k / n_in
        say("select_ex all taken", dims, conn, k, n_in)
        want, _ = oracle.select_ex(p.ref, b, s, f, mask, conn)
        got = gpu_ex(p.ref, b, s, f, mask, conn)
        assert np.array_equal(got, want), (dims, conn, k)
