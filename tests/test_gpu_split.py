"""Multiply-accumulate of the untransformed-x route on fp16 matrix instructions (values split in two halves): edges of its
tiles and chunks, its power-of-two scales, and values that are not finite."""
import sys

import numpy as np
import pytest
import torch

from paper_1606_05688_amd import binding as B

pytestmark = pytest.mark.gpu


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def _rand(seed, S, f, fo, n, k):
    r = np.random.default_rng(seed)
    inp = r.uniform(-1, 1, (S, f) + tuple(n)).astype(np.float32)
    w = (r.standard_normal((fo, f) + tuple(k)) * (f * k[0] * k[1] * k[2]) ** -0.5).astype(np.float32)
    return inp, w


def _run(inp, w, route="xdirect"):
    d = torch.device("cuda:0")
    ti, tw = (t if isinstance(t, torch.Tensor) else torch.from_numpy(t) for t in (inp, w))
    out = B.znni_conv3d_fft(ti.to(d), tw.to(d), None, mac_reference=route)
    torch.cuda.synchronize()
    return out


# Row tiles 1 to 5 and two row blocks; outputs along x one below, at and above 64 per column tile and the widest tiles;
# input images below, at and above a quad, a group of sixteen and a chunk of thirty-two; slots that leave a step of four
# partly empty (quads x taps odd); several inputs.
EDGES = [(1, 1, 1, 1, 63), (1, 3, 16, 2, 64), (2, 4, 17, 3, 65), (1, 5, 33, 4, 128), (1, 15, 48, 5, 129),
         (1, 16, 49, 6, 192), (1, 17, 64, 7, 193), (3, 31, 65, 8, 20), (1, 33, 80, 9, 127), (1, 32, 81, 1, 130),
         (1, 7, 32, 3, 257), (1, 9, 16, 9, 255), (1, 35, 160, 2, 33), (1, 12, 5, 1, 16)]


@pytest.mark.parametrize("case", EDGES, ids=lambda c: "S%d_f%dx%d_kx%d_nox%d" % c)
def test_tile_and_chunk_edges_match_oracle(oracle, case):
    S, f, fo, kx, nox = case
    n, k = (nox + kx - 1, 9, 8), (kx, 2, 3)
    inp, w = _rand(sum(case), S, f, fo, n, k)
    _say(f"[split] {case}")
    got = _run(inp, w).cpu().numpy().astype(np.float64)
    exp = oracle.conv3d(inp, w, None, relu=False)
    assert np.all(np.abs(got - exp) <= oracle.tolerance(inp, w)[None, :, None, None, None])
    # 32-bit accuracy, not only the layer's bar: the fp32 route is 2e-7 to 7e-7 off on such layers
    assert np.linalg.norm(got - exp) <= 1e-6 * np.linalg.norm(exp)


def test_powers_of_two_pass_through_exactly():
    """Every scale is a power of two and sums stay fp32, so scaling the images or the kernels by one scales the result
    by it bit for bit."""
    inp, w = _rand(5, 1, 20, 20, (70, 10, 8), (3, 2, 3))
    base = _run(inp, w)
    for ei, ew in ((40, 0), (-60, 0), (0, 30), (0, -50), (-30, 45)):
        got = _run(np.ldexp(inp, ei), np.ldexp(w, ew))
        assert torch.equal(got, torch.ldexp(base, torch.tensor(ei + ew, device=base.device))), (ei, ew)
    assert not _run(np.zeros_like(inp), w).any() and not _run(inp, np.zeros_like(w)).any()


@pytest.mark.parametrize("late", [20, -20])
def test_chunks_of_different_magnitude(oracle, late):
    """Images of later chunks 2^20 larger (the sums are rescaled) or smaller than those of the first, output images whose
    kernels differ as much."""
    inp, w = _rand(6, 1, 40, 24, (75, 10, 8), (3, 2, 3))
    inp[:, 16:] = np.ldexp(inp[:, 16:], late)
    w[::2] = np.ldexp(w[::2], -late)
    got = _run(inp, w).cpu().numpy().astype(np.float64)
    exp = oracle.conv3d(inp, w, None, relu=False)
    for j in range(24):
        assert np.linalg.norm(got[:, j] - exp[:, j]) <= 1e-6 * np.linalg.norm(exp[:, j]), j


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -float("inf")])
def test_values_that_are_not_finite_stay_in_their_windows(bad):
    """The x axis is not transformed: a value that is not finite reaches the outputs whose taps meet its x, no others."""
    inp, w = _rand(7, 1, 18, 20, (70, 10, 8), (4, 2, 3))
    clean = _run(inp, w)
    inp[0, 17, 30, 4, 5] = bad
    got = _run(inp, w)
    hit = slice(30 - 3, 30 + 1)
    assert not torch.isfinite(got[:, :, hit]).any()
    keep = [x for x in range(67) if not 27 <= x <= 30]
    assert torch.allclose(got[:, :, keep], clean[:, :, keep], rtol=0, atol=1e-6 * float(clean.abs().max()))


@pytest.mark.parametrize("shape", [(40, 24, (75, 10, 8), (3, 2, 3)), (18, 80, (70, 12, 8), (7, 3, 2)), (5, 33, (140, 12, 8), (4, 10, 2))])
@pytest.mark.parametrize("far", [10, 17, 24, 30, 40])
def test_input_images_of_unequal_magnitude(oracle, shape, far):
    """Input images up to 2^far apart whose kernels make up for it, as in a network that is not normalised, and images
    whose kernels are that much smaller without it: every output image to 32-bit accuracy."""
    f, fo, n, k = shape
    inp, w = _rand(20, 1, f, fo, n, k)
    e = np.random.default_rng(21).integers(0, far + 1, f)
    e[:2] = 0, far
    for images in (True, False):
        x = np.ldexp(inp, e[:, None, None, None]) if images else inp
        v = np.ldexp(w, -e[:, None, None, None])
        got = _run(x, v).cpu().numpy().astype(np.float64)
        exp = oracle.conv3d(x, v, None, relu=False)
        for j in range(fo):
            assert np.linalg.norm(got[:, j] - exp[:, j]) <= 1e-6 * np.linalg.norm(exp[:, j]), (images, j)


@pytest.mark.parametrize("shape", [(18, 20, (70, 10, 8), (4, 2, 3)), (40, 80, (150, 12, 8), (7, 3, 2)), (3, 5, (300, 9, 8), (1, 2, 2)),
                                   (35, 64, (40, 10, 8), (5, 3, 2))])
@pytest.mark.parametrize("big", [1e6, 1e9, 1e13])
def test_a_large_value_stays_near_its_x(oracle, shape, big):
    """The x axis is not transformed: outputs whose taps do not meet the x of a large value keep 32-bit accuracy."""
    f, fo, n, k = shape
    inp, w = _rand(22, 1, f, fo, n, k)
    inp[0, f // 2, 25, 4, 5] = big
    got = _run(inp, w).cpu().numpy().astype(np.float64)
    exp = oracle.conv3d(inp, w, None, relu=False)
    for x in range(n[0] - k[0] + 1):
        assert np.linalg.norm(got[:, :, x] - exp[:, :, x]) <= 1e-6 * np.linalg.norm(exp[:, :, x]), x


def test_scales_whose_product_is_in_range(oracle):
    """Images and kernels near either end of the exponent range whose products are ordinary numbers."""
    inp, w = _rand(23, 1, 20, 20, (70, 10, 8), (3, 2, 3))
    for ei, ew in ((118, -100), (110, -60), (-100, 100), (-90, 60)):
        x, v = np.ldexp(inp, ei), np.ldexp(w, ew)
        got = _run(x, v).cpu().numpy().astype(np.float64)
        exp = oracle.conv3d(x, v, None, relu=False)
        assert np.linalg.norm(got - exp) <= 1e-6 * np.linalg.norm(exp), (ei, ew)


def test_kept_kernels_keep_the_scales_of_their_input_images(oracle):
    S, f, fo, n, k = 1, 18, 20, (70, 10, 8), (3, 2, 3)
    inp, w = _rand(24, S, f, fo, n, k)
    e = np.arange(f) * 2
    w = np.ldexp(w, -e[:, None, None, None])
    d = torch.device("cuda:0")
    tw, ws = torch.from_numpy(w).to(d), B.alloc_workspace(S, f, fo, n, k)
    B.znni_conv3d_fft(torch.from_numpy(inp).to(d), tw, None, workspace=ws, mac_reference="xdirect")
    x = np.ldexp(_rand(25, S, f, fo, n, k)[0], e[:, None, None, None])
    got = B.znni_conv3d_fft(torch.from_numpy(x).to(d), tw, None, workspace=ws, mac_reference="xdirect", keep_kernels=True)
    assert torch.equal(got, _run(x, w))


@pytest.mark.parametrize("share,shape", [(0.55, (2, 24, 90, (70, 24, 20), (3, 2, 3))), (0.9, (1, 24, 33, (40, 128, 64), (4, 2, 3))),
                                         (0.2, (1, 40, 90, (70, 24, 20), (3, 2, 3)))])
def test_a_large_value_under_a_budget(oracle, share, shape):
    """Sub-batches, slabs along the halved axis and blocks of images whose products are added up, two row blocks of output
    images: workgroups that sum again in fp32 write where the others do."""
    S, f, fo, n, k = shape
    inp, w = _rand(26, S, f, fo, n, k)
    inp[S - 1, f // 2, 20, 4, 5] = 1e10
    d = torch.device("cuda:0")
    ti, tw = torch.from_numpy(inp).to(d), torch.from_numpy(w).to(d)
    ws = torch.full((int(share * B.znni_conv3d_fft_workspace(S, f, fo, n, k)),), 0xFF, dtype=torch.uint8, device=d)
    got = B.znni_conv3d_fft_budget(ti, tw, None, workspace=ws, mac_reference="xdirect").cpu().numpy().astype(np.float64)
    exp = oracle.conv3d(inp, w, None, relu=False)
    for x in range(n[0] - k[0] + 1):
        assert np.linalg.norm(got[:, :, x] - exp[:, :, x]) <= 1e-6 * np.linalg.norm(exp[:, :, x]), x


@pytest.mark.parametrize("share,shape", [(None, (3, 5, 20, (70, 10, 8), (3, 2, 3))), (0.55, (2, 24, 90, (70, 24, 20), (3, 2, 3))),
                                         (0.9, (1, 24, 33, (40, 128, 64), (4, 2, 3))),
                                         (0.2, (1, 40, 90, (70, 24, 20), (3, 2, 3)))])
def test_input_images_of_unequal_magnitude_in_batches_and_blocks(oracle, share, shape):
    """The forward y pass scales the image an input's own number names: several inputs, sub-batches, slabs, blocks of
    input images (each with scales of its own)."""
    S, f, fo, n, k = shape
    inp, w = _rand(27, S, f, fo, n, k)
    e = np.random.default_rng(28).integers(0, 31, f)
    e[:2] = 0, 30
    x, v = np.ldexp(inp, e[:, None, None, None]), np.ldexp(w, -e[:, None, None, None])
    if share is None:
        got = _run(x, v)
    else:
        d = torch.device("cuda:0")
        size = int(share * B.znni_conv3d_fft_workspace(S, f, fo, n, k))
        got = B.znni_conv3d_fft_budget(torch.from_numpy(x).to(d), torch.from_numpy(v).to(d), None, mac_reference="xdirect",
                                       workspace=torch.full((size,), 0xFF, dtype=torch.uint8, device=d))
    got = got.cpu().numpy().astype(np.float64)
    exp = oracle.conv3d(x, v, None, relu=False)
    for s in range(S):
        for j in range(fo):
            assert np.linalg.norm(got[s, j] - exp[s, j]) <= 1e-6 * np.linalg.norm(exp[s, j]), (s, j)
