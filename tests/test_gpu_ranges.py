"""Values far apart in magnitude on the routes that multiply split halves: no route flag for layers that go four planes at a
time (Ny = Nz <= 64), "xdirect" for the others."""
import numpy as np
import pytest
import torch

from paper_1606_05688_amd import binding as B

pytestmark = pytest.mark.gpu


def _rand(seed, S, f, fo, n, k):
    r = np.random.default_rng(seed)
    inp = r.uniform(-1, 1, (S, f) + tuple(n)).astype(np.float32)
    return inp, (r.standard_normal((fo, f) + tuple(k)) * (f * np.prod(k)) ** -0.5).astype(np.float32)


def _run(inp, w, route):
    S, f, fo, n, k = inp.shape[0], inp.shape[1], w.shape[0], inp.shape[2:], w.shape[2:]
    nb, _ = B.znni_conv3d_fft_stage_work(S, f, fo, n, k, mac_reference=route)
    # planes: z and y in one kernel on either side; xdirect: one pass each; x untransformed on both
    assert nb["fwd_x"] == 0 and (nb["fwd_y"] == 0) == (nb["inv_z"] == 0) == (not route)
    print(f"[ranges] {S} x {f} -> {fo} of {tuple(n)}, {tuple(k)} {route or 'planes'}", flush=True)
    d = torch.device("cuda:0")
    out = B.znni_conv3d_fft(torch.from_numpy(inp).to(d), torch.from_numpy(w).to(d), None, mac_reference=route)
    torch.cuda.synchronize()
    return out.cpu().numpy().astype(np.float64)


# (S, f, fo, n, k), three chunks of sixteen input images; one row tile and several; rows along x of whole and of broken blocks
# of four; one by one and together
LAYERS = [(False, 8, 40, 20, (40, 24, 22), (3, 2, 3)), (False, 1, 40, 7, (42, 20, 19), (4, 2, 2)),
          (False, 8, 48, 70, (29, 39, 40), (2, 3, 2)), ("xdirect", 1, 40, 20, (75, 30, 45), (3, 2, 3)),
          ("xdirect", 2, 40, 10, (150, 12, 8), (7, 3, 2)), ("xdirect", 1, 36, 80, (60, 10, 8), (5, 3, 2))]


@pytest.mark.parametrize("layer", LAYERS, ids=lambda c: "%s_S%d_f%dx%d" % ((c[0] or "planes",) + c[1:4]))
@pytest.mark.parametrize("which", [0, 1, 2])
def test_images_that_are_zero_beyond_large_values(oracle, layer, which):
    """Sixteen images of 2^30 at the first x and of zeros behind, the others of ordinary values: outputs that meet none of
    the large values keep 32-bit accuracy, whichever chunk is the large one."""
    route, S, f, fo, n, k = layer
    inp, w = _rand(30 + which, S, f, fo, n, k)
    c = slice(16 * which, 16 * which + 16)
    inp[:, c, 4:] = 0
    inp[:, c, :4] = np.ldexp(inp[:, c, :4], 30)
    got, exp = _run(inp, w, route), oracle.conv3d(inp, w, None, relu=False)
    for x in range(n[0] - k[0] + 1):
        assert np.linalg.norm(got[:, :, x] - exp[:, :, x]) <= 1e-6 * np.linalg.norm(exp[:, :, x]), x


def _uneven(seed, layer, far, kind):
    """Images in two groups 2^far apart, and banks under which some output images are made of the small ones alone."""
    _, S, f, fo, n, k = layer
    inp, w = _rand(seed, S, f, fo, n, k)
    if kind == "groups":            # output images of either group, the other's kernels zero
        inp[:, 1::2] = np.ldexp(inp[:, 1::2], -far)
        w[::2, 1::2] = w[1::2, ::2] = 0
    elif kind == "one":             # one output image in which the large images have no part
        inp[:, 1::2] = np.ldexp(inp[:, 1::2], -far)
        w[fo // 2, ::2] = 0
    elif kind == "crossed":         # the other group's kernels as much smaller as its images are larger
        inp[:, 1::2] = np.ldexp(inp[:, 1::2], far)
        w[::2, 1::2], w[1::2, ::2] = np.ldexp(w[::2, 1::2], -far), np.ldexp(w[1::2, ::2], -far)
    else:                           # "silent": the images whose kernels are the large ones are zero
        inp[:, ::2] = 0
        w[fo // 3, 1::2] = np.ldexp(w[fo // 3, 1::2], -far)
    return inp, w


def _each_output_image(got, exp):
    for s in range(got.shape[0]):
        for j in range(got.shape[1]):
            assert np.linalg.norm(got[s, j] - exp[s, j]) <= 1e-6 * np.linalg.norm(exp[s, j]), (s, j)


@pytest.mark.parametrize("layer", LAYERS + [(False, 9, 32, 33, (19, 16, 15), (3, 3, 3)), ("xdirect", 1, 8, 5, (70, 12, 20), (2, 11, 2))],
                         ids=lambda c: "%s_S%d_f%dx%d" % ((c[0] or "planes",) + c[1:4]))
@pytest.mark.parametrize("kind", ["groups", "one", "crossed", "silent"])
@pytest.mark.parametrize("far", [13, 20, 30])
def test_uneven_kernels_keep_every_output_image(oracle, layer, kind, far):
    """What fp32 products give: an output image is as good as the images it is made of, however large the others are."""
    inp, w = _uneven(40, layer, far, kind)
    _each_output_image(_run(inp, w, layer[0]), oracle.conv3d(inp, w, None, relu=False))


@pytest.mark.parametrize("share,S,f,fo,n,k", [(0.6, 20, 6, 5, (30, 32, 32), (3, 3, 3)), (0.9, 8, 96, 64, (20, 48, 48), (3, 3, 3)),
                                              (0.3, 1, 70, 50, (24, 24, 24), (3, 3, 3))])
@pytest.mark.parametrize("kind", ["crossed", "silent"])
def test_uneven_kernels_under_a_budget(oracle, share, S, f, fo, n, k, kind):
    """Sub-batches, slabs and blocks of images: kernel transforms made again belong to their rows and images."""
    inp, w = _uneven(41, (False, S, f, fo, n, k), 24, kind)
    d = torch.device("cuda:0")
    ws = torch.full((int(share * B.znni_conv3d_fft_workspace(S, f, fo, n, k)),), 0xFF, dtype=torch.uint8, device=d)
    print(f"[ranges] {kind}, divided {B.znni_conv3d_fft_sublayers(S, f, fo, n, k, ws.numel())[0]}", flush=True)
    got = B.znni_conv3d_fft_budget(torch.from_numpy(inp).to(d), torch.from_numpy(w).to(d), None, workspace=ws)
    _each_output_image(got.cpu().numpy().astype(np.float64), oracle.conv3d(inp, w, None, relu=False))


@pytest.mark.parametrize("layer", LAYERS[:4], ids=lambda c: "%s_S%d_f%dx%d" % ((c[0] or "planes",) + c[1:4]))
def test_uneven_kernels_that_were_kept(oracle, layer):
    route, S, f, fo, n, k = layer
    inp, w = _uneven(42, layer, 24, "crossed")
    d = torch.device("cuda:0")
    tw, ws = torch.from_numpy(w).to(d), B.alloc_workspace(S, f, fo, n, k)
    B.znni_conv3d_fft(torch.from_numpy(_rand(43, S, f, fo, n, k)[0]).to(d), tw, None, workspace=ws, mac_reference=route)
    got = B.znni_conv3d_fft(torch.from_numpy(inp).to(d), tw, None, workspace=ws, mac_reference=route, keep_kernels=True)
    _each_output_image(got.cpu().numpy().astype(np.float64), oracle.conv3d(inp, w, None, relu=False))


# rows along x of 1 to 3 planes in the last block of four, one to five row tiles, one input and a batch, planes one by one too
PLANE_LAYERS = [(1, 18, 20, (41, 16, 15), (4, 2, 3)), (8, 40, 66, (30, 20, 20), (5, 3, 2)), (9, 3, 5, (39, 14, 14), (1, 2, 2)),
                (2, 20, 40, (47, 24, 23), (7, 3, 3)), (24, 12, 12, (18, 28, 28), (3, 2, 3)), (1, 70, 90, (33, 12, 12), (9, 2, 2))]


@pytest.mark.parametrize("layer", PLANE_LAYERS, ids=lambda c: "S%d_f%dx%d" % c[:3])
@pytest.mark.parametrize("big", [1e6, 1e9, 1e13])
def test_a_large_value_stays_near_its_x(oracle, layer, big):
    """The x axis is not transformed: outputs whose taps do not meet the x of a large value keep 32-bit accuracy."""
    S, f, fo, n, k = layer
    inp, w = _rand(50, S, f, fo, n, k)
    inp[S - 1, f // 2, n[0] // 2, 4, 5] = big
    got, exp = _run(inp, w, False), oracle.conv3d(inp, w, None, relu=False)
    for s in range(S):
        for x in range(n[0] - k[0] + 1):
            assert np.linalg.norm(got[s, :, x] - exp[s, :, x]) <= 1e-6 * np.linalg.norm(exp[s, :, x]), (s, x)


@pytest.mark.parametrize("layer", PLANE_LAYERS, ids=lambda c: "S%d_f%dx%d" % c[:3])
@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -float("inf")])
def test_values_that_are_not_finite_stay_in_their_windows(layer, bad):
    """A value that is not finite reaches the outputs of its input whose taps meet its x, no others."""
    S, f, fo, n, k = layer
    inp, w = _rand(51, S, f, fo, n, k)
    clean = _run(inp, w, False)
    x = n[0] // 2
    inp[S - 1, f - 1, x, 4, 5] = bad
    got = _run(inp, w, False)
    hit = range(max(0, x - k[0] + 1), min(x + 1, n[0] - k[0] + 1))
    assert not np.isfinite(got[S - 1][:, hit.start:hit.stop]).any()
    keep = [q for q in range(n[0] - k[0] + 1) if q not in hit]
    tol = 1e-6 * np.abs(clean).max()
    assert np.allclose(got[S - 1][:, keep], clean[S - 1][:, keep], rtol=0, atol=tol)
    assert np.allclose(got[:S - 1], clean[:S - 1], rtol=0, atol=tol)


@pytest.mark.parametrize("share,S,f,fo,n,k", [(0.6, 20, 6, 5, (30, 32, 32), (3, 3, 3)), (0.9, 8, 96, 64, (20, 48, 48), (3, 3, 3)),
                                              (0.3, 1, 70, 50, (26, 24, 24), (3, 3, 3))])
def test_a_large_value_under_a_budget(oracle, share, S, f, fo, n, k):
    """Sub-batches, slabs, and blocks of images whose products are added up: waves that sum again in fp32 write where the
    others do."""
    inp, w = _rand(52, S, f, fo, n, k)
    inp[S - 1, f // 2, 14, 4, 5] = 1e10
    d = torch.device("cuda:0")
    ws = torch.full((int(share * B.znni_conv3d_fft_workspace(S, f, fo, n, k)),), 0xFF, dtype=torch.uint8, device=d)
    sub = B.znni_conv3d_fft_sublayers(S, f, fo, n, k, ws.numel())[0]
    print(f"[ranges] large value, divided {sub}", flush=True)
    assert sub != (S, f, fo)
    got = B.znni_conv3d_fft_budget(torch.from_numpy(inp).to(d), torch.from_numpy(w).to(d), None, workspace=ws).cpu().numpy().astype(np.float64)
    exp = oracle.conv3d(inp, w, None, relu=False)
    for s in range(S):
        for x in range(n[0] - k[0] + 1):
            assert np.linalg.norm(got[s, :, x] - exp[s, :, x]) <= 1e-6 * np.linalg.norm(exp[s, :, x]), (s, x)
