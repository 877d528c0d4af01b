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
