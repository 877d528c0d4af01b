"""Small layers whose kernels' first stage runs beside the forward transforms (one launch for three; tests/test_planes_host.py's
route): bit for bit what the separate kernels give, which the profiled call still launches, and the oracle's values."""
import numpy as np
import pytest
import torch

from paper_1606_05688_amd import binding as B

pytestmark = pytest.mark.gpu

# Every length up to 64, at it and below it; last blocks of one to four planes; one image and more images than a workgroup has
# waves; banks of one value and of several turns; kernels of one tap along an axis; padded row and column tiles
CASES = [(1, 2, 3, (16, 16, 16), (3, 3, 3)), (1, 1, 1, (7, 8, 8), (1, 1, 1)), (2, 5, 3, (9, 10, 9), (2, 4, 3)), (1, 7, 17, (13, 12, 11), (4, 2, 2)),
         (3, 3, 2, (14, 13, 14), (1, 5, 2)), (1, 20, 5, (17, 19, 20), (2, 2, 3)), (1, 4, 33, (18, 24, 23), (3, 1, 2)), (7, 2, 2, (15, 28, 27), (2, 3, 1)),
         (1, 8, 8, (32, 32, 31), (5, 5, 5)), (1, 3, 50, (11, 36, 35), (3, 2, 2)), (1, 6, 2, (40, 40, 39), (7, 2, 2)), (2, 2, 4, (20, 47, 48), (2, 6, 3)),
         (1, 5, 5, (30, 56, 55), (3, 3, 3)), (1, 8, 8, (64, 64, 64), (5, 5, 5)), (1, 1, 70, (9, 63, 62), (2, 2, 7)), (1, 21, 1, (12, 16, 15), (9, 2, 2))]


def _rand(seed, S, f, fo, n, k):
    r = np.random.default_rng(seed)
    inp = r.uniform(-1, 1, (S, f) + tuple(n)).astype(np.float32)
    w = (r.standard_normal((fo, f) + tuple(k)) * (f * np.prod(k)) ** -0.5).astype(np.float32)
    return inp, w, r.standard_normal(fo).astype(np.float32)


# kernels as they come; input images' kernels of other magnitudes, which move to the images; kernels of zeros and of infinities
@pytest.mark.parametrize("kind", ["even", "moved", "zeros", "infinite"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "S%d_f%dx%d_n%s_k%s" % (c[0], c[1], c[2], "x".join(map(str, c[3])), "x".join(map(str, c[4]))))
def test_one_launch_equals_three(oracle, case, kind):
    S, f, fo, n, k = case
    inp, w, b = _rand(S + f + fo, S, f, fo, n, k)
    e = np.arange(f) % 5 * 8 - 16
    if kind == "moved":
        w *= np.exp2(e)[None, :, None, None, None].astype(np.float32)
        inp *= np.exp2(-e)[None, :, None, None, None].astype(np.float32)
    elif kind == "zeros":
        w[:, ::2] = 0
        w[fo // 2] = 0
    elif kind == "infinite":
        w[0, f - 1, 0, 0, 0] = np.inf
    d = torch.device("cuda:0")
    ti, tw, tb = (torch.from_numpy(t).to(d) for t in (inp, w, b))
    ws = B.alloc_workspace(S, f, fo, n, k)
    ws.fill_(0xFF)                                           # NaN patterns: nothing may be read before it is written
    got = B.znni_conv3d_fft(ti, tw, tb, relu=True, workspace=ws)
    kept = B.znni_conv3d_fft(ti, tw, tb, relu=True, workspace=ws, keep_kernels=True)
    want, _ = B.znni_conv3d_fft_profile(ti, tw, tb, relu=True)
    torch.cuda.synchronize()
    assert torch.equal(got.view(torch.int32), want.view(torch.int32))
    assert torch.equal(kept.view(torch.int32), want.view(torch.int32))
    if kind != "infinite":
        exp = oracle.conv3d(inp, w, b, relu=True)
        assert np.linalg.norm(got.cpu().numpy() - exp) <= 1e-6 * np.linalg.norm(exp)
