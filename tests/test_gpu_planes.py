"""Small images that go untransformed along x, four planes at a time (no flag names this route: it is taken for batches of
lengths up to 64 and for small layers), against the oracle, and divided against whole."""
import numpy as np
import pytest
import torch

from paper_1606_05688_amd import binding as B

pytestmark = pytest.mark.gpu


def _rand(seed, S, f, fo, n, k):
    r = np.random.default_rng(seed)
    inp = r.uniform(-1, 1, (S, f) + tuple(n)).astype(np.float32)
    w = (r.standard_normal((fo, f) + tuple(k)) * (f * np.prod(k)) ** -0.5).astype(np.float32)
    return inp, w, r.standard_normal(fo).astype(np.float32)


def _is_planes(S, f, fo, n, k):
    """One kernel per side transforms z and y, and nothing transforms x."""
    nb, _ = B.znni_conv3d_fft_stage_work(S, f, fo, n, k)
    return nb["fwd_x"] == 0 and nb["fwd_y"] == 0 and nb["inv_z"] == 0


# Every length up to 64, at it and below it (planes together); last blocks of one to four planes on both sides; y and z of different extents
CASES = [(8, 2, 3, (8, 8, 7), (2, 3, 2)), (9, 3, 17, (13, 10, 9), (3, 2, 4)), (8, 5, 2, (12, 12, 11), (2, 2, 1)),
         (10, 17, 5, (15, 13, 14), (4, 3, 3)), (8, 4, 33, (18, 16, 16), (1, 5, 2)), (17, 3, 4, (20, 19, 20), (3, 1, 3)),
         (8, 33, 6, (25, 24, 23), (2, 3, 5)), (11, 2, 5, (27, 28, 26), (4, 4, 4)), (8, 6, 49, (34, 32, 31), (5, 3, 2)),
         (8, 1, 2, (9, 33, 36), (2, 2, 2)), (12, 4, 3, (41, 40, 39), (3, 6, 3)), (8, 20, 20, (22, 47, 48), (5, 5, 5)),
         # y lengths from 8 to 64 as single inputs and as batches
         (1, 3, 2, (35, 36, 35), (3, 2, 2)), (1, 1, 1, (19, 39, 40), (9, 1, 2)), (2, 5, 3, (51, 56, 53), (4, 4, 4)),
         (16, 16, 4, (20, 18, 20), (2, 3, 2)), (40, 8, 40, (17, 24, 22), (3, 3, 3)), (40, 8, 8, (28, 35, 36), (3, 2, 5)),
         (1, 1, 1, (7, 8, 8), (1, 1, 1)), (1, 2, 3, (16, 16, 16), (3, 3, 3)), (1, 70, 90, (9, 9, 10), (9, 9, 9)),
         (8, 3, 8, (51, 51, 51), (5, 5, 5)), (9, 5, 4, (30, 64, 63), (6, 7, 7)), (8, 3, 2, (66, 61, 64), (4, 3, 9))]
# Four planes one after the other (where they are many) at every length that has it, forward and inverse, and every pair of
# row and column tiles of the multiply-accumulate: with CASES all kernels of the route (tests/test_planes_host.py counts them)
CASES += [(5, 17, 13, (66, 27, 27), (2, 2, 2)), (9, 17, 17, (43, 40, 40), (2, 2, 2)), (9, 9, 17, (50, 56, 56), (2, 2, 2)),
          (1, 20, 66, (7, 23, 23), (7, 2, 2)), (5, 17, 17, (70, 16, 16), (2, 2, 2)), (3, 17, 79, (18, 20, 19), (2, 2, 2)),
          (12, 20, 49, (7, 47, 47), (2, 2, 2)), (17, 17, 33, (41, 7, 7), (2, 2, 2)), (12, 17, 49, (39, 10, 9), (2, 2, 2)),
          (24, 17, 33, (53, 7, 7), (2, 2, 2)), (3, 17, 33, (67, 19, 19), (2, 2, 2)), (12, 17, 66, (35, 9, 10), (2, 2, 2))]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "S%d_f%dx%d_n%s_k%s" % (c[0], c[1], c[2], "x".join(map(str, c[3])), "x".join(map(str, c[4]))))
def test_planes_match_oracle(oracle, case):
    S, f, fo, n, k = case
    assert _is_planes(S, f, fo, n, k)
    inp, w, b = _rand(S + f + fo, S, f, fo, n, k)
    print(f"[planes] {case}", flush=True)
    d = torch.device("cuda:0")
    ws = B.alloc_workspace(S, f, fo, n, k)
    ws.fill_(0xFF)                                           # NaN patterns: nothing may be read before it is written
    got = B.znni_conv3d_fft(*(torch.from_numpy(t).to(d) for t in (inp, w, b)), relu=True, workspace=ws)
    torch.cuda.synchronize()
    got = got.cpu().numpy().astype(np.float64)
    exp = oracle.conv3d(inp, w, b, relu=True)
    assert np.all(np.abs(got - exp) <= oracle.tolerance(inp, w)[None, :, None, None, None])
    assert np.linalg.norm(got - exp) <= 1e-6 * np.linalg.norm(exp)


def test_images_of_other_magnitudes(oracle):
    """Kernels that make up for their images' magnitudes: the powers of two that the forward kernel applies."""
    S, f, fo, n, k = 8, 12, 10, (20, 24, 24), (3, 3, 3)
    assert _is_planes(S, f, fo, n, k)
    inp, w, b = _rand(3, S, f, fo, n, k)
    e = np.array([0, 12, -15, 18, -18, 3, 0, 9, -9, 16, -4, 1])
    x, v = inp * np.exp2(e)[None, :, None, None, None].astype(np.float32), w * np.exp2(-e)[None, :, None, None, None].astype(np.float32)
    d = torch.device("cuda:0")
    got = B.znni_conv3d_fft(*(torch.from_numpy(t).to(d) for t in (x, v, b)))
    torch.cuda.synchronize()
    exp = oracle.conv3d(inp, w, b, relu=False)
    err = np.linalg.norm(got.cpu().numpy() - exp) / np.linalg.norm(exp)
    print(f"[planes] magnitudes apart: {err:.2e}", flush=True)
    assert err <= 1e-6


# share of the workspace: sub-batches of eight inputs and more; and so wide a bank that it goes through the halved axis in
# slabs, with the whole layer's result
@pytest.mark.parametrize("S,f,fo,n,k,share", [(20, 4, 5, (30, 32, 32), (3, 3, 3), 0.6), (8, 96, 96, (20, 48, 48), (3, 3, 3), 0.9)])
def test_divided_is_whole(S, f, fo, n, k, share):
    assert _is_planes(S, f, fo, n, k)
    d = torch.device("cuda:0")
    ti, tw, tb = (torch.from_numpy(t).to(d) for t in _rand(7, S, f, fo, n, k))
    ws = torch.empty(int(B.znni_conv3d_fft_workspace(S, f, fo, n, k) * share), dtype=torch.uint8, device=d)
    ws.fill_(0xFF)
    sub, _ = B.znni_conv3d_fft_sublayers(S, f, fo, n, k, ws.numel())
    assert sub != (S, f, fo)
    print(f"[planes] divided {sub}", flush=True)
    got = B.znni_conv3d_fft_budget(ti, tw, tb, relu=True, workspace=ws)
    whole = B.znni_conv3d_fft(ti, tw, tb, relu=True)
    torch.cuda.synchronize()
    assert torch.equal(got, whole)


def test_kept_kernel_transforms(oracle):
    S, f, fo, n, k = 9, 7, 6, (22, 28, 28), (4, 3, 2)
    assert _is_planes(S, f, fo, n, k)
    d = torch.device("cuda:0")
    inp, w, b = _rand(1, S, f, fo, n, k)
    tw, tb = torch.from_numpy(w).to(d), torch.from_numpy(b).to(d)
    ws = B.alloc_workspace(S, f, fo, n, k)
    B.znni_conv3d_fft(torch.from_numpy(inp).to(d), tw, tb, workspace=ws)
    other = torch.from_numpy(_rand(2, S, f, fo, n, k)[0]).to(d)
    kept = B.znni_conv3d_fft(other, tw, tb, workspace=ws, keep_kernels=True).clone()
    assert torch.equal(kept, B.znni_conv3d_fft(other, tw, tb))
