"""Layers whose planes are cut into overlapping tiles (no flag names this route; tests/test_tiles_host.py says that these
layers take it), against the oracle, against whole planes, and in turns against all at once."""
import numpy as np
import pytest
import torch

from paper_1606_05688_amd import binding as B

pytestmark = pytest.mark.gpu

# With few products each, every kernel of the route (the host test counts them)
CASES = [(1, 33, 1, (5, 159, 121), (5, 1, 1)), (3, 1, 1, (54, 74, 150), (1, 2, 2)),
         (3, 2, 1, (36, 89, 155), (1, 2, 2)), (2, 2, 33, (49, 31, 67), (1, 1, 1)),
         (1, 1, 43, (9, 100, 156), (1, 2, 2)), (3, 1, 11, (65, 126, 61), (1, 2, 2)),
         (3, 1, 3, (48, 138, 88), (1, 3, 1)), (3, 28, 1, (6, 73, 122), (1, 2, 2)),
         (3, 2, 1, (64, 104, 165), (1, 2, 2)), (3, 2, 2, (72, 120, 139), (3, 5, 3)),
         (3, 2, 10, (50, 161, 79), (2, 4, 4)), (3, 5, 1, (29, 63, 163), (2, 1, 1)),
         (1, 2, 72, (37, 42, 58), (1, 1, 1)), (1, 1, 28, (6, 179, 172), (1, 3, 1)),
         (1, 1, 17, (23, 158, 128), (1, 1, 2)), (1, 2, 41, (29, 124, 61), (1, 1, 1)),
         (2, 2, 23, (53, 73, 57), (1, 1, 1)), (1, 1, 76, (34, 58, 75), (2, 1, 1)),
         (2, 1, 56, (18, 38, 146), (1, 2, 1)), (1, 1, 25, (36, 105, 68), (1, 1, 4)),
         (1, 1, 24, (70, 33, 158), (1, 3, 1)), (1, 1, 61, (9, 153, 160), (1, 1, 2)),
         (1, 5, 52, (37, 49, 61), (1, 1, 1)), (1, 1, 36, (35, 109, 60), (1, 2, 2))]
# Long sums, wide kernels, odd numbers of tiles, extents of one tile along y or z, chunks of input images that end short
CASES += [(1, 21, 19, (40, 97, 97), (3, 3, 3)), (2, 33, 7, (35, 101, 70), (5, 4, 7)), (1, 50, 18, (21, 130, 75), (7, 2, 3)),
          (1, 18, 70, (30, 67, 120), (2, 6, 5)), (1, 17, 17, (11, 200, 201), (4, 9, 8)), (3, 20, 20, (26, 80, 40), (3, 3, 5))]


def rand(seed, S, f, fo, n, k):
    r = np.random.default_rng(seed)
    inp = r.uniform(-1, 1, (S, f) + tuple(n)).astype(np.float32)
    w = (r.standard_normal((fo, f) + tuple(k)) * (f * np.prod(k)) ** -0.5).astype(np.float32)
    return inp, w, r.standard_normal(fo).astype(np.float32)


def _id(c):
    return "S%d_f%dx%d_n%s_k%s" % (c[0], c[1], c[2], "x".join(map(str, c[3])), "x".join(map(str, c[4])))


@pytest.mark.parametrize("case", CASES, ids=_id)
def test_tiles_match_oracle(oracle, case):
    S, f, fo, n, k = case
    inp, w, b = rand(S + f + fo, S, f, fo, n, k)
    print(f"[tiles] {case}", flush=True)
    d = torch.device("cuda:0")
    ti, tw, tb = (torch.from_numpy(t).to(d) for t in (inp, w, b))
    ws = B.alloc_workspace(S, f, fo, n, k)
    ws.fill_(0xFF)                                           # NaN patterns: nothing may be read before it is written
    got = B.znni_conv3d_fft(ti, tw, tb, relu=True, workspace=ws)
    whole = B.znni_conv3d_fft(ti, tw, tb, relu=True, mac_reference="xdirect")
    torch.cuda.synchronize()
    got, whole = (t.cpu().numpy().astype(np.float64) for t in (got, whole))
    exp = oracle.conv3d(inp, w, b, relu=True)
    tol = oracle.tolerance(inp, w)[None, :, None, None, None]
    assert np.all(np.abs(got - exp) <= tol)
    # 32-bit transforms and sums are 1e-7 to 6e-7 off
    assert np.linalg.norm(got - exp) <= 1e-6 * np.linalg.norm(exp)
    assert np.linalg.norm(got - whole) <= 1.5e-6 * np.linalg.norm(exp)


# no bias and no transfer function; shares at which inputs take turns, and pairs of one input
@pytest.mark.parametrize("case,share", [((1, 24, 20, (40, 130, 128), (3, 3, 3)), 0.5), ((3, 20, 18, (30, 96, 90), (3, 4, 2)), 0.6),
                                        ((1, 40, 40, (33, 150, 150), (5, 3, 3)), 0.3)], ids=str)
def test_turns_equal_all_at_once(case, share):
    S, f, fo, n, k = case
    d = torch.device("cuda:0")
    ti, tw, _ = (torch.from_numpy(t).to(d) for t in rand(7, S, f, fo, n, k))
    size = int(B.znni_conv3d_fft_workspace(S, f, fo, n, k) * share)
    ws = torch.full((size + 4096,), 0xFF, dtype=torch.uint8, device=d)       # NaN patterns, and a guard behind the budget
    got = B.znni_conv3d_fft_budget(ti, tw, None, workspace=ws[:size])
    whole = B.znni_conv3d_fft(ti, tw, None)
    torch.cuda.synchronize()
    assert torch.equal(got, whole)
    assert bool((ws[size:] == 0xFF).all())


# The whole layer's tiles leave no room for a pair: tiles of another length (tests/test_tiles_host.py says so), other roundings
OTHER_LENGTH = [((1, 84, 2, (67, 70, 66), (1, 2, 1)), 0.22), ((1, 67, 9, (46, 111, 106), (2, 2, 2)), 0.22),
                ((1, 16, 14, (70, 157, 82), (1, 5, 3)), 0.75)]


@pytest.mark.parametrize("case,share", OTHER_LENGTH, ids=str)
def test_turns_of_another_length(oracle, case, share):
    S, f, fo, n, k = case
    d = torch.device("cuda:0")
    inp, w, b = rand(8, S, f, fo, n, k)
    ti, tw, tb = (torch.from_numpy(t).to(d) for t in (inp, w, b))
    size = int(B.znni_conv3d_fft_workspace(S, f, fo, n, k) * share)
    ws = torch.full((size + 4096,), 0xFF, dtype=torch.uint8, device=d)
    got = B.znni_conv3d_fft_budget(ti, tw, tb, relu=True, workspace=ws[:size])
    torch.cuda.synchronize()
    assert bool((ws[size:] == 0xFF).all())
    got, exp = got.cpu().numpy().astype(np.float64), oracle.conv3d(inp, w, b, relu=True)
    assert np.all(np.abs(got - exp) <= oracle.tolerance(inp, w)[None, :, None, None, None])
    assert np.linalg.norm(got - exp) <= 1e-6 * np.linalg.norm(exp)


def test_kept_kernel_transforms_and_replays():
    S, f, fo, n, k = 2, 20, 18, (30, 96, 90), (3, 4, 2)
    d = torch.device("cuda:0")
    inp, w, b = rand(1, S, f, fo, n, k)
    ti, tw, tb = (torch.from_numpy(t).to(d) for t in (inp, w, b))
    ws = B.alloc_workspace(S, f, fo, n, k)
    B.znni_conv3d_fft(ti, tw, tb, workspace=ws)
    ti.copy_(torch.from_numpy(rand(2, S, f, fo, n, k)[0]))
    want = B.znni_conv3d_fft(ti, tw, tb)
    out = torch.empty_like(want)
    assert torch.equal(B.znni_conv3d_fft(ti, tw, tb, workspace=ws, out=out, keep_kernels=True), want)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            B.znni_conv3d_fft(ti, tw, tb, workspace=ws, out=out)
    torch.cuda.current_stream().wait_stream(s)
    for _ in range(3):
        out.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        ti.mul_(-0.5)
        want = B.znni_conv3d_fft(ti, tw, tb)


# kernels that make up for their images' magnitudes, and one output image without the large ones
@pytest.mark.parametrize("kind", ["moved", "one"])
def test_images_of_other_magnitudes(oracle, kind):
    S, f, fo, n, k = 1, 20, 18, (20, 90, 100), (3, 3, 3)
    inp, w, _ = rand(3, S, f, fo, n, k)
    e = np.arange(f) % 7 * 6 - 18
    x, v = inp * np.exp2(e)[None, :, None, None, None].astype(np.float32), w.copy()
    if kind == "moved":
        v *= np.exp2(-e)[None, :, None, None, None].astype(np.float32)
    else:
        v[5, e > -18] = 0
    d = torch.device("cuda:0")
    got = B.znni_conv3d_fft(torch.from_numpy(x).to(d), torch.from_numpy(v).to(d), None).cpu().numpy().astype(np.float64)
    exp = oracle.conv3d(x, v, None, relu=False)
    for j in range(fo):
        assert np.linalg.norm(got[:, j] - exp[:, j]) <= 1e-6 * np.linalg.norm(exp[:, j]), j


@pytest.mark.parametrize("value", [1e6, 1e11, float("nan"), float("inf")])
def test_a_large_value_stays_near_its_x_and_in_its_input(value):
    S, f, fo, n, k = 2, 20, 18, (36, 96, 90), (3, 4, 2)
    d = torch.device("cuda:0")
    inp, w, _ = rand(5, S, f, fo, n, k)
    tw = torch.from_numpy(w).to(d)
    clean = B.znni_conv3d_fft(torch.from_numpy(inp).to(d), tw, None).cpu().numpy()
    x = 17
    inp[1, 3, x, 40, 50] = value
    got = B.znni_conv3d_fft(torch.from_numpy(inp).to(d), tw, None).cpu().numpy()
    keep = [q for q in range(n[0] - k[0] + 1) if not x - k[0] < q <= x]
    tol = 1.5e-6 * np.linalg.norm(clean[1][:, keep]) / np.sqrt(clean[1][:, keep].size)
    assert np.sqrt(np.mean((got[1][:, keep] - clean[1][:, keep]) ** 2)) <= tol
    assert np.sqrt(np.mean((got[0] - clean[0]) ** 2)) <= tol
