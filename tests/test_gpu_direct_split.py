"""Direct convolution of narrow layers on fp16 matrix instructions (values split in two halves): edges of its tiles and
slots, scales, values that are not finite."""
import numpy as np
import pytest
import torch

from paper_1606_05688_amd import binding as B

pytestmark = pytest.mark.gpu


def _rand(seed, S, f, fo, n, k):
    r = np.random.default_rng(seed)
    inp = r.uniform(-1, 1, (S, f) + tuple(n)).astype(np.float32)
    w = (r.standard_normal((fo, f) + tuple(k)) * (f * k[0] * k[1] * k[2]) ** -0.5).astype(np.float32)
    b = (r.standard_normal(fo) * np.sqrt(0.1)).astype(np.float32)
    return inp, w, b


def _run(inp, w, b=None, relu=False):
    d = torch.device("cuda:0")
    out = B.znni_conv3d_direct(torch.from_numpy(inp).to(d), torch.from_numpy(w).to(d),
                               torch.from_numpy(b).to(d) if b is not None else None, relu=relu)
    torch.cuda.synchronize()
    return out


# five to twenty images (part of an octet, whole octets, a part of a second and third), one to five row tiles and two row
# blocks, output rows below, at and above one, two and many column tiles, z remainders of 1, 2 and 3 behind groups of
# four, one to sixteen steps of slots, several inputs, kernels flat along each axis, more tiles than workgroups
CASES = [(1, 5, 1, (4, 5, 16), (2, 2, 2)), (1, 8, 80, (13, 9, 50), (2, 2, 2)), (2, 7, 33, (9, 10, 35), (2, 3, 1)),
         (1, 6, 12, (12, 11, 21), (3, 3, 3)), (1, 8, 44, (5, 17, 130), (1, 4, 1)), (3, 9, 17, (6, 6, 19), (1, 1, 3)),
         (1, 16, 16, (10, 33, 34), (2, 2, 2)), (1, 20, 64, (7, 8, 36), (1, 2, 2)), (1, 8, 90, (6, 7, 33), (2, 1, 2)),
         (1, 5, 5, (3, 3, 3), (3, 3, 3)), (1, 8, 16, (40, 70, 90), (1, 2, 1)), (1, 12, 20, (20, 9, 17), (7, 1, 1)),
         (5, 8, 49, (2, 3, 66), (1, 1, 1))]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "S%d_f%dx%d_n%s_k%s" % (c[0], c[1], c[2], "x".join(map(str, c[3])), "x".join(map(str, c[4]))))
def test_tile_and_slot_edges_match_oracle(oracle, case):
    S, f, fo, n, k = case
    inp, w, b = _rand(sum(n) + fo, S, f, fo, n, k)
    for relu, bias in ((False, None), (True, b)):
        got = _run(inp, w, bias, relu).cpu().numpy().astype(np.float64)
        exp = oracle.conv3d(inp, w, bias, relu=relu)
        # 32-bit accuracy: sums of at most 448 products, each off by 2^-23 of itself at most, in sums rounded once per
        # matrix product
        assert np.linalg.norm(got - exp) <= 5e-7 * np.linalg.norm(exp)
        assert np.all(np.abs(got - exp) <= oracle.tolerance(inp, w)[None, :, None, None, None])


def test_scales_are_powers_of_two():
    inp, w, _ = _rand(3, 1, 8, 20, (9, 10, 40), (2, 2, 2))
    base = _run(inp, w)
    for ei, ew in ((50, 0), (-70, 0), (0, 40), (0, -60)):
        assert torch.equal(_run(np.ldexp(inp, ei), np.ldexp(w, ew)), torch.ldexp(base, torch.tensor(ei + ew, device=base.device)))
    assert not _run(np.zeros_like(inp), w).any() and not _run(inp, np.zeros_like(w)).any()


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -float("inf")])
def test_values_that_are_not_finite(oracle, bad):
    """They reach the outputs whose windows hold them, as fp32 arithmetic has it (an infinity times a finite weight is an
    infinity), and no others."""
    inp, w, _ = _rand(4, 1, 8, 20, (9, 10, 40), (2, 2, 2))
    clean = _run(inp, w)
    inp[0, 3, 4, 5, 20] = bad
    got = _run(inp, w)
    win = (slice(None), slice(None), slice(3, 5), slice(4, 6), slice(19, 21))
    hit = torch.zeros_like(got, dtype=torch.bool)
    hit[win] = True
    assert torch.allclose(got[~hit], clean[~hit], rtol=0, atol=1e-6 * float(clean.abs().max()))
    if np.isnan(bad):
        assert torch.isnan(got[win]).all()
    else:
        assert torch.isinf(got[win]).all()
        # window corner (3, 4, 19) meets the value with the first tap of the flipped kernel
        assert torch.equal(torch.sign(got[0, :, 3, 4, 19]), torch.sign(torch.from_numpy(w[:, 3, 0, 0, 0]).to(got.device)) * np.sign(bad))


def test_axis_of_more_than_a_million(oracle):
    """Column tiles beyond a tile's edge store nothing, however long the axis they would land on."""
    inp, w, b = _rand(8, 1, 8, 8, (1200000, 1, 1), (2, 1, 1))
    got = _run(inp, w, b).cpu().numpy().astype(np.float64)
    exp = oracle.conv3d(inp, w, b)
    assert np.linalg.norm(got - exp) <= 5e-7 * np.linalg.norm(exp)
    assert np.all(np.abs(got - exp) <= oracle.tolerance(inp, w)[None, :, None, None, None])


def _close(oracle, inp, w, rel=2e-6):
    """Every output to `rel` of the sum of the magnitudes it adds up: what fp32 sums of up to 448 products give (the
    square root of their number times 2^-24, three standard deviations), however far apart the magnitudes in the layer lie."""
    got = _run(inp, w).cpu().numpy().astype(np.float64)
    bad = np.abs(got - oracle.conv3d(inp, w)) > rel * oracle.conv3d(np.abs(inp), np.abs(w)) + 1e-44
    assert not bad.any(), (int(bad.sum()), bad.size, np.argwhere(bad)[:4].tolist())


@pytest.mark.parametrize("big", [1e6, 1e9, 1e12, -float(np.finfo(np.float32).max)])
def test_a_large_value_leaves_its_neighbours_alone(oracle, big):
    inp, w, _ = _rand(9, 1, 8, 20, (9, 10, 40), (2, 2, 2))
    inp[0, 3, 4, 5, 20] = big
    _close(oracle, inp, w)


@pytest.mark.parametrize("shape", [(8, 20, (9, 10, 40), (2, 2, 2)), (11, 70, (8, 9, 35), (2, 1, 3)), (6, 17, (7, 9, 40), (1, 1, 1))])
def test_magnitudes_far_apart(oracle, shape):
    """Voxels over 2^80; input images up to 2^36 apart whose kernels make up for it; kernels with far smaller outer taps
    on images of single points; sparse images."""
    f, fo, n, k = shape
    r = np.random.default_rng(10)
    inp, w, _ = _rand(10, 1, f, fo, n, k)
    _close(oracle, np.ldexp(inp, r.integers(-40, 40, inp.shape)), w)
    e = r.integers(-18, 18, f)
    _close(oracle, np.ldexp(inp, e[:, None, None, None]), np.ldexp(w, -e[:, None, None, None]))
    points = np.where(r.random(inp.shape) < 0.01, inp, 0).astype(np.float32)
    _close(oracle, points, w)
    taps = np.indices(k).sum(0)
    _close(oracle, points, np.ldexp(w, -15 * taps))
    _close(oracle, np.maximum(inp, 0), w)


def test_scales_whose_product_is_in_range(oracle):
    """Images and kernels near either end of the exponent range whose products are ordinary numbers."""
    inp, w, _ = _rand(11, 1, 8, 20, (9, 10, 40), (2, 2, 2))
    for ei, ew in ((125, -100), (118, -66), (-110, 100), (-100, 60)):
        _close(oracle, np.ldexp(inp, ei), np.ldexp(w, ew))


def test_infinite_kernel_values(oracle):
    """An infinite kernel value gives an infinity of its product's sign, in its output image only."""
    inp, w, _ = _rand(12, 1, 8, 20, (9, 10, 40), (2, 2, 2))
    clean = _run(inp, w)
    w[7, 2, 0, 1, 1] = float("inf")
    got = _run(inp, w)
    assert torch.isinf(got[0, 7]).all()
    met = torch.from_numpy(inp[0, 2, 1:, :-1, :-1]).to(got.device)           # the voxel that tap meets (kernel flipped)
    assert torch.equal(torch.sign(got[0, 7]), torch.sign(met))
    keep = [j for j in range(20) if j != 7]
    assert torch.allclose(got[:, keep], clean[:, keep], rtol=0, atol=1e-6 * float(clean.abs().max()))


def test_replays_of_a_captured_call():
    """Tiles handed out from a counter that every call clears: replays of a graph, with eager calls between them."""
    inp, w, b = _rand(13, 1, 8, 80, (40, 30, 90), (2, 2, 2))
    d = torch.device("cuda:0")
    ti, tw, tb = (torch.from_numpy(t).to(d) for t in (inp, w, b))
    ws = torch.empty(B.znni_conv3d_direct_workspace(1, 8, 80, (40, 30, 90), (2, 2, 2)), dtype=torch.uint8, device=d)
    out = torch.empty((1, 80, 39, 29, 89), device=d)
    eager = _run(inp, w, b)
    B.znni_conv3d_direct(ti, tw, tb, out=out, workspace=ws)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        B.znni_conv3d_direct(ti, tw, tb, out=out, workspace=ws)
    for _ in range(4):
        out.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, eager)
        assert torch.equal(_run(inp, w, b), eager)
