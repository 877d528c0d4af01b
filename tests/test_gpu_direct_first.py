"""Direct convolution of layers of few taps (csrc/direct_first.hip) against the fp64 oracle; tests/test_direct_first_host.py shows
that these layers run there and reach all of its kernels."""
import numpy as np
import pytest
import torch

from paper_1606_05688_amd import binding as B

pytestmark = pytest.mark.gpu

# Tiles of 32, 64 and 128 columns with one column, all but one and all of them in use; last rows of a tile, one row; ends of rows of
# one to four outputs; one to five row tiles and two blocks of them, the last ragged; one and two steps of taps, 16, 32 and 64
# of them; tiles of up to 7 and up to 13 values a thread; turns of one and of several tiles; several inputs
CASES = [(1, 3, 10, (38, 34, 35), (3, 2, 2)), (8, 3, 16, (30, 34, 35), (3, 2, 2)), (3, 1, 16, (33, 40, 66), (1, 4, 4)), (1, 4, 30, (24, 40, 66), (2, 2, 3)),
         (2, 2, 17, (30, 39, 130), (4, 2, 2)), (2, 1, 48, (20, 33, 131), (3, 3, 3)), (1, 1, 41, (60, 66, 67), (3, 3, 3)), (4, 1, 64, (20, 36, 34), (3, 3, 3)),
         (1, 2, 33, (26, 37, 63), (3, 3, 3)), (1, 4, 16, (50, 60, 130), (2, 2, 2)), (1, 1, 40, (30, 40, 97), (4, 4, 4)), (1, 4, 90, (14, 50, 131), (2, 2, 3)),
         (1, 2, 100, (22, 33, 71), (2, 2, 3)), (2, 3, 80, (32, 40, 66), (2, 2, 2)), (2, 4, 55, (24, 40, 129), (2, 2, 2)), (2, 4, 20, (30, 50, 64), (2, 4, 2)),
         (1, 3, 75, (60, 40, 66), (3, 1, 3)), (2, 2, 8, (40, 64, 64), (4, 4, 2)), (1, 4, 32, (98, 7, 140), (2, 3, 2)), (2, 1, 64, (33, 33, 34), (4, 4, 2)),
         (2, 4, 9, (40, 66, 70), (2, 3, 1)), (1, 1, 24, (40, 61, 62), (3, 3, 3)),
         (1, 1, 75, (40, 64, 66), (3, 3, 3)), (2, 4, 48, (20, 40, 130), (2, 2, 2)), (2, 4, 78, (30, 64, 130), (2, 2, 2))]


def _run(inp, w, b=None, relu=False):
    d = torch.device("cuda:0")
    out = B.znni_conv3d_direct(torch.from_numpy(inp).to(d), torch.from_numpy(w).to(d), None if b is None else torch.from_numpy(b).to(d), relu=relu)
    torch.cuda.synchronize()
    return out


def _rand(seed, S, f, fo, n, k):
    r = np.random.default_rng(seed)
    w = (r.standard_normal((fo, f) + tuple(k)) * (f * np.prod(k)) ** -0.5).astype(np.float32)
    return r.uniform(-1, 1, (S, f) + tuple(n)).astype(np.float32), w, r.standard_normal(fo).astype(np.float32)


@pytest.mark.parametrize("case", CASES, ids=lambda c: "S%d_f%dx%d_n%s_k%s" % (c[0], c[1], c[2], "x".join(map(str, c[3])), "x".join(map(str, c[4]))))
def test_matches_oracle(oracle, case):
    S, f, fo, n, k = case
    print(case, flush=True)
    inp, w, b = _rand(sum(n) + fo, S, f, fo, n, k)
    for relu, bias in ((False, None), (True, b)):
        got, exp = _run(inp, w, bias, relu).cpu().numpy().astype(np.float64), oracle.conv3d(inp, w, bias, relu=relu)
        # 32-bit accuracy: at most 64 products, each off by 2^-22 of itself at most, in sums rounded once per matrix product
        assert np.linalg.norm(got - exp) <= 5e-7 * np.linalg.norm(exp)
        assert np.all(np.abs(got - exp) <= oracle.tolerance(inp, w)[None, :, None, None, None])
    # magnitudes that halves of one scale do not hold (images or kernels): fp32, at most 64 products rounded once each
    far = np.exp2(np.random.default_rng(5).integers(-40, 1, n)).astype(np.float32)
    odd = np.arange(k[2]) % 2
    for x, v in ((inp * far, w), (inp, w * np.exp2(-30.0 * odd).astype(np.float32)), (inp, w * np.exp2(-45.0 * odd).astype(np.float32))):
        got, exp, mag = _run(x, v).cpu().numpy().astype(np.float64), oracle.conv3d(x, v, None, relu=False), oracle.conv3d(np.abs(x), np.abs(v), None, relu=False)
        assert np.all(np.abs(got - exp) <= 64 * 2.0 ** -24 * mag)


def test_scales_are_powers_of_two():
    inp, w, _ = _rand(3, *CASES[5])
    base = _run(inp, w)
    for ei, ew in ((50, 0), (-70, 0), (0, 40), (0, -60)):
        assert torch.equal(_run(np.ldexp(inp, ei), np.ldexp(w, ew)), torch.ldexp(base, torch.tensor(ei + ew, device=base.device)))
    assert not _run(np.zeros_like(inp), w).any() and not _run(inp, np.zeros_like(w)).any()


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -float("inf")])
def test_values_that_are_not_finite(bad):
    """They reach the outputs whose windows hold them and no others."""
    S, f, fo, n, k = CASES[5]
    inp, w, _ = _rand(4, S, f, fo, n, k)
    clean = _run(inp, w)
    inp[0, 0, 7, 9, 127] = bad
    got = _run(inp, w)
    win = (slice(0, 1), slice(None), slice(5, 8), slice(7, 10), slice(125, 128))
    hit = torch.zeros_like(got, dtype=torch.bool)
    hit[win] = True
    assert torch.allclose(got[~hit], clean[~hit], rtol=0, atol=1e-6 * float(clean.abs().max()))
    assert (torch.isnan(got[win]) if np.isnan(bad) else torch.isinf(got[win])).all()


@pytest.mark.parametrize("low", [16, 19, 36, 38])
@pytest.mark.parametrize("where", ["images", "kernels"])
def test_values_far_below_others_of_their_scale(oracle, where, low):
    """Results made of values that share a scale with far larger ones, which they never meet, are as good as any: a rounding of
    2^-24 for each of K sums whose size grows with the square root of their terms, sqrt(K / 2) 2^-24 together."""
    S, f, fo, n, k = {"images": CASES[5], "kernels": CASES[4]}[where]
    r = np.random.default_rng(low)
    inp, w = (np.where(r.random(s) < 0.5, -1, 1) * r.uniform(1, 2, s) for s in ((S, f) + n, (fo, f) + k))
    K = f * int(np.prod(k))
    keep = np.ones([a - b + 1 for a, b in zip(n, k)], dtype=bool)
    if where == "images":                                    # one column of every 32
        inp *= 2.0 ** -low
        inp[..., 5::32] = 1
        for z in range(k[2]):
            keep[..., 5 - z::32] = False
    else:                                                    # the second image has the large kernels, and no values
        w[:, 0] *= 2.0 ** -low
        w[:, 1] = 1
        inp[:, 1] = 0
        K //= 2
    inp, w = inp.astype(np.float32), w.astype(np.float32)
    exp = oracle.conv3d(inp, w, None, relu=False)[:, :, keep]
    got = _run(inp, w).cpu().numpy().astype(np.float64)[:, :, keep]
    assert np.linalg.norm(got - exp) <= np.sqrt(K / 2) * 2.0 ** -24 * np.linalg.norm(exp)
