"""Multiply-accumulate without x transform: every strip width it is dealt in, over one input and over several, with waves
that have no strip, against the oracle."""
import numpy as np
import pytest
import torch

from paper_1606_05688_amd import binding as B

pytestmark = pytest.mark.gpu

# (S, outputs along x), whole and ragged strips, over all row tiles
STRIPS = {1: (1, 60), 2: (1, 122), 3: (5, 47), 4: (3, 58), 5: (1, 305), 6: (6, 33), 7: (2, 250)}
CASES = [(s, fo) for s in STRIPS for fo in (7, 31, 48, 50, 70)] + [(3, 97), (5, 129)]


# (S, f, fo, n, k): with CASES every pair of row tiles (1 to 5) and column tiles (1 to 5, with four and five row tiles to 3), sums
# running and stepwise: all kernels (tests/test_planes_host.py counts them)
LAYERS = [(3, 17, 3, (133, 10, 9), (2, 2, 2)), (3, 17, 3, (77, 10, 9), (4, 2, 2)), (3, 17, 3, (195, 8, 14), (2, 2, 2)),
          (3, 17, 3, (261, 10, 9), (2, 2, 2)), (3, 17, 3, (138, 10, 9), (4, 2, 2)), (3, 17, 20, (78, 10, 9), (2, 2, 2)),
          (2, 17, 3, (202, 20, 9), (4, 2, 2)), (2, 17, 3, (263, 20, 9), (4, 2, 2)), (5, 17, 20, (58, 20, 9), (2, 2, 2)),
          (6, 17, 40, (35, 20, 9), (2, 2, 2)), (3, 17, 97, (66, 10, 9), (2, 2, 2)), (5, 17, 66, (34, 20, 9), (2, 2, 2)),
          (5, 17, 20, (275, 8, 9), (2, 2, 2)), (6, 17, 20, (55, 20, 9), (5, 2, 2)), (5, 17, 40, (37, 20, 10), (4, 2, 2)),
          (5, 17, 40, (207, 8, 9), (2, 2, 2)), (5, 21, 97, (37, 10, 9), (4, 2, 2)), (5, 17, 20, (266, 8, 9), (4, 2, 2)),
          (5, 17, 40, (66, 20, 14), (2, 2, 2)), (6, 17, 66, (41, 20, 9), (4, 2, 2)), (2, 17, 40, (197, 20, 9), (4, 2, 2)),
          (8, 17, 17, (3, 9, 9), (3, 2, 2)), (5, 17, 33, (3, 11, 12), (3, 2, 2)), (5, 17, 17, (5, 14, 14), (5, 2, 2)),
          (5, 17, 33, (5, 12, 12), (5, 2, 2)), (5, 17, 66, (3, 11, 11), (3, 2, 2)), (8, 17, 49, (5, 9, 9), (5, 2, 2)),
          (8, 17, 66, (5, 9, 10), (5, 2, 2)), (3, 17, 33, (73, 31, 32), (4, 2, 2))]


def _check(oracle, S, f, fo, n, k, seed):
    r = np.random.default_rng(seed)
    inp = r.uniform(-1, 1, (S, f) + n).astype(np.float32)
    w = (r.standard_normal((fo, f) + k) * (f * np.prod(k)) ** -0.5).astype(np.float32)
    b = r.standard_normal(fo).astype(np.float32)
    print(f"[strips] {S} x {f} -> {fo} of {n}, {k}", flush=True)
    d = torch.device("cuda:0")
    got = B.znni_conv3d_fft(*(torch.from_numpy(t).to(d) for t in (inp, w, b)), relu=True, mac_reference="xdirect")
    torch.cuda.synchronize()
    got = got.cpu().numpy().astype(np.float64)
    exp = oracle.conv3d(inp, w, b, relu=True)
    assert np.all(np.abs(got - exp) <= oracle.tolerance(inp, w)[None, :, None, None, None])
    assert np.linalg.norm(got - exp) <= 1e-6 * np.linalg.norm(exp)


def strip_layer(strip, fo):
    S, nox = STRIPS[strip]
    kx = (5, 3, 4, 7, 2)[(strip * fo) % 5]
    return S, (3, 16, 21, 36)[(strip + fo) % 4], fo, (nox + kx - 1, 8, 10), (kx, 3, 2)


@pytest.mark.parametrize("strip,fo", CASES, ids=lambda v: str(v))
def test_strips_match_oracle(oracle, strip, fo):
    _check(oracle, *strip_layer(strip, fo), strip * 1000 + fo)


@pytest.mark.parametrize("layer", LAYERS, ids=lambda c: "S%d_f%dx%d_n%s_k%d" % (c[0], c[1], c[2], c[3][0], c[4][0]))
def test_every_tile_matches_oracle(oracle, layer):
    _check(oracle, *layer, sum(layer[3]))
