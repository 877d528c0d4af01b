"""Multiply-accumulate without x transform: every strip width it is dealt in, over one input and over several, with waves
that have no strip, against the oracle."""
import numpy as np
import pytest
import torch

from paper_1606_05688_amd import binding as B

pytestmark = pytest.mark.gpu

# (S, outputs along x) that take strips of 1 to 5 column tiles, whole and ragged; the narrow row tiles take all of them, four
# and five row tiles up to three
STRIPS = {1: (1, 60), 2: (1, 122), 3: (5, 47), 4: (3, 58), 5: (1, 305), 6: (6, 33), 7: (2, 250)}
CASES = [(s, fo) for s in STRIPS for fo in (7, 31, 48, 50, 70)] + [(3, 97), (5, 129)]


@pytest.mark.parametrize("strip,fo", CASES, ids=lambda v: str(v))
def test_strips_match_oracle(oracle, strip, fo):
    S, nox = STRIPS[strip]
    f = (3, 16, 21, 36)[(strip + fo) % 4]
    kx = (5, 3, 4, 7, 2)[(strip * fo) % 5]
    n, k = (nox + kx - 1, 8, 10), (kx, 3, 2)
    r = np.random.default_rng(strip * 1000 + fo)
    inp = r.uniform(-1, 1, (S, f) + n).astype(np.float32)
    w = (r.standard_normal((fo, f) + k) * (f * np.prod(k)) ** -0.5).astype(np.float32)
    b = r.standard_normal(fo).astype(np.float32)
    print(f"[strips] {S} x {f} -> {fo}, {nox} outputs, {kx} taps", flush=True)
    d = torch.device("cuda:0")
    got = B.znni_conv3d_fft(*(torch.from_numpy(t).to(d) for t in (inp, w, b)), relu=True, mac_reference="xdirect")
    torch.cuda.synchronize()
    got = got.cpu().numpy().astype(np.float64)
    exp = oracle.conv3d(inp, w, b, relu=True)
    assert np.all(np.abs(got - exp) <= oracle.tolerance(inp, w)[None, :, None, None, None])
    assert np.linalg.norm(got - exp) <= 1e-6 * np.linalg.norm(exp)
