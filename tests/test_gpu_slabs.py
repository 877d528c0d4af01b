"""Layers under a workspace budget whose kernel transforms do not fit but whose spectra do: run in slabs along the halved
axis, bit for bit the whole-layer result, inside the workspace given."""
import numpy as np
import pytest
import torch

from paper_1606_05688_amd import binding as B

pytestmark = pytest.mark.gpu

# (S, f, fo, n, k, share of the whole-layer workspace): taps along x in shifted reads and in blocks of eight, kernels of
# more than nine taps along y, two inputs, one slab short of the whole bank and many small slabs, a ragged last slab
CASES = [(1, 24, 20, (40, 64, 64), (5, 3, 3), 0.5), (1, 20, 24, (40, 64, 60), (3, 3, 3), 0.8), (1, 20, 24, (30, 130, 60), (7, 10, 2), 0.5),
         (2, 24, 33, (40, 128, 64), (4, 2, 3), 0.9), (1, 40, 48, (20, 64, 130), (6, 3, 3), 0.95)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "S%d_f%dx%d_n%s_k%s_%d%%" % (c[0], c[1], c[2], "x".join(map(str, c[3])), "x".join(map(str, c[4])), int(100 * c[5])))
def test_slabs_equal_the_whole_layer_call(case):
    S, f, fo, n, k, share = case
    r = np.random.default_rng(f + fo)
    d = torch.device("cuda:0")
    x = torch.from_numpy(r.uniform(-1, 1, (S, f) + n).astype(np.float32)).to(d)
    w = torch.from_numpy((r.standard_normal((fo, f) + k) * (f * np.prod(k)) ** -0.5).astype(np.float32)).to(d)
    b = torch.from_numpy(r.standard_normal(fo).astype(np.float32)).to(d)
    budget = int(share * B.znni_conv3d_fft_workspace(S, f, fo, n, k))
    assert B.znni_conv3d_fft_sublayers(S, f, fo, n, k, budget)[0] != (S, f, fo)
    ws = torch.full((budget + 4096,), 0xFF, dtype=torch.uint8, device=d)     # NaN patterns, and a guard behind the budget
    got = B.znni_conv3d_fft_budget(x, w, b, relu=True, workspace=ws[:budget])
    whole = B.znni_conv3d_fft(x, w, b, relu=True)
    torch.cuda.synchronize()
    assert torch.equal(got, whole)
    assert bool((ws[budget:] == 0xFF).all())
