"""Host side of the routes a call takes, by the kernels it would launch (a preloaded recorder stands in for the launches)."""
import os
import subprocess
import sys

import pytest

from paper_1606_05688_amd import binding as B

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("rec") / "launch_recorder.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "launch_recorder.c")], check=True)
    return so


def test_blocks_of_one_output_block_take_one_route(recorder):
    """Products of several blocks of input images are added up in one set of spectra: all of them in the same layout."""
    env = dict(os.environ)
    env["LD_PRELOAD"] = recorder + (":" + env["LD_PRELOAD"] if env.get("LD_PRELOAD") else "")
    r = subprocess.run([sys.executable, os.path.join(HERE, "routes_driver.py"), B.lib()._name, recorder, "1500"], env=env,
                       capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stdout[-1000:] + r.stderr[-3000:]
    assert "one route each" in r.stdout


# (S, f, fo, n, k, route): measured on the routes that take the layer, the fastest one named, or one that is level with it
# (10 -> 44 and 18 -> 122 untransformed either way; 50 -> 8 of 19^3 47 us on both routes but the third)
@pytest.mark.parametrize("layer", [(1, 10, 44, 59, 3, "xdirect"), (1, 8, 8, 64, 5, "planes"), (1, 7, 1, 65, 7, "xdirect"),
                                   (1, 80, 80, 100, 5, "xdirect"), (1, 50, 8, 19, 7, "planes"), (7, 88, 1, 37, 2, "full x"),
                                   (4, 4, 118, 19, 3, "planes"), (7, 103, 7, 54, 3, "full x"), (1, 45, 30, 16, 7, "planes"),
                                   (1, 18, 122, 41, 6, "xdirect"), (3, 83, 6, 41, 5, "xdirect"), (64, 80, 80, 51, 5, "planes"),
                                   (8, 32, 32, 64, 7, "planes"), (1, 9, 121, 14, 7, "planes"), (1, 32, 32, 64, 7, "xdirect")],
                         ids=lambda c: "S%d_f%dx%d_n%d_k%d_%s" % c)
def test_small_images_take_the_faster_route(layer):
    S, f, fo, n, k, route = layer
    nbytes, flops = B.znni_conv3d_fft_stage_work(S, f, fo, n, k)
    fused = nbytes["fwd_y"] == 0 and nbytes["inv_z"] == 0
    assert ("full x" if nbytes["fwd_x"] else "planes" if fused else "xdirect") == route
    # the products are the method's, however the rows lie
    untransformed = B.znni_conv3d_fft_stage_work(S, f, fo, n, k, mac_reference="xdirect")[1]
    assert (flops == untransformed) == (route != "full x")


# few pencils and long sums: a wave of the untransformed route would walk through the whole sum alone (us there and transformed:
# 386 and 202, 397 and 225, 285 and 175, 225 and 132); wide banks make up for it (1855 and 2382, 610 and 901)
@pytest.mark.parametrize("layer,transformed", [((1, 1104, 2, 8, 7), True), ((1, 1343, 5, 9, 6), True), ((1, 1225, 6, 8, 5), True),
                                               ((1, 1232, 4, 7, 5), True), ((1, 991, 237, 13, 7), False), ((1, 873, 334, 9, 4), False),
                                               ((1, 1061, 69, 7, 4), False), ((1, 27, 8, 9, 7), False), ((1, 96, 3, 10, 9), False),
                                               ((4, 121, 3, 11, 9), True)], ids=str)
def test_long_sums_of_few_pencils(layer, transformed):
    nbytes, _ = B.znni_conv3d_fft_stage_work(*layer)
    assert (nbytes["fwd_x"] > 0) == transformed


def test_closer_direct_sums_are_not_left_for_little():
    """Direct sums of few products are closer to 64 bits than transforms (1.8e-8 sqrt(products) of the result, 1.4e-8 on split
    halves, next to 2e-7): layers that rates alone give to the direct kernels stay there."""
    direct = [(1, 4, 4, (188, 175, 251), (5, 2, 1)), (1, 2, 50, (181, 198, 159), (3, 3, 4)), (1, 3, 18, (305,) * 3, (3,) * 3),
              (1, 3, 20, (60,) * 3, (3,) * 3), (1, 11, 5, (112, 105, 104), (4, 2, 1)), (1, 19, 4, (53,) * 3, (2,) * 3)]
    # sums of more products, and layers that transforms are far ahead at
    transformed = [(1, 4, 16, (72,) * 3, (4,) * 3), (1, 2, 46, (24,) * 3, (4,) * 3), (1, 54, 11, (116,) * 3, (2,) * 3), (1, 40, 40, (128,) * 3, (3,) * 3)]
    for layers, want in ((direct, "direct"), (transformed, "fft")):
        for layer in layers:
            assert B.znni_conv3d_choose(*layer)[0] == want, layer
