"""Walks random layers under a memory budget and looks at what each call launches (run by tests/test_routes_host.py in a
process whose LD_PRELOAD names the launch recorder; no GPU, no torch).

usage: routes_driver.py <libznni.so> <recorder.so> <number of layers>
"""
import ctypes
import re
import sys

import numpy as np


def i3(v):
    return (ctypes.c_int * 3)(*[int(q) for q in v])


def family(name):
    """Which layout of output spectra a multiply-accumulate kernel writes; None for other kernels."""
    if "k_mac_planes" in name:
        return "four planes"
    if "k_mac_xd" in name or "k_mac_xb" in name:
        return "x not transformed"
    return "x transformed" if re.search(r"k_mac", name) else None


def blocks(launches):
    """For every output block the families of its multiply-accumulates and the kernel that starts its inverse."""
    out, macs = [], []
    for name in launches:
        if family(name):
            macs.append(family(name))
        elif macs and not re.search(r"k_twiddles|k_kprep|fwd|k_pass(_long)?ILi\d+ELi\d+ELi[0126]E", name):
            out.append((macs, name))
            macs = []
    assert not macs
    return out


def main(path, recorder, count):
    rec = ctypes.CDLL(recorder)
    rec.recorded_launches.restype = ctypes.c_char_p
    L = ctypes.CDLL(path)
    sz, vp = ctypes.c_size_t, ctypes.c_void_p
    rng = np.random.default_rng(11)
    ran = divided = ragged = 0
    seen = set()
    layers = [(1, 91, 38, (18, 18, 18), (6, 6, 6), 0.8), (1, 88, 14, (23, 23, 23), (6, 6, 6), 0.8),
              (1, 77, 83, (17, 17, 17), (7, 7, 7), 0.8), (1, 115, 27, (17, 28, 27), (6, 3, 5), 0.6),
              (1, 40, 20, (100, 100, 100), (5, 5, 5), 0.5), (1, 24, 40, (24, 20, 16), (5, 5, 2), 0.25)]
    while len(layers) < count:
        f, fo = (int(np.exp(rng.uniform(0, np.log(128)))) for _ in range(2))
        S = int(rng.choice((1, 1, 1, 2, 9)))
        base = np.exp(rng.uniform(np.log(6), np.log(110)))
        n = [max(1, int(base * rng.uniform(0.7, 1.5))) for _ in range(3)]
        k = [int(min(rng.integers(1, 8), m)) for m in n]
        layers.append((S, f, fo, n, k, float(rng.uniform(0.1, 1.0))))
    for S, f, fo, n, k, share in layers:
        full, sub, need = sz(0), i3((0, 0, 0)), sz(0)
        if L.znni_conv3d_fft_workspace_v(S, f, fo, i3(n), i3(k), ctypes.byref(full)):
            continue
        budget = int(full.value * share)
        if L.znni_conv3d_fft_sublayers_v(S, f, fo, i3(n), i3(k), sz(budget), sub, ctypes.byref(need)):
            continue
        divided += sub[1] < f
        ragged += sub[1] < f and f % sub[1] > 0
        for flags in (0, 4, 8, 16, 32, 128):
            rec.recorded_launches()
            rc = L.znni_conv3d_fft_budget_v(S, f, fo, i3(n), i3(k), vp(1 << 12), vp(1 << 12), None, vp(1 << 12), flags,
                                            vp(1 << 20), sz(budget), None)
            assert rc == 0, (rc, S, f, fo, n, k, share, flags)
            names = rec.recorded_launches().decode().split()
            assert names and "?" not in names
            for macs, inverse in blocks(names):
                assert len(set(macs)) == 1, f"{S} x {f} -> {fo} of {n}, kernels {k}, flags {flags}: {macs}"
                # and the inverse reads what they wrote (pass 7: rows of x as they are)
                assert (macs[0] == "x not transformed") == bool(re.search(r"k_pass(_long)?ILi\d+ELi\d+ELi7E", inverse)), inverse
                assert (macs[0] == "four planes") == ("k_inv_yz_planes" in inverse), inverse
                seen.add(macs[0])
            ran += 1
    print(f"{ran} calls, {divided} layers in blocks of input images, {ragged} with a smaller last block: one route each")
    assert divided > 20 and ragged > 10 and len(seen) == 3


if __name__ == "__main__":
    main(sys.argv[1], sys.argv[2], int(sys.argv[3]))
