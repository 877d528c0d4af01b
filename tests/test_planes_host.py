"""Host side of the four-planes route: under a memory budget all blocks of input images of an output block write their
products in one layout, and the inverse that follows reads that one (a preloaded recorder stands in for the launches)."""
import ctypes
import os
import subprocess
import sys

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))


def _i3(v):
    return (ctypes.c_int * 3)(*[int(q) for q in v])


def walk(path, recorder, count):
    rec, L = ctypes.CDLL(recorder), ctypes.CDLL(path)
    rec.recorded_launches.restype = ctypes.c_char_p
    sz, vp = ctypes.c_size_t, ctypes.c_void_p
    rng = np.random.default_rng(5)
    mixed = planes = ran = 0
    while ran < count:
        S = int(rng.choice((1, 1, 1, 2, 9, 20)))
        f, fo = (int(np.exp(rng.uniform(0, np.log(128)))) for _ in range(2))
        base = int(np.exp(rng.uniform(np.log(8), np.log(64))))
        n = (int(base * rng.uniform(0.6, 1.5)), base, base)
        k = [int(min(rng.integers(1, 10), m)) for m in n]
        full = sz(0)
        if L.znni_conv3d_fft_workspace_v(S, f, fo, _i3(n), _i3(k), ctypes.byref(full)):
            continue
        budget = sz(int(full.value * rng.uniform(0.1, 1.0)))
        sub, need = _i3((0, 0, 0)), sz(0)
        if L.znni_conv3d_fft_sublayers_v(S, f, fo, _i3(n), _i3(k), budget, sub, ctypes.byref(need)):
            continue
        rec.recorded_launches()
        rc = L.znni_conv3d_fft_budget_v(S, f, fo, _i3(n), _i3(k), vp(1 << 12), vp(1 << 12), None, vp(1 << 12), 0, vp(1 << 20), budget, None)
        assert rc == 0, (rc, S, f, fo, n, k)
        state = None                                         # of the output block: forward and products in planes or not
        for name in rec.recorded_launches().decode().split():
            assert name != "?"
            here = "planes" in name
            if "k_mac" in name or "k_fwd" in name:
                assert state in (None, here), (S, f, fo, n, k, name)
                state = here
                planes += here
            elif "k_inv" in name or "ELi7E" in name or "ELi3E" in name and "k_pass" in name:
                assert state in (None, here), (S, f, fo, n, k, name)
                state = None
        mixed += sub[1] < f and f % sub[1] > 0
        ran += 1
    print(f"{ran} calls, {planes} launches in planes, {mixed} with a smaller last block")
    assert planes > 100 and mixed > 10


def test_blocks_of_one_output_block_share_a_layout(tmp_path):
    from paper_1606_05688_amd import binding as B            # (not in the walking process: torch's kernels would fill the record)
    so = str(tmp_path / "launch_recorder.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "launch_recorder.c")], check=True)
    env = dict(os.environ)
    env["LD_PRELOAD"] = so + (":" + env["LD_PRELOAD"] if env.get("LD_PRELOAD") else "")
    r = subprocess.run([sys.executable, os.path.abspath(__file__), B.lib()._name, so], env=env, capture_output=True, text=True,
                       timeout=600, cwd=os.path.dirname(HERE))
    assert r.returncode == 0, r.stdout[-1000:] + r.stderr[-3000:]


if __name__ == "__main__":
    walk(sys.argv[1], sys.argv[2], 1200)
