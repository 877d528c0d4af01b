"""Host side of the four-planes route (a preloaded recorder stands in for the launches).  Under a memory budget all blocks of
input images of an output block take one layout, and the inverse that follows reads that one; and the layers of the GPU tests reach
every kernel of the route and of the multiply-accumulate without x transform."""
import ctypes
import json
import os
import re
import subprocess
import sys

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))


def _i3(v):
    return (ctypes.c_int * 3)(*[int(q) for q in v])


# the passes' kinds as they are numbered in the kernels' names
PASS_FWD, PASS_INV = {0: "fwd_z", 1: "fwd_y", 2: "fwd_x", 6: "fwd_x"}, {3: "inv_x", 4: "inv_y", 5: "inv_z", 7: "inv_y of rows"}


def classify(name):
    """("fwd" / "mac" / "inv" / None, whether in planes)"""
    planes = "planes" in name
    m = re.search(r"k_pass(?:_long)?ILi\d+ELi\d+ELi(\d)E", name)
    if m:
        return ("fwd" if int(m.group(1)) in PASS_FWD else "inv"), planes
    for word, step in (("k_mac", "mac"), ("k_fwd", "fwd"), ("k_inv", "inv")):
        if word in name:
            return step, planes
    assert "k_twiddles" in name or "k_kprep" in name, name
    return None, planes


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
        state, last = None, None                             # of the output block: in planes or not; the step before
        for name in rec.recorded_launches().decode().split():
            assert name != "?"
            step, here = classify(name)
            if not step:
                continue
            if last == "inv" and step != "inv":              # the next output block
                state = None
            assert state in (None, here), (S, f, fo, n, k, name)
            state, last = here, step
            planes += here
        assert last == "inv"
        mixed += sub[1] < f and f % sub[1] > 0
        ran += 1
    print(f"{ran} calls, {planes} launches in planes, {mixed} with a smaller last block")
    assert planes > 100 and mixed > 10


def slabs(path, recorder, count):
    """Slabs along the halved axis give the whole layer's result bit for bit: every one runs the whole layer's kernel (a strip's
    width decides which values share a scale)."""
    rec, L = ctypes.CDLL(recorder), ctypes.CDLL(path)
    rec.recorded_launches.restype = ctypes.c_char_p
    sz, vp = ctypes.c_size_t, ctypes.c_void_p
    rng = np.random.default_rng(6)
    found = 0
    for _ in range(count):
        S, f, fo = int(rng.choice((1, 1, 2, 9))), int(rng.integers(8, 128)), int(rng.integers(8, 128))
        base = int(np.exp(rng.uniform(np.log(16), np.log(160))))
        n, k = (int(base * rng.uniform(0.2, 1.0)) + 9, base, base), [int(v) for v in rng.integers(1, 10, 3)]
        full = sz(0)
        if L.znni_conv3d_fft_workspace_v(S, f, fo, _i3(n), _i3(k), ctypes.byref(full)):
            continue
        names = []
        for share in (1.0, rng.uniform(0.4, 1.0)):
            rec.recorded_launches()
            rc = L.znni_conv3d_fft_budget_v(S, f, fo, _i3(n), _i3(k), vp(1 << 12), vp(1 << 12), None, vp(1 << 12), 0, vp(1 << 20),
                                            sz(int(full.value * share)), None)
            if rc == 0:
                names.append(rec.recorded_launches().decode().split())
        if len(names) < 2 or sum("k_kprep_z" in v for v in names[1]) != 1:
            continue
        whole, parts = ([v for v in w if "k_mac" in v] for w in names)
        found += len(parts) > 1
        assert set(parts) == set(whole), (S, f, fo, n, k, whole, parts)
    print(f"{found} layers in slabs")
    assert found > 20


def reach(path, recorder, layers):
    """Prints the kernels of the two families that none of the layers launches."""
    rec, L = ctypes.CDLL(recorder), ctypes.CDLL(path)
    rec.recorded_launches.restype = rec.registered_kernels.restype = ctypes.c_char_p
    vp, seen = ctypes.c_void_p, set()
    for flags, (S, f, fo, n, k) in json.loads(layers):
        full = ctypes.c_size_t(0)
        assert L.znni_conv3d_fft_workspace_v(S, f, fo, _i3(n), _i3(k), ctypes.byref(full)) == 0
        assert L.znni_conv3d_fft_v(S, f, fo, _i3(n), _i3(k), vp(1 << 12), vp(1 << 12), None, vp(1 << 12), flags, vp(1 << 20), full, None) == 0
        seen |= set(rec.recorded_launches().decode().split())
    every = [k for k in rec.registered_kernels().decode().split() if "planes" in k or "k_mac_xd" in k]
    print(f"{len(every)} kernels")
    assert len(every) > 50 and not set(every) - seen, sorted(set(every) - seen)


def _driven(tmp_path, *args):
    from paper_1606_05688_amd import binding as B            # (not in the walking process: torch's kernels would fill the record)
    so = str(tmp_path / "launch_recorder.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "launch_recorder.c")], check=True)
    env = dict(os.environ)
    env["LD_PRELOAD"] = so + (":" + env["LD_PRELOAD"] if env.get("LD_PRELOAD") else "")
    r = subprocess.run([sys.executable, os.path.abspath(__file__), B.lib()._name, so, *args], env=env, capture_output=True,
                       text=True, timeout=600, cwd=os.path.dirname(HERE))
    assert r.returncode == 0, r.stdout[-1000:] + r.stderr[-3000:]


def test_blocks_of_one_output_block_share_a_layout(tmp_path):
    _driven(tmp_path, "walk")


def test_slabs_run_the_whole_layers_kernel(tmp_path):
    _driven(tmp_path, "slabs")


def test_gpu_layers_reach_every_kernel(tmp_path):
    import test_gpu_planes as P
    import test_gpu_strips as T
    layers = [(0, c) for c in P.CASES] + [(16, T.strip_layer(*c)) for c in T.CASES] + [(16, c) for c in T.LAYERS]
    _driven(tmp_path, "reach", json.dumps(layers))


if __name__ == "__main__":
    if sys.argv[3] == "walk":
        walk(sys.argv[1], sys.argv[2], 1200)
    elif sys.argv[3] == "slabs":
        slabs(sys.argv[1], sys.argv[2], 4000)
    else:
        reach(sys.argv[1], sys.argv[2], sys.argv[4])
