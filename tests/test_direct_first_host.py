"""Host side of the direct convolution of few taps (a preloaded recorder stands in for the launches): the layers of its GPU test run
there and reach all of its kernels, and random layers take one direct kernel or the other."""
import ctypes
import json
import os
import subprocess
import sys

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))


def _i3(v):
    return (ctypes.c_int * 3)(*[int(q) for q in v])


def reach(path, recorder, layers):
    rec, L = ctypes.CDLL(recorder), ctypes.CDLL(path)
    rec.recorded_launches.restype = rec.registered_kernels.restype = ctypes.c_char_p
    vp = ctypes.c_void_p

    def run(S, f, fo, n, k):
        full = ctypes.c_size_t(0)
        if L.znni_conv3d_direct_workspace_v(S, f, fo, _i3(n), _i3(k), ctypes.byref(full)):
            return None
        call = lambda short: L.znni_conv3d_direct_v(S, f, fo, _i3(n), _i3(k), vp(1 << 12), vp(1 << 12), None, vp(1 << 12), 0, vp(1 << 20),
                                                    ctypes.c_size_t(full.value - short), None)
        rec.recorded_launches()
        assert call(1) != 0 and not rec.recorded_launches()           # the workspace stays what the call asks for
        assert call(0) == 0
        return rec.recorded_launches().decode().split()

    seen = set()
    for layer in json.loads(layers):
        names = run(*layer)
        assert len(names) == 1 and "k_direct_first" in names[0], (layer, names)
        seen |= set(names)
    every = {v for v in rec.registered_kernels().decode().split() if "k_direct_first" in v}
    assert len(every) == 13 and not every - seen, sorted(every - seen)
    # one kernel or the other, at most 64 taps; both are in use
    rng, count = np.random.default_rng(4), [0, 0]
    for _ in range(3000):
        S, f, fo = int(rng.choice((1, 1, 2, 8))), int(rng.integers(1, 9)), int(np.exp(rng.uniform(0, 5)))
        n, k = [int(np.exp(rng.uniform(1, 5.8))) for _ in range(3)], [int(v) for v in rng.integers(1, 6, 3)]
        k = [min(a, b) for a, b in zip(k, n)]
        names = run(S, f, fo, n, k)
        if names is None:
            continue
        first = "k_direct_first" in names[0]
        count[first] += 1
        assert not first or (len(names) == 1 and 12 < f * k[0] * k[1] * k[2] <= 64)
    print(count)
    assert min(count) > 300


def test_gpu_layers_reach_every_kernel(tmp_path):
    import test_gpu_direct_first as T
    from paper_1606_05688_amd import binding as B            # (not in the walking process: torch's kernels would fill the record)
    so = str(tmp_path / "launch_recorder.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "launch_recorder.c")], check=True)
    env = dict(os.environ)
    env["LD_PRELOAD"] = so + (":" + env["LD_PRELOAD"] if env.get("LD_PRELOAD") else "")
    r = subprocess.run([sys.executable, os.path.abspath(__file__), B.lib()._name, so, json.dumps(T.CASES)], env=env, capture_output=True,
                       text=True, timeout=600, cwd=os.path.dirname(HERE))
    assert r.returncode == 0, r.stdout[-1000:] + r.stderr[-3000:]


def test_estimate_counts_the_turns_that_are_launched():
    """One row tile: three workgroups on each of 256 compute units, so that the step to a second turn lies behind 768 tiles."""
    from paper_1606_05688_amd import binding as B

    def us(tiles):                                           # one tile of 8 x 32 outputs for every x
        prim, est = ctypes.c_int(), (ctypes.c_float * 2)()
        assert B.lib().znni_conv3d_choose_v(1, 1, 4, _i3((tiles + 2, 10, 34)), _i3((3, 3, 3)), ctypes.byref(prim), est) == 0
        return est[1]

    assert us(760) - us(500) < us(780) - us(760)


if __name__ == "__main__":
    reach(sys.argv[1], sys.argv[2], sys.argv[3])
