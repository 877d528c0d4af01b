"""Host side of the route that cuts planes into tiles, and of small layers in four launches (a preloaded recorder stands in for
the launches): the layers of their GPU tests take them and reach all of their kernels, and a budget is kept."""
import ctypes
import json
import os
import subprocess
import sys

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))


def _i3(v):
    return (ctypes.c_int * 3)(*[int(q) for q in v])


def _open(path, recorder):
    rec, L = ctypes.CDLL(recorder), ctypes.CDLL(path)
    rec.recorded_launches.restype = rec.registered_kernels.restype = ctypes.c_char_p
    vp = ctypes.c_void_p

    def run(S, f, fo, n, k, share=1.0, flags=0):
        """Kernels launched, None where the call is refused."""
        full = ctypes.c_size_t(0)
        if L.znni_conv3d_fft_workspace_v(S, f, fo, _i3(n), _i3(k), ctypes.byref(full)):
            return None
        call = L.znni_conv3d_fft_v if share == 1.0 else L.znni_conv3d_fft_budget_v
        rec.recorded_launches()
        rc = call(S, f, fo, _i3(n), _i3(k), vp(1 << 12), vp(1 << 12), None, vp(1 << 12), flags, vp(1 << 20),
                  ctypes.c_size_t(int(full.value * share)), None)
        return rec.recorded_launches().decode().split() if rc == 0 else None

    return rec, run


def reach(path, recorder, layers):
    rec, run = _open(path, recorder)
    seen = set()
    for layer in json.loads(layers):
        names = run(*layer)
        assert any("k_fwd_tiles" in v for v in names), layer
        assert not any("tiles" in v for v in run(*layer, flags=16)), layer        # a form by name: whole planes
        seen |= set(names)
    every = {v for v in rec.registered_kernels().decode().split() if "tiles" in v}
    assert len(every) > 40 and not every - seen, sorted(every - seen)


def lengths(path, recorder, layers):
    """Turns of tiles of another length than the whole layer's."""
    _, run = _open(path, recorder)
    for layer, share in json.loads(layers):
        whole, turns = ([v for v in run(*layer, share=q) if "k_fwd_tiles" in v] for q in (1.0, share))
        assert len(whole) == 1 and turns and whole[0] not in turns, (layer, whole, turns)


def small(path, recorder, layers):
    """Four launches, of every kernel that has the first stage beside it."""
    rec, run = _open(path, recorder)
    seen = set()
    for layer in json.loads(layers):
        names = run(*layer)
        assert len(names) == 4 and "k_fwd_zy_small" in names[0], (layer, names)
        seen |= set(names)
    every = {v for v in rec.registered_kernels().decode().split() if "k_fwd_zy_small" in v}
    assert len(every) == 14 and not every - seen, sorted(every - seen)


def walk(path, recorder, count):
    """Every step of the route belongs to it, a transform on either side of a product, whatever the budget."""
    _, run = _open(path, recorder)
    rng = np.random.default_rng(9)
    tiled = turns = 0
    for _ in range(int(count)):
        S, f, fo = int(rng.choice((1, 1, 2, 5))), int(np.exp(rng.uniform(0, 4.5))), int(np.exp(rng.uniform(0, 4.5)))
        n, k = [int(np.exp(rng.uniform(2, 5.6))) for _ in range(3)], [int(v) for v in rng.integers(1, 10, 3)]
        for share in (1.0, float(rng.uniform(0.2, 0.95))):
            names = run(S, f, fo, n, [min(a, b) for a, b in zip(k, n)], share)
            steps = [v for v in names or [] if "tiles" in v]
            if not steps:
                continue
            tiled += 1
            turns += len(steps) > 3
            assert len(steps) % 3 == 0 and len(steps) + 3 == len(names), (S, f, fo, n, k, share)
            for q in range(0, len(steps), 3):
                assert [next(w for w in ("k_fwd", "k_mac", "k_inv") if w in v) for v in steps[q:q + 3]] == ["k_fwd", "k_mac", "k_inv"]
            assert len(set(steps)) == 3
    print(f"{tiled} calls in tiles, {turns} in turns")
    assert tiled > 300 and turns > 50


def _driven(tmp_path, *args):
    from paper_1606_05688_amd import binding as B            # (not in the walking process: torch's kernels would fill the record)
    so = str(tmp_path / "launch_recorder.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "launch_recorder.c")], check=True)
    env = dict(os.environ)
    env["LD_PRELOAD"] = so + (":" + env["LD_PRELOAD"] if env.get("LD_PRELOAD") else "")
    r = subprocess.run([sys.executable, os.path.abspath(__file__), B.lib()._name, so, *args], env=env, capture_output=True,
                       text=True, timeout=600, cwd=os.path.dirname(HERE))
    assert r.returncode == 0, r.stdout[-1000:] + r.stderr[-3000:]


def test_gpu_layers_reach_every_kernel(tmp_path):
    import test_gpu_tiles as T
    _driven(tmp_path, "reach", json.dumps(T.CASES))


def test_gpu_budgets_take_another_length(tmp_path):
    import test_gpu_tiles as T
    _driven(tmp_path, "lengths", json.dumps(T.OTHER_LENGTH))


def test_work_of_a_call_in_tiles():
    """48 -> 48 images of 320^3, 5^3 kernels: 10 x 10 tiles of length 36 (32 outputs of 316 an axis), 50 pairs; by form, whole planes."""
    from paper_1606_05688_amd import binding as B
    f = fo = 48
    n, k, no, N, pairs = 320, 5, 316, 36, 50
    x, y, bank = 8 * f * n * N * N * pairs, 8 * fo * no * N * N * pairs, 8 * (N // 2 + 1) * N * f * fo * k
    nb, fl = B.znni_conv3d_fft_call_work(1, f, fo, n, k)
    assert {q: v for q, v in nb.items() if v} == {"kernel_prep": 4 * f * fo * k ** 3 + bank, "fwd_z": 4 * f * n ** 3 + x,
                                                  "mac": x + bank + y, "inv_y": y + 4 * fo * no ** 3}
    assert {q: v for q, v in fl.items() if v} == {"mac": 8 * k * f * fo * no * N * N * pairs}
    assert B.znni_conv3d_fft_call_work(1, f, fo, n, k, keep_kernels=True)[0]["kernel_prep"] == 0
    for form in ("xdirect", "single", "generic_passes"):
        assert B.znni_conv3d_fft_call_work(1, f, fo, n, k, mac_reference=form) == B.znni_conv3d_fft_stage_work(1, f, fo, n, k, mac_reference=form)
    assert B.znni_conv3d_fft_call_work(8, 32, 32, 64, 7) == B.znni_conv3d_fft_stage_work(8, 32, 32, 64, 7)


def test_small_layers_take_four_launches(tmp_path):
    import test_gpu_small as S
    _driven(tmp_path, "small", json.dumps(S.CASES))


def test_steps_belong_together(tmp_path):
    _driven(tmp_path, "walk", "1500")


if __name__ == "__main__":
    {"reach": reach, "lengths": lengths, "small": small, "walk": walk}[sys.argv[3]](sys.argv[1], sys.argv[2], sys.argv[4])
