"""The library in a process that never loads torch: there the run-time kernels are
compiled by ROCm's own compiler, not by the one that torch brings along.  Small
adjoint calls (whose last block adds the partial sums) of one-pass and block
kernels, one block and several: every output written, and right."""
import os
import subprocess
import sys

import numpy as np
import pytest

from ami_inputs import DEFAULT_Q, k_samples, matsubara_freqs, random_self_energy
from oracle.evaluate import energies_from_k, evaluate_terms, gradients, momentum_gradients, term_magnitudes

from parity import gradient_scales, oracle_terms, pole_distance

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BETA, T_HOP, MU = 4.0, 1.0, 0.1
CASES = [(2, (0, 2, 0), 300, 2), (4, (0, 4, 1), 1, 1), (4, (0, 4, 1), 700, 1), (4, (0, 4, 9), 1, 1),
         (4, (0, 4, 9), 300, 1), (5, (0, 5, 0), 1, 1), (5, (0, 5, 0), 130, 2)]

CHILD = r"""
import ctypes, sys
import numpy as np
root, work = sys.argv[1], sys.argv[2]
sys.path[:0] = [root, root + "/tests"]
import paper_2311_17189_amd as amd
from ami_inputs import DEFAULT_Q, random_self_energy
lib = amd.load_library()
path = next(l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l)
hip = ctypes.CDLL(path)
hip.hipMalloc.argtypes = [ctypes.c_void_p, ctypes.c_size_t]
hip.hipMemcpy.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_int]

def ok(e):
    assert e == 0, e

def put(a):
    a = np.ascontiguousarray(a)
    p = ctypes.c_void_p()
    ok(hip.hipMalloc(ctypes.byref(p), max(a.nbytes, 8)))
    ok(hip.hipMemcpy(p, a.ctypes.data, a.nbytes, 1))
    return p.value

def get(p, like):
    a = np.empty_like(like)
    ok(hip.hipMemcpy(a.ctypes.data, p, a.nbytes, 2))
    return a

q = np.array(DEFAULT_Q, dtype=np.float64)
for c in range(int(sys.argv[3])):
    z = np.load(f"{work}/in{c}.npz")
    d = random_self_energy(int(z["order"]), tuple(int(v) for v in z["seed"]))
    terms = amd.Terms.from_diagram(d)
    n_e, n_f = z["k"].shape[0], z["w"].shape[0]
    nan = float("nan")
    outs = dict(k=np.full(z["k"].shape, nan), mu=np.full(1, nan), t=np.full(1, nan), beta=np.full(1, nan),
                w=np.full((n_f, d.alpha.shape[1] - d.n_int), complex(nan, nan)), out=np.full((n_f, n_e), complex(nan, nan)),
                out_sum=np.full(n_f, complex(nan, nan)))
    dev = {n: put(a) for n, a in outs.items()}
    k, w, cot = put(z["k"]), put(z["w"].reshape(n_f, -1)), put(z["cot"])
    e = lib.amiEvaluateHubbardAdjoint(terms._h, k, n_e, z["k"].shape[1], q.ctypes.data, float(z["t"]), float(z["mu"]), w,
                                      n_f, float(z["beta"]), 0.0, cot, None, dev["k"], dev["mu"], dev["t"], dev["beta"],
                                      dev["w"], dev["out"], dev["out_sum"], None)
    assert e == 0, lib.amiLastError()
    ok(hip.hipDeviceSynchronize())
    np.savez(f"{work}/out{c}.npz", **{n: get(dev[n], a) for n, a in outs.items()})
    print("case", c, "done", flush=True)
assert "torch" not in sys.modules
"""


def test_small_adjoints_without_torch(tmp_path):
    q = np.array(DEFAULT_Q)
    cases = []
    for c, (order, seed, n_e, n_f) in enumerate(CASES):
        d = random_self_energy(order, seed)
        terms = oracle_terms(d)
        w = np.asarray(matsubara_freqs(n_f, BETA))
        k = k_samples(10 * n_e + 200, d.n_int, seed=(95, order))
        E = energies_from_k(d.alpha, k, q, T_HOP, MU)
        keep = np.flatnonzero(pole_distance(terms, d.n_int, E, w, 0.0).min(axis=0) > 0.02)[:n_e]
        assert len(keep) == n_e
        k, E = np.ascontiguousarray(k[keep]), np.ascontiguousarray(E[keep])
        rng = np.random.default_rng((96, c))
        cot = rng.standard_normal((n_f, n_e)) + 1j * rng.standard_normal((n_f, n_e))
        np.savez(tmp_path / f"in{c}.npz", order=order, seed=np.array(seed), k=k, w=w, cot=cot, t=T_HOP, mu=MU, beta=BETA)
        cases.append((d, terms, k, E, w, cot))
    env = dict(os.environ, AMIGPU_CACHE_DIR=str(tmp_path / "cache"))
    res = subprocess.run([sys.executable, "-c", CHILD, ROOT, str(tmp_path), str(len(cases))], env=env,
                         capture_output=True, text=True, timeout=100)
    assert res.returncode == 0, res.stdout[-1000:] + res.stderr[-2000:]
    for c, (d, terms, k, E, w, cot) in enumerate(cases):
        got = np.load(tmp_path / f"out{c}.npz")
        for name in got.files:
            assert np.isfinite(got[name]).all(), (CASES[c], name, "not written")
        sc = gradient_scales(terms, d.n_int, E, w, BETA, cot, 0.0, hubbard=(d.alpha, k, q, T_HOP, MU))
        dE, db, dw = gradients(terms, d.n_int, E, w, BETA, cot)
        dk, dmu, dt = momentum_gradients(d.alpha, k, q, T_HOP, MU, dE)
        for name, ref in (("k", dk), ("mu", dmu), ("t", dt), ("beta", db), ("w", dw)):
            ref = np.asarray(ref, dtype=got[name].dtype).reshape(got[name].shape)
            assert np.all(np.abs(got[name] - ref) <= 1e-10 * sc[name]), (CASES[c], name)
        ref = evaluate_terms(terms, d.n_int, E, w, BETA).astype(np.complex128)
        mag = term_magnitudes(terms, d.n_int, E, w, BETA)
        assert np.all(np.abs(got["out"] - ref) <= 1e-10 * mag), CASES[c]
        assert np.all(np.abs(got["out_sum"] - ref.sum(axis=1)) <= 1e-10 * mag.sum(axis=1)), CASES[c]
