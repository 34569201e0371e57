"""The generated sources of the block kernels on the CPU: the code generator
under AddressSanitizer and UndefinedBehaviorSanitizer
(tests/cpu_math/block_source.cpp), and the generated code against the oracle, a
host thread per wave (tests/cpu_math/jit_check_block.cpp)."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from ami_inputs import (DEFAULT_Q, complex_energies, k_samples, matsubara_freqs, random_self_energy, real_freqs,
                        uniform_energies)
from oracle.evaluate import energies_from_k, evaluate_terms, gradients, momentum_gradients, term_magnitudes

from parity import check, gradient_scales, oracle_terms, pole_distance

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2311_17189_amd", "csrc")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path_factory.mktemp("block_source") / "block_source")
    srcs = [os.path.join(CSRC, f) for f in ("construct.cpp", "graph.cpp", "codegen.cpp", "abi.cpp")]
    subprocess.run([cxx, "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-I", os.path.join(ROOT, "include"), os.path.join(HERE, "cpu_math", "block_source.cpp"), *srcs,
                    "-o", exe], check=True, capture_output=True, text=True)

    def run(d, *args):
        text = [f"{d.alpha.shape[0]} {d.eps.shape[1]} {d.alpha.shape[1]} {d.n_int}",
                " ".join(str(int(v)) for v in np.asarray(d.alpha).ravel()),
                " ".join(str(int(v)) for v in np.asarray(d.eps).ravel())]
        env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:abort_on_error=1")
        for k in ("LD_PRELOAD", "AMIGPU_JIT_BLOCK_WAVES"):
            env.pop(k, None)
        res = subprocess.run([exe, *[str(a) for a in args]], input="\n".join(text) + "\n", capture_output=True,
                             text=True, env=env)
        assert res.returncode == 0, res.stderr[-2000:]
        return res.stdout

    return run


@pytest.mark.parametrize("order,seed", [(5, (0, 5, 4)), (6, (0, 6, 0))])
def test_a_handle_keeps_its_waves(driver, order, seed):
    """The launch takes the count chosen first; the source must hold the same
    one, also when the override changes in between."""
    first, again, source = (int(v) for v in driver(random_self_energy(order, seed), "override").split())
    assert first > 0 and again == first and source == first


ADJOINT, COMPLEX, FORWARD = 8192, 16384, 32768
WAVES = {(4, (0, 4, 9)): 2, (5, (0, 5, 4)): 2, (5, (0, 5, 0)): 4, (6, (0, 6, 0)): 4, (6, (5, 6, 4)): 8}


def _program(src, tmp_path):
    body = "\n".join(l for l in src.splitlines()
                     if l.strip() not in ('#include "kargs.hpp"', '#include "jit_kernel.hpp"'))
    gen = tmp_path / "block.inc"
    gen.write_text(body)
    exe = str(tmp_path / "block")
    subprocess.run([shutil.which("g++"), "-O1", "-std=c++17", "-ffp-contract=off", "-pthread", "-I",
                    os.path.join(HERE, "cpu_math", "shim"), f'-DAMI_GENERATED="{gen}"',
                    os.path.join(HERE, "cpu_math", "jit_check_block.cpp"), "-o", exe], check=True, capture_output=True)
    return exe


def _numbers(a):
    a = np.asarray(a).ravel()
    return " ".join(f"{float(z.real)!r} {float(z.imag)!r}" if np.iscomplexobj(a) else repr(float(z)) for z in a)


# 76 terms (two waves, the values by one of them), 136, 264, 560 (four), 2512 in 224 groups (eight)
@pytest.mark.parametrize("order,seed,kernel,momentum,n_f,n", [
    (4, (0, 4, 9), ADJOINT, True, 1, 60), (4, (0, 4, 9), ADJOINT, False, 3, 60), (5, (0, 5, 4), ADJOINT, False, 1, 40),
    (5, (0, 5, 0), ADJOINT, True, 3, 40), (6, (5, 6, 4), ADJOINT, False, 1, 10),
    (5, (0, 5, 0), COMPLEX, False, 1, 30), (5, (0, 5, 0), COMPLEX, False, 3, 30),
    (6, (0, 6, 0), FORWARD, True, 9, 20), (6, (5, 6, 4), FORWARD, False, 9, 10)])
def test_generated_block_kernels_match_oracle(driver, tmp_path, order, seed, kernel, momentum, n_f, n):
    d = random_self_energy(order, seed)
    src = driver(d, "source", kernel, int(momentum))
    assert src, "the solution must split over the waves of a block"
    if kernel == ADJOINT:
        assert f"constexpr int NW = {WAVES[order, seed]}," in src
    exe = _program(src, tmp_path)
    beta, e_reg, t, mu = 4.0, 0.0 if momentum else 0.03, 1.0, 0.1
    q = np.array(DEFAULT_Q)
    w = np.concatenate([matsubara_freqs(n_f, beta)[: (n_f + 1) // 2], real_freqs(n_f, -1.0, 1.0, 0.1)[: n_f // 2]])
    if momentum:
        x = k_samples(10 * n + 100, d.n_int, seed=(93, order))
        E = energies_from_k(d.alpha, x, q, t, mu)
    elif kernel == COMPLEX:
        x = E = complex_energies(10 * n + 100, d.n_eps, seed=(93, order), a=3.0, eta=0.05)
    else:
        x = E = uniform_energies(10 * n + 100, d.n_eps, seed=(93, order), a=3.0)
    terms = oracle_terms(d)
    keep = np.flatnonzero(pole_distance(terms, d.n_int, E, w, e_reg).min(axis=0) > 0.02)[:n]
    assert len(keep) == n
    x, E = np.ascontiguousarray(x[keep]), np.ascontiguousarray(E[keep])
    rng = np.random.default_rng(94)
    cot = rng.standard_normal((n_f, n)) + 1j * rng.standard_normal((n_f, n))
    lines = [f"{n} {n_f} {beta!r} {e_reg!r} {t!r} {mu!r}", _numbers(q[:2 * (d.alpha.shape[1] - d.n_int)]), _numbers(w)]
    for s in range(n):
        lines.append(_numbers(x[s]) + ("" if kernel == FORWARD else " " + _numbers(cot[:, s])))
    res = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True, check=True)
    out = np.array([[float(v) for v in l.split()] for l in res.stdout.strip().splitlines()])
    vals = (out[:, 0:2 * n_f:2] + 1j * out[:, 1:2 * n_f:2]).T
    ref = evaluate_terms(terms, d.n_int, E, w, beta, e_reg).astype(np.complex128)
    scale = term_magnitudes(terms, d.n_int, E, w, beta, e_reg).astype(np.float64)
    check(vals, ref, scale, pole_distance(terms, d.n_int, E, w, e_reg), label=f"block kernel {kernel} values")
    if kernel == FORWARD:
        return
    rest = out[:, 2 * n_f:]
    hub = (d.alpha, x, q, t, mu) if momentum else None
    sc = gradient_scales(terms, d.n_int, E, w, beta, cot, e_reg, hubbard=hub)
    dE, db, dw = gradients(terms, d.n_int, E, w, beta, cot, e_reg)
    if kernel == COMPLEX:
        g, want, rest = rest[:, 0:2 * d.n_eps:2] + 1j * rest[:, 1:2 * d.n_eps:2], dE, rest[:, 2 * d.n_eps:]
    elif momentum:
        want, dmu, dt = momentum_gradients(d.alpha, x, q, t, mu, dE)
        g, rest = rest[:, :2 * d.n_int], rest[:, 2 * d.n_int:]
        assert abs(rest[:, 1].sum() - float(dmu)) <= 1e-10 * sc["mu"]
        assert abs(rest[:, 2].sum() - float(dt)) <= 1e-10 * sc["t"]
    else:
        g, want, rest = rest[:, :d.n_eps], dE, rest[:, d.n_eps:]
    want = np.asarray(want).astype(np.complex128 if kernel == COMPLEX else np.float64).reshape(g.shape)
    assert np.max(np.abs(g - want) / np.maximum(sc["k" if momentum else "E"], 1e-300)) <= 1e-10
    assert abs(rest[:, 0].sum() - float(db)) <= 1e-10 * sc["beta"]
    gw = rest[:, (1 if kernel == COMPLEX else 3):].sum(axis=0)
    assert np.max(np.abs(gw[0::2] + 1j * gw[1::2] - dw.astype(np.complex128).ravel())) <= 1e-10 * sc["w"]


def test_several_rows_of_a_large_solution_take_eight_waves(driver):
    """2804 terms: four waves for one row, whose groups' cotangents through several
    would overflow the registers."""
    d = random_self_energy(6, (5, 6, 2))
    for kernel, waves in ((ADJOINT, 4), (65536, 8)):
        assert f"constexpr int NW = {waves}," in driver(d, "source", kernel, 1)
