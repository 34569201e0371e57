"""Truncation errors of the polynomials of device_common.hpp, evaluated exactly
with the coefficients as they stand there, within the bounds its comments
state; the errors of a leaf's slope over its arguments; the complex leaf at the
largest imaginary arguments its entry points admit."""
import math
import os
import random
import re
import shutil
import subprocess

import pytest

mp = pytest.importorskip("mpmath")

HERE = os.path.dirname(os.path.abspath(__file__))
HEADER = os.path.join(os.path.dirname(HERE), "paper_2311_17189_amd", "csrc", "device_common.hpp")
mp.mp.prec = 200


def _coefficients(name, first):
    """The Horner coefficients (highest power first) of variable `name` in the
    function whose body starts at `first`."""
    text = open(HEADER).read()
    text = text[text.index(first):]
    text = text[:text.index("\n}\n")]
    num = r"(-?0x[0-9a-f.]+p[+-]\d+|-?0\.5)"
    out = re.findall(rf"\b{name} = {num};", text) + re.findall(rf"\b{name} = fma\({name}, \w+, {num}\);", text)
    return [mp.mpf(float.fromhex(c) if "x" in c else float(c)) for c in out]


def _grid(a, b):
    return [mp.mpf(a) + (mp.mpf(b) - a) * i / 3000 for i in range(3001)]


def _log2_max(errors):
    return float(mp.log(max(abs(e) for e in errors), 2))


def test_cos_of_half_pi():
    p = _coefficients("p", "double cos_red(double x)")
    assert len(p) == 8
    assert _log2_max(mp.cos(r) - (1 + r * r * mp.polyval(p, r * r)) for r in _grid(0, mp.pi / 2)) < -57.2


def test_sin_and_cos_of_quarter_pi():
    s, c = (_coefficients(n, "void sincos_cosm1(double x") for n in ("ps", "pc"))
    assert len(s) == 6 and len(c) == 7
    xs = _grid(mp.mpf(2) ** -20, mp.pi / 4)
    assert _log2_max(mp.sin(r) - r * (1 + r * r * mp.polyval(s, r * r)) for r in xs) < -59.1
    assert _log2_max(mp.cos(r) - (1 + r * r * mp.polyval(c, r * r)) for r in xs) < -63.9


def test_exp():
    q = _coefficients("q", "void exp_reduce(double z")
    assert len(q) == 10
    xs = [r for r in _grid(-mp.log(2) / 2, mp.log(2) / 2) if abs(r) > mp.mpf(2) ** -20]
    assert _log2_max((mp.expm1(r) - r * (1 + r * mp.polyval(q, r))) / mp.expm1(r) for r in xs) < -55.5
    assert _log2_max((mp.exp(r) - 1 - r * (1 + r * mp.polyval(q, r))) / mp.exp(r) for r in xs) < -56.8


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    out = str(tmp_path_factory.mktemp("math") / "math_check")
    subprocess.run([cxx, "-O1", "-std=c++17", "-ffp-contract=off", "-I", os.path.join(HERE, "cpu_math", "shim"),
                    os.path.join(HERE, "cpu_math", "math_check.cpp"), "-o", out], check=True, capture_output=True)
    return out


def _run(exe, what, lines):
    res = subprocess.run([exe, what], input="\n".join(lines) + "\n", capture_output=True, text=True, check=True)
    return [[float(v) for v in l.split()] for l in res.stdout.splitlines()]


# the errors (rms, units of 2^-53) of the form by e^-|y| with selections by the sign of y
@pytest.mark.parametrize("kind,sigma,bound", [("u", 1, 1.37), ("v", -1, 1.29)])
def test_slope_is_as_accurate_as_the_form_before(exe, kind, sigma, bound):
    rng = random.Random(5)
    ys = [math.exp(rng.uniform(math.log(1e-8), math.log(600.0))) * rng.choice((-1, 1)) for _ in range(8000)]
    mp.mp.prec = 120
    total = 0.0
    for y, (_, dv) in zip(ys, _run(exe, kind, [repr(y) for y in ys])):
        e = mp.exp(mp.mpf(y))
        want = -e / (1 + e) ** 2 if sigma > 0 else e / mp.expm1(mp.mpf(y)) ** 2
        total += float((dv - want) / want * 2 ** 53) ** 2
    assert math.sqrt(total / len(ys)) <= bound


# relative to |f|, as for small arguments: a few ulp of the parts, and of Im y's sine and cosine
@pytest.mark.parametrize("kind,sigma", [("F", 1), ("B", -1)])
def test_complex_leaf_at_large_imaginary_arguments(exe, kind, sigma):
    rng = random.Random(6)
    args = [(rng.uniform(-20, 20), rng.choice((-1, 1)) * rng.uniform(1e6, 6e6)) for _ in range(2000)]
    mp.mp.prec = 160
    for (yr, yi), (fr, fi) in zip(args, _run(exe, kind, [f"{a!r} {b!r}" for a, b in args])):
        d = sigma * mp.exp(mp.mpc(yr, yi)) + 1
        if abs(d) < 0.05:                   # next to a pole of the leaf the argument's rounding counts
            continue
        want = 1 / d
        assert abs(mp.mpc(fr, fi) - want) <= 16 * mp.mpf(2) ** -53 * abs(want) * max(1, 1 / abs(d)), (yr, yi)
