"""The generated sources of the block kernels on the CPU: the code generator
under AddressSanitizer and UndefinedBehaviorSanitizer
(tests/cpu_math/block_source.cpp)."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from ami_inputs import random_self_energy

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
