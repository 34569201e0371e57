"""What amiTermsSpecialize compiles ahead for a handle whose variant was set
before, read from the disk cache (the compilation needs no device)."""
import subprocess
import sys

import pytest

pytest.importorskip("paper_2311_17189_amd")

CODE = """
import sys
import paper_2311_17189_amd as amd
from ami_inputs import random_self_energy
T = amd.Terms.from_diagram(random_self_energy(int(sys.argv[1]), eval(sys.argv[2])))
T.set_variant(getattr(amd, "VARIANT_" + sys.argv[3]))
try:
    T.specialize(False)
except amd.AmiError:        # without a device it ends at the load
    pass
"""


# 264 terms, energies: kernel 256 is the one-pass adjoint at complex energies, 128 the real
# adjoint's leaf pass
@pytest.mark.parametrize("variant,ahead", [("SPECIALIZED", 256), ("TWO_PASS", 128)])
def test_forced_variants_kernels_are_compiled_ahead(tmp_path, variant, ahead):
    import os
    env = dict(os.environ, AMIGPU_CACHE_DIR=str(tmp_path),
               PYTHONPATH=os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
    subprocess.run([sys.executable, "-c", CODE, "5", "(0, 5, 0)", variant], check=True, env=env)
    kernels = set()
    for f in tmp_path.glob("*.hip"):
        text = f.read_text()
        at = text.index("#define AMI_JIT_KERNELS ") + 24
        kernels.add(int(text[at:text.index("\n", at)]))
    assert {8192, 16384, ahead} <= kernels
