"""AUTO names a fallback from a block kernel, so a call whose name carries no
note ran it: with another kernel's code object in the block kernel's place in
the disk cache (its entry is then missing), the passes serve the call and
amiLastVariant says why."""
import shutil

import pytest

from ami_inputs import DEFAULT_Q, complex_energies, k_samples, matsubara_freqs, random_self_energy

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
amd = pytest.importorskip("paper_2311_17189_amd")

DEV = "cuda"
BETA = 5.0
BLOCK = {"forward": 32768, "adjoint": 8192, "complex": 16384}


# 560 terms: the forward's two passes, the adjoint in passes; 264: one pass at complex energies
@pytest.mark.parametrize("path,order,seed,name", [("forward", 6, (0, 6, 0), "specialized two-pass"),
                                                  ("adjoint", 6, (0, 6, 0), "specialized passes"),
                                                  ("complex", 5, (0, 5, 0), "specialized complex")])
def test_fallback_is_named(path, order, seed, name, tmp_path, monkeypatch):
    monkeypatch.setenv("AMIGPU_CACHE_DIR", str(tmp_path))
    d = random_self_energy(order, seed)
    w = torch.from_numpy(matsubara_freqs(1, BETA)).to(DEV)
    gs = torch.ones(1, dtype=torch.complex128, device=DEV)
    k = torch.from_numpy(k_samples(200, d.n_int, seed=(74, order))).to(DEV)
    E = torch.from_numpy(complex_energies(200, d.n_eps, seed=(75, order), a=3.0, eta=0.25 / (BETA * d.n_int))).to(DEV)

    def run(T):
        if path == "forward":
            return amd.evaluate_hubbard(T, k, DEFAULT_Q, 1.0, 0.0, w, BETA, want_sum=True)
        if path == "adjoint":
            return amd.evaluate_hubbard_adjoint(T, k, DEFAULT_Q, 1.0, 0.0, w, BETA, grad_sum=gs)
        return amd.evaluate_complex_adjoint(T, E, w, BETA, grad_sum=gs)

    run(amd.Terms.from_diagram(d))
    assert amd.last_variant() == name
    (block,) = [f for f in tmp_path.glob("*.hip") if f"#define AMI_JIT_KERNELS {BLOCK[path]}\n" in f.read_text()]
    forced = amd.Terms.from_diagram(d)
    forced.set_variant(amd.VARIANT_SPECIALIZED if path == "complex" else amd.VARIANT_TWO_PASS)
    want = run(forced)
    other = [f for f in tmp_path.glob("*.hsaco") if f.stem != block.stem][0]
    shutil.copy(other, block.with_suffix(".hsaco"))
    got = run(amd.Terms.from_diagram(d))
    assert amd.last_variant().startswith(name + " (not in a block: ")
    for a, b in zip(got, want):
        assert torch.equal(a, b)
