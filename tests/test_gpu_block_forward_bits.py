"""The block forward's values and row sums are those of the two passes over a
workspace bit for bit (the persistent batch, which runs the passes' tile
functions, equals an AUTO call by it)."""
import pytest

from ami_inputs import DEFAULT_Q, k_samples, matsubara_freqs, random_self_energy, uniform_energies

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
amd = pytest.importorskip("paper_2311_17189_amd")

DEV = "cuda"
BETA = 4.0


# four waves per block and eight; one row, several rows of a wave, several row parts
@pytest.mark.parametrize("seed", [(0, 6, 0), (5, 6, 4)])
@pytest.mark.parametrize("momentum", [False, True], ids=["energies", "momenta"])
def test_bits_of_the_passes(seed, momentum):
    d = random_self_energy(6, seed)
    auto, passes = amd.Terms.from_diagram(d), amd.Terms.from_diagram(d)
    passes.set_variant(amd.VARIANT_TWO_PASS)
    for n_e, n_f in [(1, 1), (63, 3), (64, 9), (65, 1), (130, 41), (20000, 5), (70001, 1)]:
        print(f"block forward bits {seed} momentum {momentum} n_e {n_e} n_f {n_f}", flush=True)
        w = torch.from_numpy(matsubara_freqs(n_f, BETA)).to(DEV)
        x = k_samples(n_e, d.n_int, seed=(76, n_e)) if momentum else uniform_energies(n_e, d.n_eps, seed=(76, n_e), a=3.0)
        x = torch.from_numpy(x).to(DEV)
        res = [amd.evaluate_hubbard(T, x, DEFAULT_Q, 1.0, 0.1, w, BETA, want_sum=True) if momentum
               else amd.evaluate(T, x, w, BETA, 0.03, want_sum=True) for T in (auto, passes)]
        for a, b in zip(*res):
            assert torch.equal(torch.view_as_real(a), torch.view_as_real(b))
