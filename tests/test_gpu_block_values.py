"""Values of the real adjoint at up to 128 terms on the block kernel (solutions
whose one-pass adjoint spills): the forward's bit for bit on the energy input,
and the row sums those of the one-pass adjoint."""
import pytest

from ami_inputs import matsubara_freqs, random_self_energy, real_freqs, uniform_energies

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
np = pytest.importorskip("numpy")
amd = pytest.importorskip("paper_2311_17189_amd")

DEV = "cuda"
BETA = 5.0


# 76, 82 and 112 terms
@pytest.mark.parametrize("order,seed", [(4, (0, 4, 9)), (4, (0, 4, 25)), (5, (0, 5, 14))])
def test_values_are_the_forwards(order, seed):
    d = random_self_energy(order, seed)
    T, one_pass = amd.Terms.from_diagram(d), amd.Terms.from_diagram(d)
    one_pass.set_variant(amd.VARIANT_SPECIALIZED)
    for n_e, n_f in [(1, 1), (63, 3), (64, 1), (130, 2), (5001, 1), (3000, 5)]:
        print(f"block values {seed} n_e {n_e} n_f {n_f}", flush=True)
        w = np.concatenate([matsubara_freqs(n_f, BETA)[: (n_f + 1) // 2], real_freqs(n_f, -1.0, 1.0, 0.1)[: n_f // 2]])
        E = torch.from_numpy(uniform_energies(n_e, d.n_eps, seed=(72, order, n_e), a=4.0)).to(DEV)
        wt = torch.from_numpy(w).to(DEV)
        gs = torch.ones(n_f, dtype=torch.complex128, device=DEV)
        want, _ = amd.evaluate(T, E, wt, BETA, 1e-3, want_sum=True)
        res = []
        for t in (T, one_pass):
            out = torch.empty((n_f, n_e), dtype=torch.complex128, device=DEV)
            out_sum = torch.empty((n_f,), dtype=torch.complex128, device=DEV)
            amd.evaluate_adjoint(t, E, wt, BETA, 1e-3, grad_sum=gs, out=out, out_sum=out_sum)
            assert torch.equal(torch.view_as_real(out), torch.view_as_real(want))
            res.append(out_sum)
        assert torch.equal(torch.view_as_real(res[0]), torch.view_as_real(res[1]))
