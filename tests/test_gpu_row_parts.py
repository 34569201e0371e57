"""The one-pass forwards split the frequency rows of few samples over blocks:
every row's values must be those of a call with that row alone, whatever the
number of parts (none below four rows, several for few samples, an odd last
part), and the row sums the sums of the values."""
import numpy as np
import pytest

from ami_inputs import complex_energies, k_samples, matsubara_freqs, random_self_energy, real_freqs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
amd = pytest.importorskip("paper_2311_17189_amd")

DEV = "cuda"


@pytest.mark.parametrize("n_e,n_f", [(1, 3), (1, 4), (257, 37), (5000, 16), (70000, 100), (300000, 40)])
@pytest.mark.parametrize("cplx", [False, True], ids=["momenta", "complex"])
def test_rows_equal_single_row_calls(n_e, n_f, cplx):
    d = random_self_energy(3, (0, 3, 6))
    T = amd.Terms.from_diagram(d)
    beta = 4.0
    w = np.concatenate([matsubara_freqs(n_f, beta)[: n_f // 2], real_freqs(n_f, -3.0, 3.0, 0.05)[: n_f - n_f // 2]])
    wt = torch.from_numpy(w).to(DEV)
    if cplx:
        x = torch.from_numpy(complex_energies(n_e, d.n_eps, seed=80, a=3.0, eta=0.02)).to(DEV)
        call = lambda ww: amd.evaluate_complex(T, x, ww, beta, want_sum=True)
    else:
        x = torch.from_numpy(k_samples(n_e, d.n_int, seed=81)).to(DEV)
        call = lambda ww: amd.evaluate_hubbard(T, x, [0.3, -1.1], 1.0, 0.1, ww, beta, want_sum=True)
    out, out_sum = call(wt)
    again, again_sum = call(wt)
    torch.cuda.synchronize()
    assert torch.equal(out, again) and torch.equal(out_sum, again_sum)
    for f in sorted({0, 1, n_f // 2, n_f - 2, n_f - 1}):
        one, _ = call(wt[f:f + 1])
        torch.cuda.synchronize()
        assert torch.equal(one[0], out[f]), f
    scale = out.abs().sum(dim=1)
    assert torch.all((out.sum(dim=1) - out_sum).abs() <= 1e-13 * scale)
