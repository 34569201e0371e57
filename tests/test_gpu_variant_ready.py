"""The kernels a forced variant takes in place of AUTO's block kernels are ready
after amiSetVariant, whether amiTermsSpecialize or an AUTO call made the block
kernels ready before: the allocation-free adjoint, which loads nothing, is
served and equals the ordinary entry point."""
import pytest

from ami_inputs import DEFAULT_Q, k_samples, matsubara_freqs, random_self_energy

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
amd = pytest.importorskip("paper_2311_17189_amd")

DEV = "cuda"
BETA = 5.0


@pytest.mark.parametrize("specialize", [True, False], ids=["specialized", "called"])
# 136 terms: the adjoint in passes; 76: in one pass
@pytest.mark.parametrize("order,seed,variant", [(5, (0, 5, 4), "TWO_PASS"), (4, (0, 4, 9), "SPECIALIZED")])
def test_no_alloc_after_a_change_of_variant(order, seed, variant, specialize):
    d = random_self_energy(order, seed)
    T = amd.Terms.from_diagram(d)
    T.upload()
    k = torch.from_numpy(k_samples(300, d.n_int, seed=(73, order))).to(DEV)
    w = torch.from_numpy(matsubara_freqs(2, BETA)).to(DEV)
    gs = torch.ones(2, dtype=torch.complex128, device=DEV)
    if specialize:
        T.specialize(True)
    else:
        amd.evaluate_hubbard_adjoint(T, k, DEFAULT_Q, 1.0, 0.0, w, BETA, grad_sum=gs)
    T.set_variant(getattr(amd, "VARIANT_" + variant))
    got = amd.evaluate_hubbard_adjoint_no_alloc(T, k, DEFAULT_Q, 1.0, 0.0, w, BETA, grad_sum=gs)
    want = amd.evaluate_hubbard_adjoint(T, k, DEFAULT_Q, 1.0, 0.0, w, BETA, grad_sum=gs)
    for a, b in zip(got, want):
        assert torch.equal(a, b)
