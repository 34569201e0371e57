"""The recorded launches of a batch form a chain, two branches or four, by their
work: every output and row sum must be the per-diagram call's, bit for bit,
replay after replay, also with fewer items than streams."""
import pytest

from ami_inputs import DEFAULT_Q, k_samples, matsubara_freqs, random_self_energy

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
amd = pytest.importorskip("paper_2311_17189_amd")

DEV = "cuda"
BETA = 5.0


# (orders of the items, samples, rows): chains, two branches, four
@pytest.mark.parametrize("orders,n_e,n_f", [((2,), 100, 1), ((2, 3), 1000, 3), ((2, 3, 4), 257, 4), ((2, 3, 4, 5, 6), 2000, 2),
                                            ((4, 5), 200001, 16), ((3, 4, 5), 120000, 16), ((2, 3, 4, 5, 6), 50000, 16),
                                            ((4, 5), 1000000, 16), ((4, 5, 5, 6, 6), 300001, 16)])
def test_branches_equal_per_diagram_calls(orders, n_e, n_f):
    items = []
    for i, order in enumerate(orders):
        d = random_self_energy(order, (0, order, i))
        T = amd.Terms.from_diagram(d)
        items.append({"terms": T, "ext_freqs": torch.from_numpy(matsubara_freqs(n_f, BETA)).to(DEV), "beta": BETA,
                      "k": torch.from_numpy(k_samples(n_e, d.n_int, seed=(95, i))).to(DEV), "q": list(DEFAULT_Q), "t": 1.0,
                      "mu": 0.05, "out": torch.empty((n_f, n_e), dtype=torch.complex128, device=DEV),
                      "out_sum": torch.empty((n_f,), dtype=torch.complex128, device=DEV)})
    want = [amd.evaluate_hubbard(it["terms"], it["k"], it["q"], it["t"], it["mu"], it["ext_freqs"], BETA, want_sum=True)
            for it in items]
    b = amd.Batch(items)
    assert b.info()["specialized_items"] == len(items)
    for _ in range(3):
        for it in items:
            it["out"].zero_()
            it["out_sum"].zero_()
        b.run()
        torch.cuda.synchronize()
        for it, (out, out_sum) in zip(items, want):
            assert torch.equal(torch.view_as_real(it["out"]), torch.view_as_real(out))
            assert torch.equal(torch.view_as_real(it["out_sum"]), torch.view_as_real(out_sum))
