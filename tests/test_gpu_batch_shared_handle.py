"""A batch whose items share one handle (one diagram at several temperatures,
chemical potentials, external momenta, sample counts and rows): every item's
values and row sums must be its own per-diagram call's, bit for bit, replay
after replay, also when the inputs change between the replays."""
import pytest

from ami_inputs import DEFAULT_Q, k_samples, matsubara_freqs, random_self_energy, uniform_energies

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
amd = pytest.importorskip("paper_2311_17189_amd")

DEV = "cuda"
# (samples, rows) of the items: growing, shrinking and equal partial sums
SIZES = {6: [(100, 1), (5000, 3), (700, 8), (700, 8), (20011, 2), (64, 1)],
         9: [(3000, 4), (257, 2), (9001, 1), (65, 16), (12000, 5), (3000, 4), (1, 1), (513, 3), (40000, 2)]}


# 52 terms: one pass; 2804 terms: block forward
@pytest.mark.parametrize("order,seed", [(4, (0, 4, 1)), (6, (5, 6, 0))])
@pytest.mark.parametrize("n_items", [6, 9])
@pytest.mark.parametrize("momentum", [True, False], ids=["momenta", "energies"])
def test_items_of_one_handle(order, seed, n_items, momentum):
    d = random_self_energy(order, seed)
    T = amd.Terms.from_diagram(d)
    items, inputs = [], []
    for i, (n_e, n_f) in enumerate(SIZES[n_items]):
        beta = 3.0 + 0.5 * i
        it = {"terms": T, "ext_freqs": torch.from_numpy(matsubara_freqs(n_f, beta)).to(DEV), "beta": beta,
              "out": torch.empty((n_f, n_e), dtype=torch.complex128, device=DEV),
              "out_sum": torch.empty((n_f,), dtype=torch.complex128, device=DEV)}
        if momentum:
            x = [k_samples(n_e, d.n_int, seed=(97, i, r)) for r in range(3)]
            it.update(q=[q + 0.1 * i for q in DEFAULT_Q], t=1.0, mu=0.05 * i)
            it["k"] = torch.from_numpy(x[0]).to(DEV)
        else:
            x = [uniform_energies(n_e, d.n_eps, seed=(98, i, r), a=4.0) for r in range(3)]
            it["energies"] = torch.from_numpy(x[0]).to(DEV)
        items.append(it)
        inputs.append([torch.from_numpy(v).to(DEV) for v in x])
    b = amd.Batch(items)
    assert b.info()["specialized_items"] == n_items
    for r in range(3):
        for it, x in zip(items, inputs):
            (it["k"] if momentum else it["energies"]).copy_(x[r])
            it["out"].zero_()
            it["out_sum"].zero_()
        b.run()
        torch.cuda.synchronize()
        for i, it in enumerate(items):
            if momentum:
                out, out_sum = amd.evaluate_hubbard(T, it["k"], it["q"], it["t"], it["mu"], it["ext_freqs"], it["beta"],
                                                    want_sum=True)
            else:
                out, out_sum = amd.evaluate(T, it["energies"], it["ext_freqs"], it["beta"], want_sum=True)
            assert torch.equal(torch.view_as_real(it["out"]), torch.view_as_real(out)), (r, i)
            assert torch.equal(torch.view_as_real(it["out_sum"]), torch.view_as_real(out_sum)), (r, i)
