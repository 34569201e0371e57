"""The block forward (large solutions, AUTO: the waves of a block split the
group sums of its 64 samples, then take whole rows) against the two passes over
a workspace, at the edges of its blocks, rows and row parts.  Both meet 1e-10 of
the values' rounding scale against the oracle elsewhere, so they differ by at
most twice that."""
import numpy as np
import pytest

from ami_inputs import DEFAULT_Q, k_samples, matsubara_freqs, random_self_energy, real_freqs, uniform_energies
from oracle.evaluate import energies_from_k, term_magnitudes

from parity import oracle_terms, pole_distance

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
amd = pytest.importorskip("paper_2311_17189_amd")

DEV = "cuda"
BETA, E_REG = 4.0, 0.03


# 560 terms: four waves per block; 2512 terms in 224 groups: eight
@pytest.mark.parametrize("seed", [(0, 6, 0), (5, 6, 4)])
@pytest.mark.parametrize("momentum", [False, True], ids=["energies", "momenta"])
def test_block_forward_edges(seed, momentum):
    d = random_self_energy(6, seed)
    terms = oracle_terms(d)
    auto, passes = amd.Terms.from_diagram(d), amd.Terms.from_diagram(d)
    passes.set_variant(amd.VARIANT_TWO_PASS)
    # one row; rows for some of the waves; a wave's second row; parts, the last of one row
    for n_e, n_f in [(1, 1), (63, 3), (64, 9), (65, 1), (130, 41)]:
        print(f"block forward {seed} momentum {momentum} n_e {n_e} n_f {n_f}", flush=True)
        w = np.concatenate([matsubara_freqs(n_f, BETA)[: (n_f + 1) // 2], real_freqs(n_f, -1.0, 1.0, 0.1)[: n_f // 2]])
        n = 40 * n_e + 400
        x = k_samples(n, d.n_int, seed=(72, n_e)) if momentum else uniform_energies(n, d.n_eps, seed=(72, n_e), a=3.0)
        E = energies_from_k(d.alpha, x, np.array(DEFAULT_Q), 1.0, 0.1) if momentum else x
        reg = 0.0 if momentum else E_REG
        keep = np.flatnonzero(pole_distance(terms, d.n_int, E, w, reg).min(axis=0) > 0.02)[:n_e]
        assert len(keep) == n_e
        big = torch.zeros((n_e, x.shape[1] + 3), dtype=torch.float64, device=DEV)
        xt = big[:, 1:1 + x.shape[1]]                       # strided rows, 8-byte aligned
        xt.copy_(torch.from_numpy(np.ascontiguousarray(x[keep])))
        wt = torch.from_numpy(w).to(DEV)
        res = []
        for T in (auto, passes):
            if momentum:
                call = lambda **kw: amd.evaluate_hubbard(T, xt, DEFAULT_Q, 1.0, 0.1, wt, BETA, **kw)
            else:
                call = lambda **kw: amd.evaluate(T, xt, wt, BETA, E_REG, **kw)
            out, out_sum = call(want_sum=True)
            bare, _ = call()
            _, only = call(want_out=False, want_sum=True)
            torch.cuda.synchronize()
            assert amd.last_variant() == "specialized two-pass"
            assert torch.equal(out, bare) and torch.equal(out_sum, only)
            res.append((out.cpu().numpy(), out_sum.cpu().numpy()))
        scale = np.stack([term_magnitudes(terms, d.n_int, E[keep], w[f:f + 1], BETA, reg)[0] for f in range(n_f)])
        a, b = res
        assert np.max(np.abs(a[0] - b[0]) / scale) <= 2e-10
        assert np.max(np.abs(a[1] - b[1]) / scale.sum(axis=1)) <= 2e-10


def test_more_samples_than_a_grid_holds():
    """Eight waves for 64 samples: past 8388607 blocks one launch has no grid,
    and the samples go in several."""
    d = random_self_energy(6, (5, 6, 4))
    T = amd.Terms.from_diagram(d)
    n = 64 * 8388607 + 100
    if torch.cuda.mem_get_info()[0] < 24 * n + (1 << 30):
        pytest.skip("not enough memory")
    flat = torch.empty(n + d.n_eps, dtype=torch.float64, device=DEV).uniform_(-3.0, 3.0)
    x = flat.as_strided((n, d.n_eps), (1, 1))               # overlapping rows: 8 bytes a sample
    w = torch.from_numpy(matsubara_freqs(1, BETA)).to(DEV)
    out, _ = amd.evaluate(T, x, w, BETA)
    for lo in (0, n - 200):
        part, _ = amd.evaluate(T, x[lo:lo + 200].clone(), w, BETA)
        torch.cuda.synchronize()
        assert torch.equal(torch.view_as_real(out[:, lo:lo + 200]), torch.view_as_real(part))
