"""The block adjoint (large solutions, AUTO: the waves of a block split the
solution of its 64 samples) against the adjoint in passes over a workspace, at
the edges of its blocks and rows: one sample, a block less one, a block, one
more, and a ragged third block; one row (whose group sums make way for their
cotangents at once) and several, beyond the waves of a block; strided rows; the
regulator; values or not.  Both meet 1e-10 of the gradients' rounding scale
against the oracle elsewhere, so they differ by at most twice that."""
import numpy as np
import pytest

from ami_inputs import DEFAULT_Q, complex_energies, k_samples, matsubara_freqs, random_self_energy, real_freqs, uniform_energies
from oracle.evaluate import energies_from_k, term_magnitudes

from parity import gradient_scales, oracle_terms, pole_distance

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
amd = pytest.importorskip("paper_2311_17189_amd")

DEV = "cuda"
BETA, E_REG = 4.0, 0.03


def _case(d, n_e, n_f, seed, momentum):
    """Inputs off the poles (where both sides lose digits), rows and cotangents."""
    terms = oracle_terms(d)
    w = np.concatenate([matsubara_freqs(n_f, BETA)[: (n_f + 1) // 2], real_freqs(n_f, -1.0, 1.0, 0.1)[: n_f // 2]])
    n = 40 * n_e + 400
    x = k_samples(n, d.n_int, seed=seed) if momentum else uniform_energies(n, d.n_eps, seed=seed, a=3.0)
    E = energies_from_k(d.alpha, x, np.array(DEFAULT_Q), 1.0, 0.1) if momentum else x
    keep = np.flatnonzero(pole_distance(terms, d.n_int, E, w, 0.0 if momentum else E_REG).min(axis=0) > 0.02)[:n_e]
    assert len(keep) == n_e
    rng = np.random.default_rng(seed)
    cot = rng.standard_normal((n_f, n_e)) + 1j * rng.standard_normal((n_f, n_e))
    cot_sum = rng.standard_normal(n_f) + 1j * rng.standard_normal(n_f)
    return terms, np.ascontiguousarray(x[keep]), np.ascontiguousarray(E[keep]), w, cot, cot_sum


# 76 terms in 16 groups and 136: two waves per block; 264 and 560: four; 2512
# terms in 224 groups: eight
@pytest.mark.parametrize("order,seed", [(4, (0, 4, 9)), (5, (0, 5, 4)), (5, (0, 5, 0)), (6, (0, 6, 0)), (6, (5, 6, 4))])
@pytest.mark.parametrize("momentum", [False, True], ids=["energies", "momenta"])
def test_block_adjoint_edges(order, seed, momentum):
    d = random_self_energy(order, seed)
    auto, passes = amd.Terms.from_diagram(d), amd.Terms.from_diagram(d)
    passes.set_variant(amd.VARIANT_TWO_PASS)
    for n_e, n_f in [(1, 1), (63, 3), (64, 1), (65, 10), (130, 2)]:
        print(f"block adjoint {seed} momentum {momentum} n_e {n_e} n_f {n_f}", flush=True)
        terms, x, E, w, cot, cot_sum = _case(d, n_e, n_f, (70, order, n_e), momentum)
        wt = torch.from_numpy(w).to(DEV)
        go, gs = torch.from_numpy(cot).to(DEV), torch.from_numpy(cot_sum).to(DEV)
        big = torch.zeros((n_e, x.shape[1] + 3), dtype=torch.float64, device=DEV)
        xt = big[:, 1:1 + x.shape[1]]                       # strided rows, 8-byte aligned
        xt.copy_(torch.from_numpy(x))
        res = []
        for T in (auto, passes):
            out = torch.empty((n_f, n_e), dtype=torch.complex128, device=DEV)
            out_sum = torch.empty((n_f,), dtype=torch.complex128, device=DEV)
            if momentum:
                g = amd.evaluate_hubbard_adjoint(T, xt, DEFAULT_Q, 1.0, 0.1, wt, BETA, grad_out=go, grad_sum=gs,
                                                 out=out, out_sum=out_sum)
                g_x, g_b, g_w = g[0], g[3], g[4]
                bare = amd.evaluate_hubbard_adjoint(T, xt, DEFAULT_Q, 1.0, 0.1, wt, BETA, grad_out=go, grad_sum=gs)
            else:
                g = amd.evaluate_adjoint(T, xt, wt, BETA, E_REG, grad_out=go, grad_sum=gs, out=out, out_sum=out_sum)
                g_x, g_b, g_w = g
                bare = amd.evaluate_adjoint(T, xt, wt, BETA, E_REG, grad_out=go, grad_sum=gs)
            torch.cuda.synchronize()
            assert amd.last_variant() == ("specialized" if T is auto and len(terms) <= 128 else "specialized passes")
            for a, b in zip(g, bare):                       # the same bits without the values
                assert torch.equal(a, b)
            res.append([v.cpu().numpy() for v in (g_x, g_b, g_w, out, out_sum)] +
                       ([g[1].item(), g[2].item()] if momentum else []))
        reg = 0.0 if momentum else E_REG
        full = cot + cot_sum[:, None]
        hub = (d.alpha, x, np.array(DEFAULT_Q), 1.0, 0.1) if momentum else None
        sc = gradient_scales(terms, d.n_int, E, w, BETA, full, reg, hubbard=hub)
        a, b = res
        assert np.max(np.abs(a[0] - b[0]) / np.maximum(sc["k" if momentum else "E"], 1e-300)) <= 2e-10
        assert abs(a[1] - b[1]) <= 2e-10 * sc["beta"]
        assert np.max(np.abs(a[2] - b[2])) <= 2e-10 * sc["w"]
        scale = np.stack([term_magnitudes(terms, d.n_int, E, w[f:f + 1], BETA, reg)[0] for f in range(n_f)])
        assert np.max(np.abs(a[3] - b[3]) / scale) <= 2e-10
        assert np.max(np.abs(a[4] - b[4]) / scale.sum(axis=1)) <= 2e-10
        for name, u, v in zip(("mu", "t"), a[5:], b[5:]):
            assert abs(u - v) <= 2e-10 * sc[name]


@pytest.mark.parametrize("order,seed", [(4, (0, 4, 1)), (5, (0, 5, 0)), (6, (0, 6, 0))])
def test_complex_block_adjoint_edges(order, seed):
    """The same at complex energies: 52 terms (one row only), 264 and 560."""
    d = random_self_energy(order, seed)
    terms = oracle_terms(d)
    auto, passes = amd.Terms.from_diagram(d), amd.Terms.from_diagram(d)
    passes.set_variant(amd.VARIANT_TWO_PASS)
    for n_e, n_f in [(1, 1), (63, 3), (64, 1), (65, 10), (130, 1)]:
        print(f"complex block adjoint {seed} n_e {n_e} n_f {n_f}", flush=True)
        w = np.concatenate([matsubara_freqs(n_f, BETA)[: (n_f + 1) // 2], real_freqs(n_f, -1.0, 1.0, 0.1)[: n_f // 2]])
        E = complex_energies(40 * n_e + 400, d.n_eps, seed=(71, order, n_e), a=3.0, eta=0.25 / (BETA * d.n_int))
        E = E[np.flatnonzero(pole_distance(terms, d.n_int, E, w, E_REG).min(axis=0) > 0.02)[:n_e]]
        assert len(E) == n_e
        rng = np.random.default_rng(n_e)
        cot = rng.standard_normal((n_f, n_e)) + 1j * rng.standard_normal((n_f, n_e))
        big = torch.zeros((n_e, d.n_eps + 2), dtype=torch.complex128, device=DEV)
        Et = big[:, 1:1 + d.n_eps]
        Et.copy_(torch.from_numpy(E))
        wt, go = torch.from_numpy(w).to(DEV), torch.from_numpy(cot).to(DEV)
        res = []
        for T in (auto, passes):
            out = torch.empty((n_f, n_e), dtype=torch.complex128, device=DEV)
            out_sum = torch.empty((n_f,), dtype=torch.complex128, device=DEV)
            g = amd.evaluate_complex_adjoint(T, Et, wt, BETA, E_REG, grad_out=go, out=out, out_sum=out_sum)
            again = amd.evaluate_complex_adjoint(T, Et, wt, BETA, E_REG, grad_out=go)
            torch.cuda.synchronize()
            for a, b in zip(g, again):
                assert torch.equal(a, b)
            res.append([v.cpu().numpy() for v in (*g, out, out_sum)])
        a, b = res
        sc = gradient_scales(terms, d.n_int, E, w, BETA, cot, E_REG)
        assert np.max(np.abs(a[0] - b[0]) / np.maximum(sc["E"], 1e-300)) <= 2e-10
        assert abs(a[1] - b[1]) <= 2e-10 * sc["beta"]
        assert np.max(np.abs(a[2] - b[2])) <= 2e-10 * sc["w"]
        scale = np.stack([term_magnitudes(terms, d.n_int, E, w[f:f + 1], BETA, E_REG)[0] for f in range(n_f)])
        assert np.max(np.abs(a[3] - b[3]) / scale) <= 2e-10
        assert np.max(np.abs(a[4] - b[4]) / scale.sum(axis=1)) <= 2e-10
