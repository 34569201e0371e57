"""The adjoint at complex energies under capture where the number of frequency
rows chooses between the one-pass and the block kernel: after an eager call with
one number of rows, a captured call with another is served by the kernel that
is loaded (nothing is compiled), and its replays equal the oracle-checked eager
results up to rounding."""
import pytest

from ami_inputs import complex_energies, matsubara_freqs, random_self_energy

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
amd = pytest.importorskip("paper_2311_17189_amd")

DEV = "cuda"
BETA = 5.0


@pytest.mark.parametrize("eager_rows,rows", [(4, 1), (1, 4)])
def test_captured_rows_after_other_rows(eager_rows, rows, tmp_path, monkeypatch):
    monkeypatch.setenv("AMIGPU_CACHE_DIR", str(tmp_path))
    d = random_self_energy(4, (0, 4, 1))            # 52 terms
    T, ref = amd.Terms.from_diagram(d), amd.Terms.from_diagram(d)
    n = 500
    E = torch.from_numpy(complex_energies(4 * n, d.n_eps, seed=(77, 4), a=3.0, eta=0.25 / (BETA * d.n_int))).to(DEV)
    w = torch.from_numpy(matsubara_freqs(4, BETA)).to(DEV)
    gs = torch.ones(4, dtype=torch.complex128, device=DEV)

    def call(terms, e, f, **kw):
        return amd.evaluate_complex_adjoint(terms, e, w[:f], BETA, grad_sum=gs[:f], **kw)

    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        call(T, E, eager_rows)                      # more samples: sizes the stream's workspace
    stream.synchronize()
    before = sorted(f.name for f in tmp_path.iterdir())
    x = E[:n].clone()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        got = call(T, x, rows)
    assert sorted(f.name for f in tmp_path.iterdir()) == before
    for r in range(3):
        x.copy_(E[r * n:(r + 1) * n])
        graph.replay()
        torch.cuda.synchronize()
        for a, b in zip(got, call(ref, x.clone(), rows)):
            assert torch.allclose(a, b, rtol=1e-9, atol=1e-9 * float(b.abs().max()))
