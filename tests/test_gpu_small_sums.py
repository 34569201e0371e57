"""Small calls have the kernel's last block add the partial sums instead of a
second launch.  Under capture the second launch stays, so a graph's replays give
the oracle for every sum and scalar gradient: the same bits, at the edges of
waves and blocks, at and past the limits, call after call on one stream, and on
two streams at once."""
import numpy as np
import pytest

from ami_inputs import complex_energies, k_samples, matsubara_freqs, random_self_energy, uniform_energies

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
amd = pytest.importorskip("paper_2311_17189_amd")

DEV = "cuda"
BETA = 4.0
SIZES = [(1, 1), (64, 2), (65, 1), (256, 3), (257, 1), (1025, 4), (2048, 1), (2049, 9), (4096, 2), (16385, 1),
         (40960, 1), (40961, 2), (65536, 1), (65537, 1)]


def _calls(kind, seed, order):
    d = random_self_energy(order, seed)
    T = amd.Terms.from_diagram(d)
    out = []
    for n_e, n_f in SIZES:
        w = torch.from_numpy(matsubara_freqs(n_f, BETA)).to(DEV)
        rng = np.random.default_rng(n_e)
        gs = torch.from_numpy(rng.standard_normal(n_f) + 1j * rng.standard_normal(n_f)).to(DEV)
        s = torch.empty((n_f,), dtype=torch.complex128, device=DEV)
        if kind == "momenta":
            x = torch.from_numpy(k_samples(n_e, d.n_int, seed=90)).to(DEV)
            out.append(lambda x=x, w=w, s=s: amd.evaluate_hubbard(T, x, [0.3, -1.1], 1.0, 0.1, w, BETA, want_sum=True,
                                                                  out_sum=s))
            out.append(lambda x=x, w=w, s=s, gs=gs: amd.evaluate_hubbard_adjoint(
                T, x, [0.3, -1.1], 1.0, 0.1, w, BETA, grad_sum=gs, out_sum=s)[1:] + (s,))
        elif kind == "energies":
            x = torch.from_numpy(uniform_energies(n_e, d.n_eps, seed=91, a=3.0)).to(DEV)
            out.append(lambda x=x, w=w, s=s: amd.evaluate(T, x, w, BETA, 0.03, want_sum=True, out_sum=s))
            out.append(lambda x=x, w=w, gs=gs: amd.evaluate_adjoint(T, x, w, BETA, 0.03, grad_sum=gs))
        else:
            x = torch.from_numpy(complex_energies(n_e, d.n_eps, seed=92, a=3.0, eta=0.02)).to(DEV)
            out.append(lambda x=x, w=w, s=s: amd.evaluate_complex(T, x, w, BETA, 0.03, want_sum=True, out_sum=s))
            out.append(lambda x=x, w=w, s=s, gs=gs: amd.evaluate_complex_adjoint(T, x, w, BETA, 0.03, grad_sum=gs,
                                                                                 out_sum=s) + (s,))
    return out


def _bits(res):
    return [torch.view_as_real(v).clone() if v.is_complex() else v.clone() for v in res if v is not None]


@pytest.mark.parametrize("kind", ["momenta", "energies", "complex"])
@pytest.mark.parametrize("order,seed", [(2, (0, 2, 0)), (4, (0, 4, 1)), (6, (0, 6, 0))])
def test_sums_of_small_calls(kind, order, seed):
    calls = _calls(kind, seed, order)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    got = [[], []]
    torch.cuda.synchronize()
    for s in streams:                            # every call sizes its workspace before the captures
        with torch.cuda.stream(s):
            for f in calls:
                f()
    torch.cuda.synchronize()
    for f in calls:
        with torch.cuda.stream(streams[0]):
            got[0].append(_bits(f()))
    torch.cuda.synchronize()
    for f in reversed(calls):                    # in another order, on the other stream
        with torch.cuda.stream(streams[1]):
            got[1].insert(0, _bits(f()))
    torch.cuda.synchronize()
    for i, f in enumerate(calls):
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=streams[0]):
            res = f()
        for _ in range(2):
            graph.replay()
            torch.cuda.synchronize()
            want = _bits(res)
            for side in got:
                assert len(want) == len(side[i]) >= 2
                for a, b in zip(side[i], want):
                    assert torch.equal(a, b), (kind, order, SIZES[i // 2], i % 2)
            with torch.cuda.stream(streams[1]):
                f()
            torch.cuda.synchronize()


def test_two_streams_at_once():
    """One handle on two streams, calls interleaved: each stream has its own count."""
    d = random_self_energy(4, (0, 4, 1))
    T = amd.Terms.from_diagram(d)
    w = torch.from_numpy(matsubara_freqs(2, BETA)).to(DEV)
    xs = [torch.from_numpy(k_samples(n, d.n_int, seed=93)).to(DEV) for n in (300, 8192, 20000)]
    call = lambda x: amd.evaluate_hubbard(T, x, [0.3, -1.1], 1.0, 0.1, w, BETA, want_out=False, want_sum=True)[1]
    want = [call(x) for x in xs]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    got = []
    for rep in range(100):
        for s in streams:
            with torch.cuda.stream(s):
                got.append((rep % 3, call(xs[rep % 3])))
    torch.cuda.synchronize()
    for i, v in got:
        assert torch.equal(torch.view_as_real(v), torch.view_as_real(want[i]))
