"""The evaluations that programs built on this framework spend their time in,
as cases that can be timed: forward values, value-and-gradient steps, complex
energies, Monte-Carlo integration and mixed batches of self-energy diagrams,
from a few hundred samples to the largest batches in use.

Diagrams are order-2 to order-6 self-energies of the Hubbard model, given by
their label rows (one propagator per word, '+', '-' or '0' per frequency slot,
the external frequency last).  Inputs are momenta uniform in the Brillouin
zone or energies uniform around the Fermi level, as a Monte-Carlo integrator
draws them.

``exact`` evaluates the same solution from its residues in plain torch float64
arithmetic, term by term, with gradients by torch's autograd.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import paper_2311_17189_amd as amd
from paper_2311_17189_amd.autograd import AmiEvaluate

TOPOLOGIES = {
    "order2": "+00 0+0 -++",
    "order3_14": "+000 0+00 00+0 +-0+ 0-++",
    "order3_17": "+000 0+00 00+0 +-0+ +0-+",
    "order4_40": "+0000 0+000 00+00 000+0 0-0++ +0-0+ 00-++",
    "order4_52": "+0000 0+000 00+00 000+0 0-0++ 0++-0 +-0+0",
    "order4_76": "+0000 0+000 00+00 000+0 ++-+- 0+-+0 +0-+0",
    "order5_136": "+00000 0+0000 00+000 000+00 0000+0 000+-+ 00-+0+ +0-00+ 0+-00+",
    "order5_264": "+00000 0+0000 00+000 000+00 0000+0 0-+++- 000++- 0+-00+ +-++0-",
    "order6_560": "+000000 0+00000 00+0000 000+000 0000+00 00000+0 0++0-00 00-0++0 000-++0 0000++- +0+0--+",
    "order6_2804": "+000000 0+00000 00+0000 000+000 0000+00 00000+0 0-+000+ +0-0++- +-000+0 +-0-++0 00+0-0+",
}
Q = (math.pi / 2, math.pi / 2)      # external momentum: the nodal Fermi point
HOP, MU = 1.0, 0.0
GAMMA = 0.05                        # broadening of real frequencies
POLE = 0.1                          # least distance of a sample from a removable pole (bandwidth 8)
BATCH = ("order2", "order3_14", "order3_17", "order4_40", "order4_52", "order4_76", "order5_136", "order5_264")


def _case(name, path, diagram, n_e, n_f, **more):
    c = {"path": path, "diagram": diagram, "n_e": n_e, "n_f": n_f, "beta": 5.0, "momentum": True, "real": False}
    c.update(more)
    return {"name": name, **c} if name else c


def listed():
    return [
        # one point of a scan over external parameters: a few hundred samples, launch latency
        _case("order2_point", "forward", "order2", 300, 2),
        # the textbook diagram inside an optimizer: values and gradients of 10^4 samples
        _case("order2_step", "step", "order2", 10_000, 1),
        # a torch training loop on energies: forward and backward with a cotangent per sample, three rows
        _case("order3_autograd", "autograd", "order3_17", 33_333, 3, momentum=False),
        # one Monte-Carlo batch of an order-4 integrand at the lowest Matsubara frequency
        _case("order4_forward", "forward", "order4_52", 1_000_000, 1),
        # the same batch with every gradient
        _case("order4_step", "step", "order4_52", 1_000_000, 1),
        # a spectrum on the real axis: 256 frequencies of one batch
        _case("order4_spectrum", "forward", "order4_52", 100_001, 256, real=True),
        # the fused integrator: momenta drawn in the kernel
        _case("order4_integral", "integral", "order4_52", 10_000_000, 1),
        # complex energies (a renormalized dispersion with a lifetime)
        _case("order4_complex", "complex", "order4_52", 1_000_000, 1, momentum=False),
        # a series of diagrams, orders 2 to 5, evaluated together at 16 Matsubara frequencies
        _case("series_batch", "batch", "", 50_000, 16),
        # a large solution at 16 Matsubara frequencies
        _case("order6_forward", "forward", "order6_2804", 200_000, 16),
        # a large solution with every gradient
        _case("order6_step", "step", "order6_2804", 200_000, 1),
        # gradients at complex energies of an order-6 solution
        _case("order6_complex_step", "complex_step", "order6_560", 200_000, 1, momentum=False),
    ]


# path: (diagrams it is drawn with, least and most samples, most frequency rows)
_RANGES = {
    "forward": (tuple(TOPOLOGIES), 100, 1_000_000, 256),
    "step": (tuple(TOPOLOGIES), 100, 1_000_000, 8),
    "autograd": (("order2", "order3_17", "order4_52"), 100, 300_000, 4),
    "integral": (("order2", "order3_17", "order4_52"), 10_000, 10_000_000, 8),
    "complex": (("order2", "order3_17", "order4_52", "order5_264"), 100, 1_000_000, 16),
    "complex_step": (("order2", "order4_52", "order5_264", "order6_560"), 100, 300_000, 4),
    "batch": (("",), 500, 50_000, 16),
}


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


@functools.lru_cache(maxsize=None)
def _most():
    works = [work(c) for c in listed()]
    return max(w["flops"] for w in works), max(w["bytes"] for w in works)


def draw(rng):
    while True:
        path = rng.choice(sorted(_RANGES))
        diagrams, lo, hi, rows = _RANGES[path]
        diagram = rng.choice(diagrams)
        n_f = _log_uniform(rng, 1, rows)
        case = _case("", path, diagram, _log_uniform(rng, lo, hi) | rng.randint(0, 1), n_f,
                     beta=rng.choice([2.0, 5.0, 10.0]))
        if path in ("autograd", "complex", "complex_step"):
            case["momentum"] = False
        elif path in ("forward", "step"):
            case["momentum"] = rng.random() < 0.7
            case["real"] = n_f > 16
        w, (flops, nbytes) = work(case), _most()
        if w["flops"] <= flops and w["bytes"] <= nbytes:
            return case


# ---- the solution of a diagram, by repeated residues -----------------------

class _Solution:
    """Leaves (sigma, energy row), denominators (energy row, frequency row) and
    terms (sign, leaves, group) of a diagram, a group being one product of
    denominators."""

    def __init__(self, text):
        rows = [[{"+": 1, "-": -1, "0": 0}[ch] for ch in word] for word in text.split()]
        self.alpha = np.array(rows, dtype=np.int8)
        n_g, n = len(rows), len(rows[0]) - 1
        self.n_g, self.n = n_g, n
        start = tuple((tuple(int(i == j) for i in range(n_g)), tuple(rows[j])) for j in range(n_g))
        terms = [(1, (), start)]
        for p in range(n):
            terms = [t for old in terms for t in self._residues(old, p)]
        merged = {}
        for sign, lv, dens in terms:
            out = []
            for e, a in dens:
                s = next((x for x in e + a if x), 1)
                sign *= s
                out.append((tuple(s * x for x in e), tuple(s * x for x in a)))
            key = (tuple(sorted(lv)), tuple(sorted(out)))
            merged[key] = merged.get(key, 0) + sign
        merged = {k: s for k, s in merged.items() if s}
        self.leaves = sorted({x for lv, _ in merged for x in lv})
        self.dens = sorted({x for _, ds in merged for x in ds})
        groups = sorted({ds for _, ds in merged})
        at_l = {x: i for i, x in enumerate(self.leaves)}
        at_d = {x: i for i, x in enumerate(self.dens)}
        at_g = {x: i for i, x in enumerate(groups)}
        self.groups = np.array([[at_d[x] for x in ds] for ds in groups], dtype=np.int64)
        self.term_leaves = np.array([[at_l[x] for x in lv] for lv, _ in merged], dtype=np.int64)
        self.sums = np.zeros((len(groups), len(merged)))        # FT_g = sums @ products of leaves
        for t, ((_, ds), s) in enumerate(merged.items()):
            self.sums[at_g[ds], t] = s
        # energies at which single terms diverge while their sum stays finite
        self.poles = np.array(sorted({e for k, e in self.leaves if k < 0} | {e for e, a in self.dens if not any(a)}),
                              dtype=np.float64).reshape(-1, n_g)

    @staticmethod
    def _residues(term, p):
        sign, lv, dens = term
        for r, (e_r, a_r) in enumerate(dens):
            c = a_r[p]
            if not c:
                continue
            e_z = tuple(-c * x for x in e_r)
            a_z = tuple(0 if i == p else -c * x for i, x in enumerate(a_r))
            others = []
            for q, (e, a) in enumerate(dens):
                if q != r:
                    m = a[p]
                    others.append((tuple(x + m * z for x, z in zip(e, e_z)),
                                   tuple(0 if i == p else x + m * z for i, (x, z) in enumerate(zip(a, a_z)))))
            yield sign * c, lv + ((1 - 2 * (sum(a_z) % 2), e_z),), tuple(others)


@functools.lru_cache(maxsize=None)
def _solution(diagram):
    return _Solution(TOPOLOGIES[diagram])


def _terms(diagram):
    sol = _solution(diagram)
    return amd.Terms(sol.alpha, np.eye(sol.n_g, dtype=np.int8), sol.n)


# ---- inputs ----------------------------------------------------------------

def _diagrams(case):
    return BATCH if case["path"] == "batch" else (case["diagram"],)


def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _freqs(case):
    n_f = case["n_f"]
    if case["real"]:
        w = np.linspace(-6.0, 6.0, n_f) + 1j * GAMMA if n_f > 1 else np.array([1j * GAMMA])
    else:
        w = 1j * (2.0 * np.arange(n_f) + 1.0) * np.pi / case["beta"]
    return torch.from_numpy(w).to(_device())


def _inputs(case, seed):
    """Samples (one tensor per diagram), frequencies and cotangents, on the GPU.

    A draw that comes nearer than POLE to a removable pole of single terms is
    drawn again, as an integrator does that keeps the digits of its integrand:
    there the terms cancel and what is left is rounding."""
    dev = _device()
    g = torch.Generator(device=dev)
    g.manual_seed(seed)

    def uniform(shape, a):
        return (2.0 * a) * torch.rand(shape, dtype=torch.float64, device=dev, generator=g) - a

    def draw_rows(sol, n):
        if case["path"] in ("complex", "complex_step"):
            eta = 0.25 / (case["beta"] * sol.n)          # inside the leaves' strip of analyticity
            return torch.complex(uniform((n, sol.n_g), 3.0), uniform((n, sol.n_g), eta))
        return uniform((n, 2 * sol.n), math.pi) if case["momentum"] else uniform((n, sol.n_g), 4.0)

    x = []
    if case["path"] != "integral":
        for name in _diagrams(case):
            sol = _solution(name)
            rows = draw_rows(sol, case["n_e"])
            poles = torch.from_numpy(sol.poles).to(dev).to(rows.dtype if rows.is_complex() else torch.float64)
            for _ in range(200):
                E = _energies(sol, rows, HOP, MU) if case["momentum"] else rows
                near = ((E @ poles.T).abs() < POLE).any(1).nonzero()[:, 0]
                if not near.numel():
                    break
                rows[near] = draw_rows(sol, near.numel())
            x.append(rows)
    n_f = case["n_f"]
    w = _freqs(case)
    if case["path"] == "autograd":
        shape = (n_f, case["n_e"])
        c_out = torch.complex(uniform(shape, 1.0), uniform(shape, 1.0))
    else:
        c_out = None
    c_sum = torch.complex(uniform((n_f,), 1.0), uniform((n_f,), 1.0))
    return x, w, c_out, c_sum


def prepare(case, seed):
    x, w, c_out, c_sum = _inputs(case, seed)
    dev = w.device
    s = {"case": case, "w": w, "c_out": c_out, "c_sum": c_sum, "seed": seed,
         "terms": [_terms(name) for name in _diagrams(case)], "x": x}
    n_e, n_f = case["n_e"], case["n_f"]
    if case["path"] == "batch":
        s["items"] = [{"terms": t, "k": k, "q": Q, "t": HOP, "mu": MU, "ext_freqs": w, "beta": case["beta"],
                       "out": torch.empty((n_f, n_e), dtype=torch.complex128, device=dev),
                       "out_sum": torch.empty((n_f,), dtype=torch.complex128, device=dev)}
                      for t, k in zip(s["terms"], x)]
        s["batch"] = amd.Batch(s["items"])
    elif case["path"] != "integral":
        # a program that evaluates batch after batch keeps its result buffers
        s["out"] = torch.empty((n_f, n_e), dtype=torch.complex128, device=dev)
        s["out_sum"] = torch.empty((n_f,), dtype=torch.complex128, device=dev)
    if case["path"] == "autograd":
        s["x"] = [x[0].requires_grad_()]
        s["beta"] = torch.tensor(case["beta"], dtype=torch.float64, requires_grad=True)
    return s


def run(s):
    case, w = s["case"], s["w"]
    path, beta, t = case["path"], case["beta"], s["terms"][0]
    if path == "batch":
        s["batch"].run()
        return {"out": [it["out"] for it in s["items"]], "out_sum": [it["out_sum"] for it in s["items"]]}
    if path == "integral":
        return {"sums": amd.integrate_hubbard(t, case["n_e"], s["seed"], Q, HOP, MU, w, beta)}
    x = s["x"][0]
    if path == "autograd":
        out, out_sum = AmiEvaluate.apply(t, x, w, s["beta"], 0.0)
        g_x, g_beta = torch.autograd.grad((out, out_sum), (x, s["beta"]), (s["c_out"], s["c_sum"]))
        return {"out": out.detach(), "out_sum": out_sum.detach(), "g_x": g_x, "g_beta": g_beta}
    out, out_sum = s["out"], s["out_sum"]
    if path == "forward":
        if case["momentum"]:
            amd.evaluate_hubbard(t, x, Q, HOP, MU, w, beta, want_sum=True, out=out, out_sum=out_sum)
        else:
            amd.evaluate(t, x, w, beta, want_sum=True, out=out, out_sum=out_sum)
        return {"out": out, "out_sum": out_sum}
    if path == "complex":
        amd.evaluate_complex(t, x, w, beta, want_sum=True, out=out, out_sum=out_sum)
        return {"out": out, "out_sum": out_sum}
    if path == "complex_step":
        g_x, g_beta, g_w = amd.evaluate_complex_adjoint(t, x, w, beta, grad_sum=s["c_sum"], out=out, out_sum=out_sum)
        return {"out": out, "out_sum": out_sum, "g_x": g_x, "g_beta": g_beta, "g_w": g_w}
    if case["momentum"]:
        g_x, g_mu, g_t, g_beta, g_w = amd.evaluate_hubbard_adjoint(
            t, x, Q, HOP, MU, w, beta, grad_sum=s["c_sum"], out=out, out_sum=out_sum)
        return {"out": out, "out_sum": out_sum, "g_x": g_x, "g_mu": g_mu, "g_t": g_t, "g_beta": g_beta, "g_w": g_w}
    g_x, g_beta, g_w = amd.evaluate_adjoint(t, x, w, beta, grad_sum=s["c_sum"], out=out, out_sum=out_sum)
    return {"out": out, "out_sum": out_sum, "g_x": g_x, "g_beta": g_beta, "g_w": g_w}


# ---- what a pass cannot do without -----------------------------------------

def work(case):
    """Each input read and each output written once; per sample the energies'
    cosines (20 operations each), the leaves (an exponential and a division,
    40), the group sums (a multiply-add per term), per frequency row the
    denominators' reciprocals (20) and the groups' products; a gradient costs
    the products about three times."""
    path = case["path"]
    cplx = path in ("complex", "complex_step")
    grad = path in ("step", "autograd", "complex_step")
    n_e, n_f = case["n_e"], case["n_f"]
    flops = nbytes = 0.0
    for name in _diagrams(case):
        sol = _solution(name)
        n_in = 2 * sol.n if case["momentum"] else sol.n_g
        per_sample = 40.0 * len(sol.leaves) * (2 if cplx else 1)
        if case["momentum"]:
            per_sample += 20.0 * 2 * sol.n_g
        per_sample += 2.0 * sol.term_leaves.shape[0] * (4 if cplx else 1) * (3 if grad else 1)
        per_row = 20.0 * len(sol.dens)
        per_row += len(sol.groups) * (6.0 * (sol.groups.shape[1] - 1) + (8 if cplx else 4)) * (3 if grad else 1)
        flops += n_e * (per_sample + n_f * per_row)
        if path == "integral":
            continue
        nbytes += n_e * ((16.0 if cplx else 8.0) * n_in * (2 if grad else 1) + 16.0 * n_f)
        if path == "autograd":
            nbytes += 16.0 * n_e * n_f
    return {"bytes": nbytes + 32.0 * n_f, "flops": flops}


# ---- the same results in plain float64 arithmetic --------------------------

def _values(sol, E, w, beta):
    """I[f, s] of the solution at energies E [s, n_g] (real or complex)."""
    dev, dt = E.device, E.dtype

    def lin(rows):
        return torch.tensor(np.array(rows, dtype=np.float64), device=dev).to(dt) @ E.T

    x = beta * lin([e for _, e in sol.leaves])
    kinds = [s for s, _ in sol.leaves]
    F = torch.stack([(1.0 / (torch.exp(x[i]) + 1.0) if dt.is_complex else torch.sigmoid(-x[i])) if k > 0
                     else -1.0 / torch.expm1(x[i]) for i, k in enumerate(kinds)])
    index = torch.from_numpy(sol.term_leaves).to(dev)
    P = F.index_select(0, index[:, 0])
    for j in range(1, index.shape[1]):
        P = P * F.index_select(0, index[:, j])
    FT = torch.from_numpy(sol.sums).to(dev).to(dt) @ P
    energy = lin([e for e, _ in sol.dens])
    coef = torch.tensor([float(a[-1]) for _, a in sol.dens], dtype=torch.float64, device=dev)
    groups = torch.from_numpy(sol.groups).to(dev)
    rows = []
    for f in range(w.shape[0]):
        rho = 1.0 / (energy + (coef * w[f])[:, None])
        R = rho.index_select(0, groups[:, 0])
        for j in range(1, groups.shape[1]):
            R = R * rho.index_select(0, groups[:, j])
        rows.append((FT * R).sum(0))
    return torch.stack(rows)


def _energies(sol, k, hop, mu):
    """2 t (cos K_x + cos K_y) + mu of every propagator's momentum."""
    a = torch.from_numpy(sol.alpha.astype(np.float64)).to(k.device)
    loops = k.reshape(k.shape[0], sol.n, 2)
    K = [loops[:, :, c] @ a[:, :sol.n].T + a[:, sol.n] * Q[c] for c in range(2)]
    return 2.0 * hop * (torch.cos(K[0]) + torch.cos(K[1])) + mu


def _philox(lo, hi, block, key0, key1):
    """Four 32-bit words of Philox4x32-10 (Salmon et al., SC'11) per counter."""
    def product(m, c):
        high = ((m >> 16) * c + (((m & 0xFFFF) * c) >> 16)) >> 16
        return high, (m * (c & 0xFFFF) + (((m * (c >> 16)) & 0xFFFF) << 16)) & 0xFFFFFFFF

    c = [lo, hi, torch.full_like(lo, block), torch.zeros_like(lo)]
    for _ in range(10):
        h0, l0 = product(0xD2511F53, c[0])
        h1, l1 = product(0xCD9E8D57, c[2])
        c = [h1 ^ c[1] ^ key0, l1, h0 ^ c[3] ^ key1, l0]
        key0, key1 = (key0 + 0x9E3779B9) & 0xFFFFFFFF, (key1 + 0xBB67AE85) & 0xFFFFFFFF
    return c


def _drawn_momenta(sol, seed, s):
    words = []
    for b in range((2 * sol.n + 3) // 4):
        words += _philox(s & 0xFFFFFFFF, s >> 32, b, seed & 0xFFFFFFFF, (seed >> 32) & 0xFFFFFFFF)
    u = (torch.stack(words[:2 * sol.n], dim=1).double() + 0.5) * 2.0 ** -32
    return (u - 0.5) * (2.0 * math.pi)


def _chunks(sol, n_e):
    step = max(1, int(3e7 / max(sol.term_leaves.shape[0], 8 * sol.groups.size)))
    return [(a, min(n_e, a + step)) for a in range(0, n_e, step)]


def exact(case, seed):
    xs, w, c_out, c_sum = _inputs(case, seed)
    path, beta, n_e = case["path"], case["beta"], case["n_e"]
    sols = [_solution(name) for name in _diagrams(case)]
    if path in ("step", "autograd", "complex_step"):
        return _exact_step(case, sols[0], xs[0], w, c_out, c_sum)
    if path == "integral":
        total = torch.zeros((w.shape[0], 4), dtype=torch.float64, device=w.device)
        for a, b in _chunks(sols[0], n_e):
            k = _drawn_momenta(sols[0], seed, torch.arange(a, b, device=w.device))
            v = _values(sols[0], _energies(sols[0], k, HOP, MU), w, beta)
            total += torch.stack([v.real.sum(1), v.imag.sum(1), (v.real ** 2).sum(1), (v.imag ** 2).sum(1)], dim=1)
        return {"sums": total}
    outs = []
    for sol, x in zip(sols, xs):
        out = torch.empty((w.shape[0], n_e), dtype=torch.complex128, device=w.device)
        for a, b in _chunks(sol, n_e):
            E = _energies(sol, x[a:b], HOP, MU) if case["momentum"] else x[a:b]
            out[:, a:b] = _values(sol, E, w, beta)
        outs.append(out)
    if path == "batch":
        return {"out": outs, "out_sum": [o.sum(1) for o in outs]}
    return {"out": outs[0], "out_sum": outs[0].sum(1)}


def _exact_step(case, sol, x, w, c_out, c_sum):
    dev = w.device
    hub, n_e = case["momentum"], case["n_e"]
    out = torch.empty((w.shape[0], n_e), dtype=torch.complex128, device=dev)
    g_x = torch.empty_like(x)
    scalars = [torch.tensor(v, dtype=torch.float64, device=dev, requires_grad=True) for v in (MU, HOP, case["beta"])]
    w = w.clone().requires_grad_()
    total = [torch.zeros_like(v) for v in (*scalars, w)]
    for a, b in _chunks(sol, n_e):
        xc = x[a:b].clone().requires_grad_()
        mu, hop, beta = scalars
        v = _values(sol, _energies(sol, xc, hop, mu) if hub else xc, w, beta)
        c = c_sum[:, None].expand(v.shape) if c_out is None else c_out[:, a:b] + c_sum[:, None]
        g = torch.autograd.grad(v, (xc, *scalars, w), c, allow_unused=True)
        out[:, a:b], g_x[a:b] = v.detach(), g[0]
        for t, d in zip(total, g[1:]):
            if d is not None:
                t += d
    res = {"out": out, "out_sum": out.sum(1), "g_x": g_x, "g_beta": total[2]}
    if case["path"] != "autograd":
        res["g_w"] = total[3].reshape(-1, 1)
    if hub:
        res.update(g_mu=total[0], g_t=total[1])
    return res
