"""Performance cases: what a user of this framework has it compute, at the sizes of its own workloads.

    listed()            the named cases
    draw(rng)           one more case of the same ranges
    prepare(case, seed) the inputs, buffers and handles a user's program holds before the call
    run(state)          one pass through the public entry points of paper_2606_05297_amd.lib
    work(case)          bytes and floating-point operations one pass cannot do without
    exact(case, seed)   the same outputs in 64 bits from plain torch

Kinds of case
    eval    energy and all angle gradients of a circuit (lib.energy_grad_adjoint): one objective call of the BFGS
            re-optimisation, the call an ADAPT run makes most often
    energy  the same call without gradients; it leaves psi and H psi
    h       H psi with energy and norm (lib.apply_H)
    score   H psi and the gradients of a whole pool (lib.score): once per ADAPT step
    eval64  the evaluation on complex128 states (lib.Adapt64.energy_grad)
    mlp     loss and gradient of the warm-start network on one batch (lib.Mlp.loss_grad)
    adapt   a whole run: creation and its first steps (lib.Adapt)
    sweep   a whole batched run over several Hamiltonian points (lib.Sweep)

Energies and gradients computed from complex64 or float32 states come back from the library as doubles whose digits
beyond single precision are the states' rounding; they are returned here as float32, the type they are good to.
The angles of whole runs are fixed only to the optimiser's tolerance; whole runs return the energies it reports.
"""
import math

import numpy as np
import torch

import workload as W
from paper_2606_05297_amd import lib

PAPER_TYPES = ("HR", "HI", "PR", "PI", "CK")


def listed():
    return [
        # the smallest workload (Bose-Hubbard chain of 3 sites, 64 amplitudes): latency of one BFGS objective call
        # with the warm-up layer and 12 ADAPT gates
        dict(name="eval_bh_l3_d4", kind="eval", model="bh", L=3, d=4, n=12, store="complex"),
        # the warm-start workload (Kitaev-Kerr, 6 modes, 262,144 amplitudes) half-way through a run
        dict(name="eval_kk_l6_d8", kind="eval", model="kk", L=6, d=8, n=30, store="complex"),
        # the Bose-Hubbard ring of 8 sites (1,679,616 amplitudes), warm-up layer and 24 gates
        dict(name="eval_bh_l8_d6", kind="eval", model="bh", L=8, d=6, n=24, store="complex"),
        # the benchmark's chain on the full complex64 tensor: 30 gates of every type of its pool
        dict(name="eval_kk_l8_d8", kind="eval", model="kk", L=8, d=8, n=30, store="complex"),
        # the same chain as the ADAPT driver keeps it: real amplitudes of the even sector, HR and PR gates
        dict(name="eval_kk_l8_d8_real", kind="eval", model="kk", L=8, d=8, n=21, store="real_even"),
        # H psi on the largest tensor
        dict(name="h_kk_l8_d8", kind="h", model="kk", L=8, d=8, store="complex"),
        # pool scoring on the benchmark's chain (28 operators) and on the ring (48 operators)
        dict(name="score_kk_l8_d8_even", kind="score", model="kk", L=8, d=8, store="even"),
        dict(name="score_bh_l8_d6", kind="score", model="bh", L=8, d=6, store="complex"),
        # the complex128 driver at the paper's size, every one-parameter generator of its pool
        dict(name="eval64_kk_l4_d6", kind="eval64", L=4, d=6, n=40),
        # one training batch of the warm-start network
        dict(name="mlp_grad_b1024", kind="mlp", B=1024),
        # the benchmark: creation of the run and its first steps, with Hessian recycling
        dict(name="adapt_kk_l8_d8", kind="adapt", L=8, d=8, steps=6),
        # a parameter sweep over both models: warm-up layers and two steps on every point
        dict(name="sweep_12_points", kind="sweep", n_bh4=2, n_bh6=2, n_kk4=4, n_kk6=4, steps=2),
    ]


def _lattice(rng, lo, hi):
    """(L, d) with lo <= d^L <= hi, spread over the logarithm of d^L, odd cutoffs among them."""
    want = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    fits = [(abs(math.log(d**L / want)), L, d) for d in range(3, 9) for L in range(2, 11) if lo <= d**L <= hi]
    near = sorted(fits)[:5]
    _, L, d = near[rng.randrange(len(near))]
    return L, d


def draw(rng):
    kind = rng.choice(["eval"] * 6 + ["energy", "h", "h", "score", "score", "eval64", "eval64", "mlp", "adapt", "sweep"])
    if kind in ("eval", "energy", "h", "score"):
        model = rng.choice(["bh", "kk"])
        c = dict(kind=kind, model=model, store="complex")
        if rng.random() < 0.25:  # the benchmark's chain in its three forms
            c.update(model="kk", L=8, d=8)
            c["store"] = rng.choice({"eval": ["complex", "even", "real_even"], "energy": ["complex", "even", "real_even"],
                                     "h": ["even", "real_even"], "score": ["complex", "even"]}[kind])
        else:
            c["L"], c["d"] = _lattice(rng, 27, 2**22)
        if kind in ("eval", "energy"):
            c["n"] = rng.randint(3, 30)
        if kind == "score":
            c["share"] = round(rng.uniform(0.3, 1.0), 3)  # of the pool's operators, as operator tiling leaves
        return c
    if kind == "eval64":
        L, d = rng.choice([(3, 5), (3, 6), (3, 7), (3, 8), (4, 4), (4, 5), (4, 6), (4, 7), (5, 6), (4, 13)])
        return dict(kind=kind, L=L, d=d, n=rng.randint(5, 60))
    if kind == "mlp":
        return dict(kind=kind, B=round(math.exp(rng.uniform(math.log(16), math.log(16384)))))
    if kind == "adapt":
        L, d = rng.choice([(3, 8), (4, 6), (4, 8), (5, 7), (5, 8), (6, 5), (6, 6), (6, 8), (8, 8)])
        return dict(kind=kind, L=L, d=d, steps=rng.randint(2, 6))
    return dict(kind=kind, n_bh4=rng.randint(0, 4), n_bh6=rng.randint(0, 3), n_kk4=rng.randint(1, 6),
                n_kk6=rng.randint(0, 4), steps=rng.randint(1, 2))


# ---------------------------------------------------------------- inputs

LAYOUTS = {"complex": lib.LAYOUT_FULL, "even": lib.LAYOUT_EVEN, "real_even": lib.LAYOUT_EVEN | lib.LAYOUT_REAL}


def _lattice_of(case, rng):
    """Hamiltonian parameters, pool, occupation and warm-up gates of a case."""
    L, d = case["L"], case["d"]
    if case.get("model") == "bh":  # ring with one boson per site, next-nearest-neighbour pool (open chain at L = 3)
        per = L != 3
        p = dict(L=L, d=d, periodic=per, J=1.0, U=float(rng.uniform(1.0, 16.0)), mu=0.0, Delta=0.0, K=0.0)
        return p, W.pool(L, "all" if L == 3 else "nn+nnn", per, W.BH_TYPES), [1] * L, W.warmup_ops(L, per)
    p = dict(L=L, d=d, periodic=False, J=1.0, U=0.0, mu=0.0, Delta=float(rng.uniform(0.4, 0.6)),
             K=float(rng.uniform(0.15, 0.25)))
    return p, W.pool(L, "nn", False, W.KITAEV_TYPES), [0] * L, []


def _part(pool, case):
    n = max(1, round(case.get("share", 1.0) * len(pool)))
    return [pool[k * len(pool) // n] for k in range(n)]


def _circuit(case, rng):
    p, pool, occ, warm = _lattice_of(case, rng)
    if case.get("store") == "real_even":
        pool = [o for o in pool if o[0] in ("HR", "PR")]
    ops = list(warm) + [pool[k] for k in rng.integers(0, len(pool), case["n"])]
    theta = np.concatenate([rng.uniform(-0.05, 0.05, len(warm)), rng.uniform(-0.5, 0.5, case["n"])])
    return p, pool, occ, ops, theta


def _paper_circuit(case, rng):
    L, d = case["L"], case["d"]
    p = dict(L=L, d=d, periodic=True, J=1.0, U=0.0, mu=float(rng.uniform(-3.1, -2.7)), Delta=0.5,
             K=float(rng.uniform(0.3, 0.6)))
    pool = W.pool(L, "all", True, PAPER_TYPES) + W.site_ops(L, ("SR", "SI", "ROT", "KERR"))
    ops = [pool[k] for k in rng.integers(0, len(pool), case["n"])]
    return p, pool, ops, rng.uniform(-0.4, 0.4, case["n"])


def _totals(L, d):
    idx = torch.arange(d**L, device="cuda")
    tot = torch.zeros_like(idx)
    for _ in range(L):
        tot += idx % d
        idx //= d
    return tot


def _half_index(L, d):
    """Flat indices, in the full tensor, of the stored amplitudes of the even sector."""
    low = d ** (L - 1)
    c = torch.arange(d**L // 2, device="cuda")
    rest, m = c % low, c // low
    t, par = rest.clone(), torch.zeros_like(c)
    for _ in range(L - 1):
        par += t % d
        t //= d
    return rest + (2 * m + par % 2) * low


def _random_state(case, seed):
    """A normalised random state of the symmetry sector the workload lives in, in the case's storage."""
    L, d = case["L"], case["d"]
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    v = torch.randn(d**L, 2, generator=g, device="cuda")
    v = v[:, 0].to(torch.complex64) if case["store"] == "real_even" else torch.view_as_complex(v)
    tot = _totals(L, d)
    v = torch.where(tot == L if case["model"] == "bh" else tot % 2 == 0, v, torch.zeros_like(v))
    v = v / torch.linalg.vector_norm(v)
    if case["store"] != "complex":
        v = v[_half_index(L, d)]
    return v.real.contiguous() if case["store"] == "real_even" else v.contiguous()


def _fock(case, occ, dtype=torch.complex64):
    k = W.fock_index(case["L"], case["d"], occ)  # the sector layouts are used from the vacuum: index 0 in both
    n = case["d"] ** case["L"] // (1 if case.get("store", "complex") == "complex" else 2)
    v = torch.zeros(n, dtype=torch.float32 if case.get("store") == "real_even" else dtype, device="cuda")
    v[k] = 1
    return v


def prepare(case, seed):
    rng = np.random.default_rng(seed)
    kind = case["kind"]
    s = dict(case)
    if kind in ("eval", "energy"):
        p, pool, occ, s["ops"], s["theta"] = _circuit(case, rng)
        s["h"] = lib.ham_from(p, layout=LAYOUTS[case["store"]])
        s["psi0"] = _fock(case, occ)
        s["psi"], s["lam"] = torch.empty_like(s["psi0"]), torch.empty_like(s["psi0"])
        s["ws"] = lib.workspace(s["h"], 0, len(s["ops"]))
    elif kind in ("h", "score"):
        p, s["pool"], _, _ = _lattice_of(case, rng)
        s["h"] = lib.ham_from(p, layout=LAYOUTS[case["store"]])
        s["pool"] = _part(s["pool"], case)
        s["psi"] = _random_state(case, seed)
        s["hpsi"] = torch.empty_like(s["psi"])
        s["ws"] = lib.workspace(s["h"], len(s["pool"]), 0)
    elif kind == "eval64":
        p, pool, s["ops"], s["theta"] = _paper_circuit(case, rng)
        s["run"] = lib.Adapt64(lib.ham_from(p), pool, _fock(case, [0] * case["L"], torch.complex128))
    elif kind == "mlp":
        X, T, nv, par = _batch(case, rng, seed)
        s["X"], s["T"], s["nv"] = torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda(), torch.from_numpy(nv).cuda()
        s["net"] = lib.Mlp(case["B"], par)
    elif kind == "adapt":
        p, s["pool"], occ, _ = _lattice_of(dict(case, model="kk"), rng)
        s["h"], s["psi0"] = lib.ham_from(p), _fock(case, occ)
    else:
        s["points"] = []
        for n, model, sizes in ((case["n_bh4"], "bh", ((4, 4), (4, 6))), (case["n_bh6"], "bh", ((6, 4), (6, 6))),
                                (case["n_kk4"], "kk", ((4, 8),)), (case["n_kk6"], "kk", ((6, 8),))):
            for k in range(n):
                L, d = sizes[k % len(sizes)]
                c = dict(L=L, d=d, model=model)
                p, pool, occ, warm = _lattice_of(c, rng)
                s["points"].append(dict(ham=lib.ham_from(p), pool=pool, psi0=_fock(c, occ), warm_ops=warm,
                                        warm_theta0=rng.uniform(-0.05, 0.05, len(warm))))
    return s


def _batch(case, rng, seed):
    B = case["B"]
    X = np.stack([np.ones(B), rng.uniform(0, 1, B), rng.uniform(0, 0.5, B), rng.integers(1, 65, B) / 64.0], axis=1)
    T = rng.normal(0, 0.3, (B, 64))
    return (X.astype(np.float32), T.astype(np.float32), rng.integers(1, 65, B).astype(np.int32),
            W.mlp_init(seed % 1000))


def run(state):
    s, kind = state, state["kind"]
    if kind == "eval":
        E, n2, g = lib.energy_grad_adjoint(s["h"], s["ops"], s["theta"], s["psi0"], s["psi"], s["lam"], s["ws"])
        return {"E": np.float32(E), "norm2": np.float32(n2), "grad": g.astype(np.float32)}
    if kind == "energy":
        E, n2, _ = lib.energy_grad_adjoint(s["h"], s["ops"], s["theta"], s["psi0"], s["psi"], s["lam"], s["ws"],
                                           grad=False)
        return {"E": np.float32(E), "norm2": np.float32(n2), "psi": s["psi"], "hpsi": s["lam"]}
    if kind == "h":
        E, n2 = lib.apply_H(s["h"], s["psi"], s["hpsi"], s["ws"])
        return {"E": np.float32(E), "norm2": np.float32(n2), "hpsi": s["hpsi"]}
    if kind == "score":
        g, E, n2 = lib.score(s["h"], s["pool"], s["psi"], s["hpsi"], s["ws"])
        return {"E": np.float32(E), "norm2": np.float32(n2), "hpsi": s["hpsi"], "grads": g.astype(np.float32)}
    if kind == "eval64":
        E, g = s["run"].energy_grad(s["ops"], s["theta"])
        return {"E": E, "grad": g}
    if kind == "mlp":
        loss, g = s["net"].loss_grad(s["X"], s["T"], s["nv"])
        return {"loss": np.float32(loss), "grad": g}
    if kind == "adapt":
        ad = lib.Adapt(s["h"], s["pool"], s["psi0"], max_iters=60, recycle_hessian=True)
        reps = [ad.step() for _ in range(s["steps"])]
        ad.close()
        return {k: np.array([r[k] for r in reps], dtype=np.float32) for k in ("E_init", "E")}
    sw = lib.Sweep(s["points"], max_iters=40)
    E = [[r["E"] for r in sw.warm_reports()]]
    for _ in range(s["steps"]):
        E.append([r["E"] for r in sw.step()[0]])
    sw.close()
    return np.array(E, dtype=np.float32)


# ---------------------------------------------------------------- what a pass cannot do without

def _amp_bytes(case):
    return {"complex": 8, "even": 4, "real_even": 2}[case.get("store", "complex")]  # per amplitude of the d^L tensor


def _gate_flops(d, n_amp, real):
    """exp(theta A) as conserved blocks, (2 d^3 + d) / 3 products per fibre of d^2 amplitudes."""
    return (2.0 if real else 8.0) * (2 * d**3 + d) / 3.0 / d**2 * n_amp


def work(case):
    """Inputs read and results written once.  An evaluation's states are its own, so its bytes are psi0's; its
    operations are the gates on one state forward and on two in reverse, the generators' products and H psi."""
    kind = case["kind"]
    if kind == "mlp":
        macs = 4 * 128 + 128 * 128 + 128 * 64
        return {"bytes": case["B"] * (4 + 64 + 1) * 4.0 + 2 * 4 * lib.MLP_NPARAMS, "flops": 6.0 * macs * case["B"]}
    if kind == "sweep":
        pts = [(n, L, d) for n, L, d in ((case["n_bh4"], 4, 5), (case["n_bh6"], 6, 5), (case["n_kk4"], 4, 8),
                                         (case["n_kk6"], 6, 8))]
        N = sum(n * float(d)**L for n, L, d in pts)
        # per step at least the scoring and two evaluations of a few gates
        return {"bytes": 8.0 * N, "flops": case["steps"] * sum(n * 8 * _gate_flops(d, float(d)**L, False) for n, L, d in pts)}
    L, d = case["L"], case["d"]
    N = float(d)**L
    real = case.get("store") == "real_even" or kind == "adapt"
    n_amp = N / 2 if case.get("store", "complex") != "complex" or kind == "adapt" else N
    w = 2.0 if real else 4.0
    f_h = w * 4 * L * n_amp
    if kind == "adapt":
        n = sum(3 * k for k in range(1, case["steps"] + 1))  # at least three evaluations a step
        return {"bytes": 8.0 * N, "flops": 3 * n * _gate_flops(d, n_amp, True) + case["steps"] * 4 * f_h}
    if kind == "eval64":
        return {"bytes": 16.0 * N, "flops": case["n"] * (3 * _gate_flops(d, N, False) + 32 * N) + f_h}
    a = _amp_bytes(case)
    if kind == "h":
        return {"bytes": 2 * a * N, "flops": f_h}
    if kind == "score":
        pairs = len(W.pairs(L, "nn", False)) if case["model"] == "kk" else 2 * L
        return {"bytes": 2 * a * N, "flops": f_h + case.get("share", 1.0) * pairs * 32 * n_amp}
    n = case["n"] + (3 * L if case["model"] == "bh" else 0)
    g = _gate_flops(d, n_amp, real)
    if kind == "energy":
        return {"bytes": 3 * a * N, "flops": case["n"] * g + f_h}
    return {"bytes": a * N, "flops": case["n"] * (3 * g + 4 * w * n_amp) + (n - case["n"]) * 16 * n_amp + f_h}


# ---------------------------------------------------------------- the same in 64 bits

C128 = torch.complex128


def _ladder(d):
    return torch.diag(torch.sqrt(torch.arange(1, d, dtype=torch.float64, device="cuda")), 1).to(C128)


def _kron(x, y):
    return torch.kron(x.contiguous(), y.contiguous())


def _generator(t, d):
    """The generator's matrix over (n_i, n_j) (index n_i d + n_j), or over n_i for a single mode."""
    a = _ladder(d)
    ad, num = a.mH.resolve_conj().contiguous(), torch.diag(torch.arange(d, device="cuda").to(C128))
    hop, pair = _kron(ad, a), _kron(a, a)
    if t == "HR":
        return hop - hop.mH
    if t == "HI":
        return 1j * (hop + hop.mH)
    if t == "DH":
        x = _kron(num @ ad, a)
        return 1j * (x + x.mH)
    if t == "PR":
        return pair - pair.mH
    if t == "PI":
        return 1j * (pair + pair.mH)
    if t == "CK":
        return 1j * _kron(num, num)
    if t == "KERR":
        return 1j * num @ num
    if t == "ROT":
        return 1j * num
    return (a @ a - ad @ ad) / 2 if t == "SR" else 1j * (a @ a + ad @ ad) / 2


class _Plain:
    """The chain's operators on a complex128 tensor, as dense matrices over the modes they act on."""

    def __init__(self, p):
        self.p, self.L, self.d, self.gen, self.eig = p, p["L"], p["d"], {}, {}

    def op(self, M, i, j, v):
        L, d = self.L, self.d
        axes = [L - 1 - i] + ([L - 1 - j] if j >= 0 else [])
        x = v.reshape([d] * L).movedim(axes, list(range(len(axes))))
        shape = x.shape
        y = M @ x.reshape(M.shape[0], -1)
        return y.reshape(shape).movedim(list(range(len(axes))), axes).reshape(-1)

    def A(self, o):
        if o[0] not in self.gen:
            self.gen[o[0]] = _generator(o[0], self.d)
        return self.gen[o[0]]

    def U(self, o, th):
        if o[0] not in self.eig:
            self.eig[o[0]] = torch.linalg.eigh((-1j * self.A(o)).cpu())
        lam, V = self.eig[o[0]]
        return ((V * torch.exp(1j * float(th) * lam)) @ V.mH.resolve_conj()).cuda()

    def H(self, v):
        p, L, d = self.p, self.L, self.d
        a = _ladder(d)
        hop, pair = _kron(a.mH.resolve_conj(), a), _kron(a, a)
        B = -p["J"] * (hop + hop.mH) + p["Delta"] * (pair + pair.mH)
        out = torch.zeros_like(v)
        for i, j in [(r, r + 1) for r in range(L - 1)] + ([(0, L - 1)] if p["periodic"] and L >= 3 else []):
            out += self.op(B, i, j, v)
        idx = torch.arange(d**L, device=v.device)
        diag = torch.zeros(d**L, dtype=torch.float64, device=v.device)
        for _ in range(L):
            n = (idx % d).to(torch.float64)
            diag += (p["U"] / 2 + p["K"]) * n * (n - 1) - p["mu"] * n
            idx = idx // d
        return out + diag * v


def _evaluate(p, ops, theta, psi, grad):
    """(E, norm2, dE/dtheta, psi, H psi) of the circuit on psi, gradients by the adjoint identity."""
    P = _Plain(p)
    us = [P.U(o, t) for o, t in zip(ops, theta)]
    for o, u in zip(ops, us):
        psi = P.op(u, o[1], o[2], psi)
    lam = P.H(psi)
    n2, E = torch.vdot(psi, psi).real, torch.vdot(psi, lam).real
    if not grad:
        return float(E / n2), float(n2), None, psi, lam
    g = torch.zeros(len(ops), dtype=torch.float64)
    for k in range(len(ops) - 1, -1, -1):
        o = ops[k]
        g[k] = 2 * torch.vdot(lam, P.op(P.A(o), o[1], o[2], psi)).real / n2
        back = us[k].mH.resolve_conj().contiguous()
        psi, lam = P.op(back, o[1], o[2], psi), P.op(back, o[1], o[2], lam)
    return float(E / n2), float(n2), g.numpy(), None, None


def exact(case, seed):
    rng = np.random.default_rng(seed)
    kind = case["kind"]
    if kind in ("adapt", "sweep"):
        return None  # where the optimiser stops is its own
    if kind == "mlp":
        return _mlp_exact(case, rng, seed)
    if kind == "eval64":
        p, _, ops, theta = _paper_circuit(case, rng)
        E, _, g, _, _ = _evaluate(p, ops, theta, _fock(case, [0] * case["L"], C128), True)
        return {"E": E, "grad": g}
    L, d, half = case["L"], case["d"], case["store"] != "complex"
    stored = _half_index(L, d) if half else None

    def out(v):
        v = v[stored] if half else v
        return v.real.contiguous() if case["store"] == "real_even" else v

    if kind in ("eval", "energy"):
        p, _, occ, ops, theta = _circuit(case, rng)
        full = torch.zeros(d**L, dtype=C128, device="cuda")
        full[W.fock_index(L, d, occ)] = 1
        E, n2, g, psi, hpsi = _evaluate(p, ops, theta, full, kind == "eval")
        if kind == "eval":
            return {"E": E, "norm2": n2, "grad": g}
        return {"E": E, "norm2": n2, "psi": out(psi), "hpsi": out(hpsi)}
    p, pool, _, _ = _lattice_of(case, rng)
    psi = _random_state(case, seed).to(C128)
    if half:
        full = torch.zeros(d**L, dtype=C128, device="cuda")
        full[stored] = psi
        psi = full
    P = _Plain(p)
    hpsi = P.H(psi)
    r = {"E": float(torch.vdot(psi, hpsi).real), "norm2": float(torch.vdot(psi, psi).real), "hpsi": out(hpsi)}
    if kind == "score":
        r["grads"] = np.array([float(2 * torch.vdot(hpsi, P.op(P.A(o), o[1], o[2], psi)).real) for o in _part(pool, case)])
    return r


def _mlp_exact(case, rng, seed):
    """Masked mean-squared error of the 4 -> 128 -> 128 -> 64 SiLU network and its gradient, by autograd."""
    X, T, nv, par = _batch(case, rng, seed)
    X, T = torch.from_numpy(X).double(), torch.from_numpy(T).double()
    w = torch.from_numpy(par).double().requires_grad_(True)
    parts, at = [], 0
    for shape, _ in W.MLP_SHAPES:
        parts.append(w[at:at + math.prod(shape)].reshape(shape))
        at += math.prod(shape)
    y = X
    for k in range(3):
        y = y @ parts[2 * k].T + parts[2 * k + 1]
        if k < 2:
            y = torch.nn.functional.silu(y)
    mask = (torch.arange(64)[None, :] < torch.from_numpy(nv)[:, None]).double()
    loss = ((y - T) ** 2 * mask).sum() / mask.sum()
    loss.backward()
    return {"loss": float(loss.detach()), "grad": w.grad.numpy()}
