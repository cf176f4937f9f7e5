"""Fused runs of gates on complex64 states against the FP64 oracle: every cutoff
they take, the sizes where the tile rule changes (three modes, four, five and
more; few and many tiles), circuits of every generator type in an order that
lets gates move past others on disjoint modes, and runs longer than one launch
takes.  Tolerances as for the gate-by-gate evaluation: 1e-5 on amplitudes,
1e-5 |E|, 1e-4 max(1, |g|).

The batched sweep runs the same passes: its larger points equal their
single-point runs bit for bit."""
import numpy as np
import pytest
import torch

import oracle as O
import workload as W
from paper_2606_05297_amd import lib

pytestmark = pytest.mark.gpu

ALL = ("HR", "HI", "DH", "PR", "PI", "CK")
CASES = [(15, 2, True, 40), (20, 2, False, 16), (9, 3, False, 30), (10, 3, True, 24), (7, 4, True, 30), (8, 4, False, 40), (6, 5, True, 30),
         (7, 5, False, 24), (6, 6, True, 40), (7, 6, False, 24), (5, 7, True, 25), (6, 7, False, 20), (5, 8, True, 40),
         (6, 8, True, 30)]


def check(ho, hl, ops, th, psi0):
    L, d = ho.L, ho.d
    x0 = torch.from_numpy(psi0).cuda()
    a, b = torch.empty_like(x0), torch.empty_like(x0)
    ws = lib.workspace(hl, 0, len(ops))
    E, n2, g = lib.energy_grad_adjoint(hl, ops, th, x0, a, b, ws)
    Eo, go, n2o = O.energy_and_grad_adjoint(ho, psi0.astype(np.complex128), ops, th)
    assert abs(E - Eo / n2o) <= 1e-5 * max(1.0, abs(Eo)) and abs(n2 - n2o) <= 1e-5
    assert np.abs(g - go).max() <= 1e-4 * max(1.0, np.abs(go).max())
    E2, m2, _ = lib.energy_grad_adjoint(hl, ops, th, x0, a, b, ws, grad=False)
    assert (E2, m2) == (E, n2)
    psi = O.ansatz_state(psi0.astype(np.complex128), ops, th, L, d)
    assert np.abs(a.cpu().numpy() - psi).max() <= 1e-5
    gs = lib.adjoint_sweep(hl, ops, th, a, b, n2, ws)  # the reverse sweep alone
    assert np.array_equal(gs, g)
    assert np.abs(a.cpu().numpy() - psi0).max() <= 1e-5


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"L{c[0]}d{c[1]}{'p' if c[2] else ''}n{c[3]}")
def test_runs_match_oracle(case):
    L, d, per, n = case
    print("[case] runs", case, flush=True)
    prm = (1.0, 0.7, 0.2, 0.4, 0.15)
    ho, hl = O.Ham(L, d, per, *prm), lib.ham(L, d, per, *prm)
    rng = np.random.default_rng(100 * L + d)
    pairs = W.pool(L, "all", per, ALL)
    ops = [pairs[k] for k in rng.integers(0, len(pairs), n)]
    # an isolated phase gate, a run of phase gates and squeezers among them
    ops[n // 4] = ("KERR", L // 2, -1)
    ops[n // 2:n // 2 + 2] = [("ROT", 0, -1), ("KERR", L - 1, -1)]
    ops[n - 3] = ("SR", 1, -1)
    check(ho, hl, ops, rng.uniform(-0.5, 0.5, n), W.random_state(L, d, seed=5))


@pytest.mark.parametrize("n", [16, 17, 40])
def test_runs_of_many_gates(n):
    """Circuits on three modes of a longer chain: one window, up to and beyond the gates of one launch."""
    L, d = 6, 6
    ho, hl = O.Ham(L, d, False, 1.0, 2.0, 0.0, 0.3, 0.0), lib.ham(L, d, False, 1.0, 2.0, 0.0, 0.3, 0.0)
    ops = [((ALL[k % 6]), *[(1, 4), (2, 4), (1, 2)][k % 3]) for k in range(n)]
    check(ho, hl, ops, np.linspace(-0.3, 0.4, n), W.random_state(L, d, seed=6))


def test_sweep_points_equal_single_runs():
    pts = [W.sweep_points()[k] for k in (24, 72, 75)]  # Bose-Hubbard L=6 d=6 with its warm-up layer, Kitaev-Kerr L=6 d=8
    lib.set_real_states(lib.REAL_OFF)
    try:
        entries = []
        for p in pts:
            x = torch.zeros(p["d"] ** p["L"], dtype=torch.complex64, device="cuda")
            x[W.fock_index(p["L"], p["d"], p["occ"])] = 1
            wops = W.warmup_ops(p["L"], p["periodic"]) if p["warm"] else []
            entries.append(dict(ham=lib.ham_from(p), pool=p["pool"], psi0=x, warm_ops=wops,
                                warm_theta0=W.warmup_theta0(len(wops), p["warm_seed"]) if wops else np.zeros(0)))
        singles = [lib.Adapt(e["ham"], e["pool"], e["psi0"], max_iters=4, warm_ops=e["warm_ops"],
                             warm_theta0=e["warm_theta0"]) for e in entries]
        sw = lib.Sweep(entries, max_iters=4)
        for _ in range(3):
            reps, _n = sw.step()
            for k, a in enumerate(singles):
                r = a.step()
                assert (reps[k]["k_sel"], reps[k]["E"], reps[k]["bfgs_evals"]) == (r["k_sel"], r["E"], r["bfgs_evals"]), k
        sw.close()
        for a in singles:
            a.close()
    finally:
        lib.set_real_states(lib.REAL_AUTO)
