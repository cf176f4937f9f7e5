"""Whole-circuit evaluation of small states by one workgroup: energy, norm,
gradients and final states against the FP64 oracle, over the cutoffs and sizes
where its decomposition changes (member slots of 2, 4 and 8, fibres that do not
fill a chunk of 16, the largest states its LDS takes and the first beyond) and
circuits of every generator type, up to and beyond its gate limit.

Tolerances as for the gate-by-gate evaluation: 1e-5 on amplitudes, 1e-5 |E|,
1e-4 max(1, |g|)."""
import numpy as np
import pytest
import torch

import oracle as O
import workload as W
from paper_2606_05297_amd import lib

pytestmark = pytest.mark.gpu

ALL = ("HR", "HI", "DH", "PR", "PI", "CK")
# (L, d, periodic, gates): last rows are the largest states of one workgroup and the first beyond
CASES = [(2, 2, False, 6), (1, 5, False, 4), (5, 2, True, 20), (13, 2, True, 30), (3, 3, True, 15), (8, 3, False, 18),
         (3, 4, False, 33), (6, 4, True, 25), (2, 5, False, 10), (4, 5, True, 20), (4, 6, True, 40), (2, 7, False, 9),
         (4, 7, True, 24), (2, 8, False, 12), (4, 8, False, 30), (3, 8, True, 70), (5, 6, True, 25), (5, 7, False, 6)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"L{c[0]}d{c[1]}{'p' if c[2] else ''}n{c[3]}")
def test_small_states_match_oracle(case):
    L, d, per, n = case
    print("[case] small", case, flush=True)
    prm = (1.0, 0.7, 0.2, 0.4, 0.15)
    ho, hl = O.Ham(L, d, per, *prm), lib.ham(L, d, per, *prm)
    pool = (W.pool(L, "all", per, ALL) if L > 1 else []) + W.site_ops(L, ("KERR", "ROT", "SR", "SI"))
    rng = np.random.default_rng(100 * L + d)
    ops = [pool[k] for k in rng.permutation(np.arange(n) * 7919 % len(pool))]
    th = rng.uniform(-0.5, 0.5, n)
    psi0 = W.random_state(L, d, seed=5)
    x0 = torch.from_numpy(psi0).cuda()
    a, b = torch.empty_like(x0), torch.empty_like(x0)
    ws = lib.workspace(hl, 0, n)
    E, n2, g = lib.energy_grad_adjoint(hl, ops, th, x0, a, b, ws)
    Eo, go, n2o = O.energy_and_grad_adjoint(ho, psi0.astype(np.complex128), ops, th)
    assert abs(E - Eo / n2o) <= 1e-5 * max(1.0, abs(Eo)) and abs(n2 - n2o) <= 1e-5
    assert np.abs(g - go).max() <= 1e-4 * max(1.0, np.abs(go).max())
    E2, m2, _ = lib.energy_grad_adjoint(hl, ops, th, x0, a, b, ws, grad=False)
    assert (E2, m2) == (E, n2)
    psi = O.ansatz_state(psi0.astype(np.complex128), ops, th, L, d)
    hpsi = O.apply_H(ho, psi)
    assert np.abs(a.cpu().numpy() - psi).max() <= 1e-5
    assert np.abs(b.cpu().numpy() - hpsi).max() <= 1e-5 * max(1.0, np.abs(hpsi).max())
    E3, _, g3 = lib.energy_grad_adjoint(hl, ops, th, x0, a, b, ws)  # bit-identical when repeated
    assert E3 == E and np.array_equal(g3, g)


@pytest.mark.parametrize("n", [0, 1, 64, 65, 256, 257])
def test_circuit_lengths(n):
    """No gate, the table build's argument limit (64) and the evaluation's (256)."""
    L, d = 3, 4
    ho, hl = O.Ham(L, d, False, 1.0, 2.0, 0.0, 0.3, 0.0), lib.ham(L, d, False, 1.0, 2.0, 0.0, 0.3, 0.0)
    pool = W.pool(L, "all", False, ALL) + W.site_ops(L, ("KERR", "SR"))
    ops, th = W.random_circuit(pool, n, seed=n)
    th = 0.2 * th
    psi0 = W.random_state(L, d, seed=1)
    x0 = torch.from_numpy(psi0).cuda()
    a, b = torch.empty_like(x0), torch.empty_like(x0)
    E, _, g = lib.energy_grad_adjoint(hl, ops, th, x0, a, b, lib.workspace(hl, 0, n))
    Eo, go, n2o = O.energy_and_grad_adjoint(ho, psi0.astype(np.complex128), ops, th)
    assert abs(E - Eo / n2o) <= 1e-5 * max(1.0, abs(Eo))
    assert n == 0 or np.abs(g - go).max() <= 1e-4 * max(1.0, np.abs(go).max())


def test_symmetry_is_kept_exactly():
    """Amplitudes outside the boson-number sector stay exactly zero."""
    L, d = 4, 6
    hl = lib.ham(L, d, True, 1.0, 2.0)
    pool = W.pool(L, "all", True, W.BH_TYPES) + W.site_ops(L, ("KERR", "ROT"))
    ops, th = W.random_circuit(pool, 40, seed=2)
    psi0 = W.random_state(L, d, seed=3, sector=("N", L))
    x0 = torch.from_numpy(psi0).cuda()
    a, b = torch.empty_like(x0), torch.empty_like(x0)
    lib.energy_grad_adjoint(hl, ops, th, x0, a, b, lib.workspace(hl, 0, 40), grad=False)
    out = O.occupations(L, d).sum(axis=-1).reshape(-1) != L
    for t in (a, b):
        assert np.count_nonzero(t.cpu().numpy()[out]) == 0
