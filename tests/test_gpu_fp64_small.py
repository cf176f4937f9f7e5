"""The one-launch complex128 evaluation (csrc/f64_small.hip) against the FP64
oracle at the edges of what it takes: groups split over 4 threads, one and
several groups a thread, powers of two (folded addresses) and other cutoffs, one
mode, circuits whose gate tables are built in several passes, no gates at all, and
the first cutoffs, states and circuits beyond it (gate by gate).

Tolerances.  A gate rounds each amplitude by at most about 2 d eps = 4.4e-16 d of
the state (sums of up to d products), so E of n gates is off by at most
2 n (4.4e-16 d) |H|, and a gradient by 2 |A| times that, with the operator norms
bounded term by term."""

import numpy as np
import pytest
import torch

import oracle as O
import workload as W
from paper_2606_05297_amd import lib

pytestmark = pytest.mark.gpu

TWO = ("HR", "HI", "DH", "PR", "PI", "CK")
ONE = ("SR", "SI", "KERR", "ROT")

CASES = [
    # L, d, periodic, gates
    (1, 8, False, 12),
    (1, 9, False, 12),  # beyond the cutoffs it takes
    (2, 2, False, 30),
    (2, 13, False, 24),
    (2, 7, False, 24),
    (3, 5, True, 40),
    (3, 8, True, 40),  # tables in several passes
    (4, 3, True, 40),
    (4, 4, True, 256),
    (4, 4, True, 257),  # one gate too many
    (4, 5, True, 30),  # two waves of groups
    (4, 6, True, 100),
    (4, 7, False, 40),
    (4, 8, True, 20),  # beyond the amplitudes it takes
    (5, 4, True, 60),
    (5, 5, True, 20),  # two groups a thread
    (6, 4, False, 20),
    (11, 2, True, 33),
]


@pytest.mark.parametrize("L,d,periodic,n", CASES, ids=lambda v: str(v))
def test_fp64_small_states(L, d, periodic, n):
    print("fp64 small", L, d, periodic, n, flush=True)
    J, U, mu, Dl, K = 0.9, 0.7, 0.3, 0.4, 0.2
    ho, hl = O.Ham(L, d, periodic, J, U, mu, Dl, K), lib.ham(L, d, periodic, J, U, mu, Dl, K)
    pool = (W.pool(L, "all", periodic, TWO) if L > 1 else []) + W.site_ops(L, ONE)
    psi0 = W.random_state(L, d, seed=7 * L + d, dtype=np.complex128)
    dev = torch.from_numpy(np.ascontiguousarray(psi0)).to("cuda")
    ad = lib.Adapt64(hl, pool, dev, max_iters=100)
    ops, th = W.random_circuit(pool, n, seed=n + d)
    h_norm = L * (2 * J * d + 2 * Dl * d + (U / 2 + K) * d * d + mu * d)
    tol = 2 * n * 4.4e-16 * d * h_norm
    Eo, go, _ = O.energy_and_grad_adjoint(ho, psi0, ops, th)
    for _ in range(2):
        E, g = ad.energy_grad(ops, th)
        assert abs(E - Eo) <= tol, (E, Eo, tol)
        assert np.abs(g - go).max() <= 2 * d * d * tol * 2, (np.abs(g - go).max(), tol)
    assert ad.energy_grad(ops, th, grad=False)[0] == E
    E0, _ = ad.energy_grad([], [])
    assert abs(E0 - O.energy_of(ho, psi0, [], [])) <= 1e-14 * h_norm
    ad.close()
