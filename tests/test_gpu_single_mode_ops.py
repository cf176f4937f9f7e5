"""A single-mode op's j is not read: whatever a caller leaves in it (0, a mode, a
number that is no mode), the results are those of j = -1, bit for bit, on every
path that takes a circuit."""
import numpy as np
import pytest
import torch

import workload as W
from paper_2606_05297_amd import lib

pytestmark = pytest.mark.gpu

JS = (0, 1, 3, 23, 77, 255, 2000000000, -5)


def with_j(ops, j):
    return [(t, i, j if t in ("KERR", "ROT", "SR", "SI") else k) for t, i, k in ops]


def circuit(L, types, n=24):
    pool = W.pool(L, "all", False, ("HR", "PI", "CK")) + W.site_ops(L, types)
    ops, th = W.random_circuit(pool, n, seed=L)
    # phase gates alone among two-mode gates: members of fused runs
    ops[2], ops[7] = ("KERR", L // 2, -1), ("ROT", 0, -1)
    return ops, th


# the one-launch evaluation, fused runs, gate by gate
@pytest.mark.parametrize("L,d", [(4, 4), (4, 6), (6, 6), (5, 8), (4, 9)])
def test_complex64(L, d):
    print("[case] complex64", L, d, flush=True)
    h = lib.ham(L, d, False, 1.0, 0.7, 0.2, 0.3, 0.1)
    ops, th = circuit(L, ("KERR", "ROT", "SR", "SI"))
    x = torch.from_numpy(W.random_state(L, d, seed=3)).cuda()
    a, b = torch.empty_like(x), torch.empty_like(x)
    ws = lib.workspace(h, len(ops), len(ops))

    def run(o):
        E, n2, g = lib.energy_grad_adjoint(h, o, th, x, a, b, ws)
        E1, _, _ = lib.energy_grad_adjoint(h, o, th, x, a, b, ws, grad=False)
        psi = a.cpu().numpy()
        return np.concatenate([[E, n2, E1], g, lib.adjoint_sweep(h, o, th, a, b, n2, ws)]), psi

    r0, p0 = run(ops)
    for j in JS:
        r, p = run(with_j(ops, j))
        assert np.array_equal(r, r0) and np.array_equal(p, p0), j


@pytest.mark.parametrize("L,d", [(3, 5), (4, 4), (4, 8), (2, 9)])
def test_complex128(L, d):
    print("[case] complex128", L, d, flush=True)
    h = lib.ham(L, d, False, 1.0, 0.7, 0.2, 0.3, 0.1)
    ops, th = circuit(L, ("KERR", "ROT", "SR", "SI"))
    x = torch.from_numpy(W.random_state(L, d, seed=3, dtype=np.complex128)).cuda()
    pool = W.pool(L, "all", False, ("HR", "PI", "CK")) + W.site_ops(L, ("KERR", "ROT", "SR", "SI"))
    ref, steps = None, None
    for j in (-1,) + JS:
        ad = lib.Adapt64(h, with_j(pool, j), x, max_iters=30)
        E, g = ad.energy_grad(with_j(ops, j), th)
        s = [(r["k_sel"], r["E"], r["g_norm2"]) for r in (ad.step(), ad.step())]
        ad.close()
        if ref is None:
            ref, steps = np.concatenate([[E], g]), s
        assert np.array_equal(np.concatenate([[E], g]), ref) and s == steps, j


@pytest.mark.parametrize("L,d", [(4, 4), (6, 6)])
def test_drivers(L, d):
    """ADAPT and the batched sweep with phase gates in the pool and the warm-up layer."""
    print("[case] drivers", L, d, flush=True)
    h = lib.ham(L, d, True, 1.0, 4.0)
    x = torch.zeros(d ** L, dtype=torch.complex64, device="cuda")
    x[W.fock_index(L, d, [1] * L)] = 1
    pool = W.pool(L, "nn", True, ("HR", "HI")) + W.site_ops(L, ("KERR", "ROT"))
    warm = W.warmup_ops(L, True)
    th = W.warmup_theta0(len(warm), 3)
    ref = None
    for j in (-1, 0, 77):
        w, p = with_j(warm, j), with_j(pool, j)
        a = lib.Adapt(h, p, x, max_iters=4, warm_ops=w, warm_theta0=th)
        sw = lib.Sweep([dict(ham=h, pool=p, psi0=x, warm_ops=w, warm_theta0=th)], max_iters=4)
        r, s = a.step(), sw.step()[0][0]
        got = [(v["k_sel"], v["E"], v["bfgs_evals"]) for v in (a.warm_report(), sw.warm_reports()[0], r, s)]
        a.close()
        sw.close()
        ref = ref or got
        assert got == ref, (j, got, ref)
