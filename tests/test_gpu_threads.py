"""Calls that write their results into the calling thread's host buffer: objects
used in turn on one thread and from several threads at once, each on a stream of
its own, give the results they give alone, bit for bit."""
import threading

import numpy as np
import pytest
import torch

import workload as W
from paper_2606_05297_amd import lib

pytestmark = pytest.mark.gpu


def together(jobs):
    """Run the jobs at once, each on a thread and a stream of its own; their results."""
    out, err = [None] * len(jobs), []
    gate = threading.Barrier(len(jobs))

    def run(k):
        try:
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                gate.wait(timeout=60)
                out[k] = [jobs[k]() for _ in range(6)]
        except Exception as e:  # noqa: BLE001
            err.append(e)

    torch.cuda.synchronize()
    ts = [threading.Thread(target=run, args=(k,)) for k in range(len(jobs))]
    for t in ts:
        t.start()
    for t in ts:
        t.join(timeout=90)
    assert not err, err
    return out


def network(seed, B):
    rng = np.random.default_rng(seed)
    X = torch.from_numpy(rng.normal(size=(B, 4)).astype(np.float32)).cuda()
    T = torch.from_numpy(rng.normal(size=(B, 64)).astype(np.float32)).cuda()
    nv = torch.from_numpy(rng.integers(0, 65, B).astype(np.int32)).cuda()
    net = lib.Mlp(B, W.mlp_init(seed))
    return lambda: np.concatenate([[net.loss_grad(X, T, nv, grad=False)[0]], *[np.atleast_1d(v) for v in
                                                                              net.loss_grad(X, T, nv)]])


def circuit(L, d, seed):
    h = lib.ham(L, d, False, 1.0, 0.5, 0.1, 0.3, 0.0)
    ops, th = W.random_circuit(W.pool(L, "all", False, ("HR", "PI")), 12, seed=seed)
    x = torch.from_numpy(W.random_state(L, d, seed=seed)).cuda()
    a, b = torch.empty_like(x), torch.empty_like(x)
    ws = lib.workspace(h, 0, 12)

    def run():
        E, n2, g = lib.energy_grad_adjoint(h, ops, th, x, a, b, ws)
        return np.concatenate([[E, n2], g])
    return run


def test_networks_and_circuits():
    print("[case] threads: networks, circuits", flush=True)
    jobs = [network(1, 70), network(2, 1000), network(3, 9000), circuit(4, 4, 1), circuit(6, 6, 2), circuit(5, 8, 3)]
    alone = [j() for j in jobs]
    for _ in range(2):  # in turn on one thread
        for j, want in zip(jobs, alone):
            assert np.array_equal(j(), want)
    for got, want in zip(together(jobs), alone):
        assert all(np.array_equal(g, want) for g in got)


def run64(L, d, seed, max_iters=20):
    h = lib.ham(L, d, False, 1.0, 0.5, 0.1, 0.3, 0.0)
    pool = W.pool(L, "all", False, ("HR", "PI", "CK")) + W.site_ops(L, ("SR", "KERR"))
    ops, th = W.random_circuit(pool, 18, seed=seed)
    x = torch.from_numpy(W.random_state(L, d, seed=seed, dtype=np.complex128)).cuda()
    ad = lib.Adapt64(h, pool, x, max_iters=max_iters)

    def run():
        E, g = ad.energy_grad(ops, th)
        return np.concatenate([[E, ad.energy_grad(ops, th, grad=False)[0]], g])
    return run


def test_complex128_and_others():
    print("[case] threads: complex128", flush=True)
    jobs = [run64(3, 4, 1), run64(3, 5, 2), run64(4, 6, 3), run64(3, 4, 4), network(4, 300), circuit(4, 4, 5)]
    alone = [j() for j in jobs]
    for j, want in zip(jobs, alone):
        assert np.array_equal(j(), want)
    for got, want in zip(together(jobs), alone):
        assert all(np.array_equal(g, want) for g in got)


def test_handles_made_on_one_thread_and_used_on_another():
    print("[case] threads: handles", flush=True)
    jobs = together([lambda: run64(3, 8, 1), lambda: run64(3, 7, 2), lambda: run64(3, 8, 3)])
    runs = [r for js in jobs for r in js[:2]]
    first = [r() for r in runs]
    for r, w in zip(runs, first):
        assert np.array_equal(r(), w)
    assert np.array_equal(first[0], first[1]) and np.array_equal(first[2], first[3])


def sweep_run(seed):
    entries = []
    for L, d in ((4, 4), (3, 8), (4, 6)):
        x = torch.zeros(d ** L, dtype=torch.complex64, device="cuda")
        x[W.fock_index(L, d, [1] * L)] = 1
        warm = W.warmup_ops(L, False)
        entries.append(dict(ham=lib.ham(L, d, False, 1.0, 1.0 + seed), pool=W.pool(L, "nn", False, W.BH_TYPES), psi0=x,
                            warm_ops=warm, warm_theta0=W.warmup_theta0(len(warm), seed)))
    torch.cuda.synchronize()

    def run():
        sw = lib.Sweep(entries, max_iters=3)
        r = sw.warm_reports() + sw.step()[0]
        sw.close()
        return np.array([[v["E"], v["k_sel"], v["bfgs_evals"]] for v in r])
    return run


def test_sweeps_at_once():
    """Rounds that write into the sweep's own host memory, from chains on side streams."""
    print("[case] threads: sweeps", flush=True)
    jobs = [sweep_run(1), sweep_run(2), circuit(4, 4, 6)]
    alone = [j() for j in jobs]
    for got, want in zip(together(jobs), alone):
        assert all(np.array_equal(g, want) for g in got)
