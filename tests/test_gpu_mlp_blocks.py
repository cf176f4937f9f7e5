"""The network's training pass at the edges of its split over workgroups: full and
ragged blocks of 16 rows, one, two and four blocks a workgroup, the row count in
and beyond the kernel, inputs that are not 16-byte aligned, rows without targets.
Tolerances as in test_gpu_mlp.py (loss 1e-5, every parameter block 1e-2: flips of
bf16 roundings)."""

import numpy as np
import pytest
import torch

import workload as W
from oracle import mlp_oracle as M
from paper_2606_05297_amd import lib

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 15, 16, 17, 4096, 4097, 8192, 8193, 12289])
def test_training_pass_at_block_edges(B):
    print("mlp blocks", B, flush=True)
    rng = np.random.default_rng(B)
    p = W.mlp_init(7) * 1.5
    X = np.stack([rng.uniform(0.5, 1.5, B), rng.uniform(0, 1, B), rng.uniform(0, 0.5, B), rng.integers(1, 65, B) / 64.0],
                 axis=1).astype(np.float32)
    T = rng.normal(0, 0.4, size=(B, 64)).astype(np.float32)
    n = rng.integers(-1, 70, size=B).astype(np.int32)  # below 0 and above 64: clamped
    n[0] = 33
    Lr, gr = M.loss_and_grad(p.astype(np.float64), X.astype(np.float64), T.astype(np.float64), np.clip(n, 0, 64))
    net = lib.Mlp(B, p)
    pad = torch.empty(B * 4 + 1, device="cuda")
    Xd = pad[1:].view(B, 4)  # 4-byte aligned only
    Xd.copy_(torch.from_numpy(X))
    args = Xd, torch.from_numpy(T).cuda(), torch.from_numpy(n).cuda()
    for _ in range(2):
        L, g = net.loss_grad(*args)
        assert abs(L - Lr) <= 1e-5 * Lr
        o = 0
        for name, shape in M.SHAPES:
            k = int(np.prod(shape))
            a, b = g[o:o + k].astype(np.float64), gr[o:o + k]
            assert np.linalg.norm(a - b) <= 1e-2 * np.linalg.norm(b), name
            o += k
    assert net.loss_grad(*args, grad=False)[0] == L
    net.close()
