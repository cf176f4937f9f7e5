"""The order in which evaluations on real states run a circuit (host only): gates
move up to join a run of three modes where they commute with all that they pass."""
import numpy as np
import pytest

import workload as W
from paper_2606_05297_amd import lib


def order_from_definition(ops, top):
    """Each gate not yet taken starts a run; later gates inside one window of three
    consecutive modes at or below `top` join it (at most 8) unless they share a mode
    with a gate that has been passed."""
    left, out = list(range(len(ops))), []
    while left:
        a = left.pop(0)
        run, passed, rest = [a], set(), []
        ok = [o[2] == o[1] + 1 and o[2] <= top for o in ops]
        for b in left:
            los = [ops[k][1] for k in run] + [ops[b][1]]
            if (ok[a] and ok[b] and len(run) < 8 and not passed & set(ops[b][1:]) and max(los) - min(los) <= 1):
                run.append(b)
            else:
                rest.append(b)
                passed |= set(ops[b][1:])
        out += run
        left = rest
    return out


@pytest.mark.parametrize("layout,top", [(lib.LAYOUT_EVEN | lib.LAYOUT_REAL, 6), (lib.LAYOUT_REAL, 7)])
def test_order_and_launched_runs(layout, top):
    h = lib.ham(8, 8, layout=layout)
    rng = np.random.default_rng(3)
    pairs = W.pool(8, "all" if layout == lib.LAYOUT_REAL else "nn", False, ("HR", "PR"))
    for n in (0, 1, 2, 7, 20, 60):
        for _ in range(8):
            ops = [pairs[k] for k in rng.integers(0, len(pairs), n)]
            at = lib.real_fusion_order(h, ops)
            assert at == order_from_definition(ops, top)
            moved = [ops[k] for k in at]
            for m in range(8):  # gates that share a mode keep their order
                assert [k for k in at if m in ops[k][1:]] == [k for k in range(n) if m in ops[k][1:]]
            assert len(lib.real_fusion_plan(h, moved)) <= len(lib.real_fusion_plan(h, ops))


def test_small_states_keep_the_order_and_errors():
    small = lib.ham(6, 8)
    ops = [("PR", 0, 1), ("PR", 3, 4), ("HR", 0, 1)]
    assert lib.real_fusion_order(small, ops) == [0, 1, 2]
    h = lib.ham(8, 8, layout=lib.LAYOUT_REAL)
    for bad in ([("HI", 0, 1)], [("HR", 0, 8)]):
        with pytest.raises(lib.FockError):
            lib.real_fusion_order(h, bad)
    assert lib.load().fock_real_fusion_order(None, None, 0, None) == -1
