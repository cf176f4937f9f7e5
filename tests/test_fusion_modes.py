"""The process-wide gate fusion mode (host only)."""
from paper_2606_05297_amd import lib


def test_default_and_range():
    L = lib.load()
    assert lib.get_gate_fusion() == lib.FUSE_AUTO
    for bad in (-1, 4):
        assert L.fock_set_gate_fusion(bad) == -1 and "mode" in lib.last_error()
    assert lib.get_gate_fusion() == lib.FUSE_AUTO
    try:
        for m in (lib.FUSE_OFF, lib.FUSE_FORWARD, lib.FUSE_ALL, lib.FUSE_AUTO):
            lib.set_gate_fusion(m)
            assert lib.get_gate_fusion() == m
    finally:
        lib.set_gate_fusion(lib.FUSE_AUTO)
