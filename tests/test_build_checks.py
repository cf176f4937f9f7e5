"""Checks of the device assembly at build time (host only)."""
import os

import pytest

from paper_2606_05297_amd import build

KERNEL = """
	.amdhsa_kernel {name}
		.amdhsa_group_segment_fixed_size {size}
		.amdhsa_private_segment_fixed_size 0
	.end_amdhsa_kernel
"""


def test_static_lds_of_every_kernel():
    text = KERNEL.format(name="a", size=0) + "s_endpgm\n" + KERNEL.format(name="b", size=2048)
    assert build.static_lds(text) == {"a": 0, "b": 2048}
    assert build.static_lds("") == {}


def test_run_kernels_with_static_lds_are_refused(monkeypatch, tmp_path):
    """check_mfma_operands on assembly as the compiler would write it."""
    monkeypatch.setattr(build, "BUILD", str(tmp_path))

    class Done:
        returncode, stdout, stderr = 0, "", ""

    def compiled(size):
        def run(cmd, **kw):
            with open(cmd[cmd.index("-o") + 1], "w") as f:
                f.write(KERNEL.format(name="k_tile_run", size=size))
            return Done()
        return run

    assert "tile_runs.hip" in build.LDS_FROM_ZERO and "tile_runs.hip" in build.MFMA_SOURCES
    monkeypatch.setattr(build.subprocess, "run", compiled(0))
    assert build.check_mfma_operands("tile_runs.hip") == 0
    monkeypatch.setattr(build.subprocess, "run", compiled(16))
    with pytest.raises(RuntimeError, match="k_tile_run has 16 bytes of static LDS"):
        build.check_mfma_operands("tile_runs.hip")
    assert build.check_mfma_operands("mlp_kernels.hip") == 0  # others may have some


def test_built_run_kernels_have_none():
    asm = os.path.join(build.BUILD, "tile_runs.s")
    if not os.path.exists(asm):
        pytest.skip("not built here")
    with open(asm) as f:
        sizes = build.static_lds(f.read())
    assert sizes and not any(sizes.values())
