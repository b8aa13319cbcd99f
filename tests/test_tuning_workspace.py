"""The autotuner's workspace holds the meshes, the deepest binning buffers and the sorted
positions and forces that a step's force evaluation uses (host-only)."""
import ctypes

import pytest

import paper_1301_0322_amd as cola


@pytest.mark.parametrize("np_side,nm", [(16, 16), (32, 64), (64, 64), (128, 384), (256, 512)])
def test_tuning_workspace_holds_sorted_positions_and_forces(np_side, nm):
    need = ctypes.c_size_t()
    with cola.Plan(cola.Config(np=np_side, nm=nm)) as p:
        assert cola.lib().cola_tuning_workspace_bytes(p._c, ctypes.byref(need)) == 0
        worst = 0
        for depth in (8, 16, 32, 64):
            if nm % depth == 0:
                p.set_bin_depth(depth)
                # workspace = meshes, binning buffers, 104 bytes a particle
                worst = max(worst, p.workspace_bytes() - 104 * np_side**3)
    assert need.value >= worst + 32 * np_side**3
