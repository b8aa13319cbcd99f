"""bench.py's bytes per launch follow the launches that a run makes: merged inverse passes up
to nm = 256, and the two forms of the steps.  Over a step they add up to the step's bytes,
plus, on Lagrangian-order arrays, the sorted positions and forces that form moves."""
import pytest

import bench
import paper_1301_0322_amd as cola


@pytest.mark.parametrize("np_side,nm", [(32, 64), (64, 128), (128, 256), (128, 384), (256, 512), (512, 1024)])
@pytest.mark.parametrize("lagrangian", [False, True])
def test_run_stage_bytes_add_up(np_side, nm, lagrangian):
    sb = bench.run_stage_bytes(np_side, nm, lagrangian)
    merged = nm <= 256
    launches = {"deposit": 1, "fft_z_fwd": 1, "fft_y_fwd": 1, "fft_x_poisson": 1, "fft_y_inv_pair": 1,
                "fft_z_inv": 1 if merged else 2, "gather_kick_drift": 1}
    if not merged:
        launches["fft_y_inv"] = 1
    if lagrangian:
        launches["gather_force"] = 1
    total = sum(sb[k] * n for k, n in launches.items())
    # positions of 16 instead of 12 bytes to the deposit and again to the gather (16), forces
    # out (16) and in (16): 4 + 16 + 16 + 16 bytes a particle
    assert total == bench.b_alg_step(np_side, nm) + (52 * np_side**3 if lagrangian else 0)
    assert ("fft_y_inv" in sb) == (not merged)
    assert ("unsort" in sb) == (not lagrangian)
    # every stage of the steps and the closing kick has its bytes
    for k in ("bin_count", "bin_scatter", "gather_finish"):
        assert sb[k] > 0


def test_default_workload_runs_on_sorted_copies():
    np_side, nm, box = bench.CONFIGS["c1"][:3]
    with cola.Plan(cola.Config(np=np_side, nm=nm, box=box)) as p:
        assert p.get_run_form() == 0
    np_side, nm, box = bench.CONFIGS["c4"][:3]
    with cola.Plan(cola.Config(np=np_side, nm=nm, box=box)) as p:
        assert p.get_run_form() == 1
