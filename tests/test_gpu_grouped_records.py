"""Whole runs, resident steps and single steps equal each other bit for bit.  The runs at
(24, 48), (16, 32), (16, 48), (32, 64), (32, 128), (192, 384) and (384, 768) keep the state
in tile-sorted copies, whose gather writes each wave's records grouped by the tile they move
to; the other runs, and all steps, work on Lagrangian-order arrays (both forms at the same
sizes: test_gpu_run_forms.py).  One tile along an axis, tiles with less than a wave, with
several batches and on the crowded list, and depths that make 256- and 512-thread tile
blocks."""
import pytest
import torch

import paper_1301_0322_amd as cola
from gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("np_side,nm,depth,box", [
    (16, 16, 16, 20.0), (24, 48, 8, 10.0), (32, 32, 32, 5.0), (48, 192, 64, 60.0), (64, 64, 64, 8.0), (96, 96, 32, 30.0),
    (16, 32, 32, 4.0), (16, 48, 16, 20.0), (32, 64, 64, 6.0), (32, 128, 8, 30.0), (192, 384, 32, 40.0), (384, 768, 64, 80.0)])
def test_grouped_records_equal_fresh_packing(np_side, nm, depth, box):
    announce(f"grouped records {np_side}/{nm} depth {depth} box {box}")
    cfg = cola.Config(np=np_side, nm=nm, box=box, n_steps=4)
    n = np_side**3
    w = torch.randn(n, generator=torch.Generator().manual_seed(np_side + nm)).cuda()
    out = {}
    for mode in ("run", "resident", "fresh"):
        with cola.Plan(cfg) as plan:
            plan.set_bin_depth(depth)
            ws = plan.workspace()
            p = cola.Particles.empty(np_side)
            x = torch.empty((3, n), device="cuda")
            v = torch.empty_like(x)
            if mode == "run":
                plan.run(w, p, x, v, ws)
            else:
                plan.set_resident_steps(1 if mode == "resident" else 0)
                plan.init_2lpt(w, p, ws)
                for i in range(cfg.n_steps):
                    plan.step(i, p, ws)
                plan.finish(p, x, v, ws)
            torch.cuda.synchronize()
            out[mode] = [t.clone() for t in (x, v, p.s, p.v)]
    for a, b, c in zip(out["run"], out["resident"], out["fresh"]):
        assert torch.isfinite(a).all()
        assert torch.equal(a, c) and torch.equal(b, c)
