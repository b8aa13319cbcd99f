"""Steps on Lagrangian-order arrays (tile-sorted positions, forces back in Lagrangian order,
a streaming kick): one particle and four per scatter thread, a grid that is not a multiple of
eight blocks, every bin depth's key, and the variants of the kick, against whole runs bit
for bit (tile-sorted ones at (16, 32) and (32, 128), Lagrangian ones at the other sizes); the
checkpoints equal the displacements after each step."""
import pytest
import torch

import paper_1301_0322_amd as cola
from gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("np_side,nm,depth,flags", [
    (16, 32, 8, 0), (24, 24, 8, cola.COLA_FLAG_KDK_STD), (48, 96, 16, cola.COLA_FLAG_U1_DRIFT),
    (32, 128, 64, cola.COLA_FLAG_NO_LPT_FRAME), (128, 128, 32, 0)])
def test_steps_and_checkpoints_equal_run(np_side, nm, depth, flags):
    announce(f"lagrangian steps {np_side}/{nm} depth {depth} flags {flags}")
    cfg = cola.Config(np=np_side, nm=nm, box=0.6 * np_side, n_steps=3, flags=flags)
    n = np_side**3
    w = torch.randn(n, generator=torch.Generator().manual_seed(nm)).cuda()
    with cola.Plan(cfg) as plan:
        plan.set_bin_depth(depth)
        ws = plan.workspace()
        p = cola.Particles.empty(np_side)
        x, v = torch.empty((3, n), device="cuda"), torch.empty((3, n), device="cuda")
        plan.run(w, p, x, v, ws)
        ref = [t.clone() for t in (x, v, p.s, p.v, p.s1, p.s2)]
        ckpt = torch.full((cfg.n_steps + 1, 3, n), float("nan"), device="cuda")
        ws.fill_(float("nan"))
        plan.run_checkpointed(w, p, x, v, ckpt, ws)
        for a, b in zip(ref, (x, v, p.s, p.v, p.s1, p.s2)):
            assert torch.equal(a, b)
        for resident in (0, 1):
            plan.set_resident_steps(resident)
            ws.fill_(float("nan"))
            plan.init_2lpt(w, p, ws)
            for i in range(cfg.n_steps):
                assert torch.equal(p.s, ckpt[i])
                plan.step(i, p, ws)
            assert torch.equal(p.s, ckpt[cfg.n_steps])
            plan.finish(p, x, v, ws)
            for a, b in zip(ref, (x, v, p.s, p.v, p.s1, p.s2)):
                assert torch.equal(a, b)
