"""Resident steps keep a copy and bins only where that is faster than a plain step (nm >= 3 np;
nm = 2 np up to np = 128 or below 0.5 Mpc/h of particle spacing; nm = np up to 96, or up to
192 below 0.4): elsewhere every step bins the caller's arrays and a resident call makes the
plain call's launches.  Results equal the plain steps' bit for bit on both sides of the
lines."""
import pytest
import torch

import paper_1301_0322_amd as cola
from gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("np_side,nm,spacing,kept", [
    (32, 32, 2.0, True), (96, 96, 1.0, True), (128, 128, 0.3, True), (128, 128, 0.8, False), (128, 256, 1.0, True),
    (192, 384, 0.4, True), (192, 384, 1.0, False), (256, 256, 0.3, False), (128, 384, 2.0, True)])
def test_resident_steps_keep_state_where_it_pays(np_side, nm, spacing, kept):
    announce(f"resident steps at {np_side}/{nm}, spacing {spacing}")
    cfg = cola.Config(np=np_side, nm=nm, box=spacing * np_side, n_steps=3)
    w = torch.randn(np_side**3, generator=torch.Generator().manual_seed(nm)).cuda()
    out, counted = {}, {}
    with cola.Plan(cfg) as plan:
        ws = plan.workspace()
        for on in (0, 1):
            plan.set_resident_steps(on)
            p = cola.Particles.empty(np_side)
            x, v = torch.empty_like(p.s), torch.empty_like(p.s)
            plan.init_2lpt(w, p, ws)
            plan.trace_enable(1)
            for i in range(cfg.n_steps):
                plan.step(i, p, ws)
            plan.finish(p, x, v, ws)
            counted[on] = plan.trace_read()["bin_count"][1]
            plan.trace_enable(0)
            out[on] = [x, v, p.s, p.v]
    for a, b in zip(out[0], out[1]):
        assert torch.isfinite(a).all() and torch.equal(a, b)
    assert counted[0] == cfg.n_steps + 1
    assert counted[1] == (1 if kept else cfg.n_steps + 1)
