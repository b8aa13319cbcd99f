"""Both forms of cola_run's steps (state in tile-sorted copies, Lagrangian-order arrays) at
the same sizes, bit for bit against each other and against the steps one by one; the
tile-sorted form at every bin depth against the FP64 oracle.  Mesh ratios 1 to 4, np = nm on
both sides of the built-in line, one tile along an axis, tiles with less than a wave of
particles, with several batches and on the crowded list."""
import functools

import numpy as np
import pytest
import torch

import paper_1301_0322_amd as cola
from gpu_util import announce, periodic_max_err, rel_l2
from oracle import cola as ocola
from oracle import cosmology as cosmo
from paper_1301_0322_amd import inputs

pytestmark = pytest.mark.gpu


def _run(plan, w):
    p = cola.Particles.empty(plan.cfg.np)
    x = torch.full_like(p.s, float("nan"))
    v = torch.full_like(p.s, float("nan"))
    ws = plan.workspace()
    ws.fill_(float("nan"))
    plan.run(w, p, x, v, ws)
    torch.cuda.synchronize()
    return [x, v, p.s, p.v, p.s1, p.s2]


# (32, 64), (64, 64, 8.0) and (32, 32) have tiles with more particles than a block has
# threads; (16, 16) is one or two tiles along an axis
@pytest.mark.parametrize("np_side,nm,depth,box,flags", [
    (16, 16, 16, 20.0, 0), (24, 24, 8, 14.0, cola.COLA_FLAG_KDK_STD), (32, 32, 32, 5.0, 0), (64, 64, 64, 8.0, 0),
    (96, 96, 32, 30.0, 0), (128, 128, 32, 60.0, 0), (48, 96, 16, 29.0, cola.COLA_FLAG_U1_DRIFT),
    (48, 192, 64, 60.0, 0), (64, 192, 16, 30.0, cola.COLA_FLAG_NO_LPT_FRAME), (96, 384, 32, 40.0, 0),
    (32, 64, 8, 6.0, 0), (64, 128, 32, 100.0, 0), (16, 48, 16, 20.0, 0), (192, 192, 32, 60.0, 0),
    (512, 512, 32, 200.0, 0)])
def test_run_forms_agree(np_side, nm, depth, box, flags):
    announce(f"run forms {np_side}/{nm} depth {depth} box {box} flags {flags}")
    cfg = cola.Config(np=np_side, nm=nm, box=box, n_steps=3, flags=flags)
    w = torch.randn(np_side**3, generator=torch.Generator().manual_seed(np_side + 3 * nm)).cuda()
    with cola.Plan(cfg) as plan:
        plan.set_bin_depth(depth)
        plan.set_run_form(0)
        sorted_form = _run(plan, w)
        plan.set_run_form(1)
        lagrangian = _run(plan, w)
        for a, b in zip(sorted_form, lagrangian):
            assert torch.isfinite(a).all() and torch.equal(a, b)
        del lagrangian
        p = cola.Particles.empty(np_side)
        ws = plan.workspace()
        plan.init_2lpt(w, p, ws)
        for i in range(cfg.n_steps):
            plan.step(i, p, ws)
        x, v = torch.empty_like(p.s), torch.empty_like(p.s)
        plan.finish(p, x, v, ws)
        for a, b in zip(sorted_form, (x, v, p.s, p.v, p.s1, p.s2)):
            assert torch.equal(a, b)


@functools.lru_cache(maxsize=1)
def _oracle_run():
    w = inputs.white_noise(32, 22)
    rx, rv, _ = ocola.run(w.astype(np.float64), cosmo.Config(np_side=32, nm_side=64))
    return w, rx.reshape(3, -1).numpy(), rv.reshape(3, -1).numpy()


# the bars of the repository's other whole-run comparisons with the oracle
@pytest.mark.parametrize("depth", [8, 16, 32, 64])
@pytest.mark.parametrize("form", [0, 1])
def test_run_form_matches_oracle(form, depth):
    announce(f"run form {form} depth {depth} against the oracle")
    w, rx, rv = _oracle_run()
    cfg = cola.Config(np=32, nm=64)
    with cola.Plan(cfg) as plan:
        plan.set_run_form(form)
        plan.set_bin_depth(depth)
        x, v = (t.cpu().numpy() for t in _run(plan, torch.from_numpy(w).cuda())[:2])
    assert periodic_max_err(x, rx, cfg.box) < 1e-3 * cfg.box
    assert rel_l2(v, rv) < 1e-4
