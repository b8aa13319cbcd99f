"""cola_autotune with a workspace that holds the sorted positions and forces of a step and with
one that holds only the binning buffers: it stays inside the bytes it is given and the tuned
plan's run equals the default's."""
import ctypes

import pytest
import torch

import paper_1301_0322_amd as cola
from gpu_util import announce

pytestmark = pytest.mark.gpu


def _run(plan, w):
    p = cola.Particles.empty(plan.cfg.np)
    x, v = torch.empty_like(p.s), torch.empty_like(p.s)
    plan.run(w, p, x, v, plan.workspace())
    torch.cuda.synchronize()
    return x, v


@pytest.mark.parametrize("np_side,nm", [(16, 48), (32, 64), (64, 64)])
@pytest.mark.parametrize("room", ["full", "lists"])
def test_autotune_stays_in_its_workspace(np_side, nm, room):
    announce(f"autotune {np_side}/{nm} {room}")
    cfg = cola.Config(np=np_side, nm=nm, box=0.5 * np_side, n_steps=2)
    w = torch.randn(np_side**3, generator=torch.Generator().manual_seed(nm)).cuda()
    with cola.Plan(cfg) as plan:
        ref = _run(plan, w)
        p = cola.Particles.empty(np_side)
        plan.init_2lpt(w, p, plan.workspace())
        need = ctypes.c_size_t()
        assert cola.lib().cola_tuning_workspace_bytes(plan._c, ctypes.byref(need)) == 0
        size = need.value // 4 - (8 * np_side**3 + 4 if room == "lists" else 0)
        ws = torch.full((size + 4096,), -7.0, device="cuda")
        used = ctypes.c_int32(-1)
        cp = p.to_c()
        status = cola.lib().cola_autotune(plan._c, ctypes.byref(cp), ws.data_ptr(), 4 * size,
                                          torch.cuda.current_stream().cuda_stream, None, ctypes.byref(used))
        assert status == 0 and used.value == 0
        torch.cuda.synchronize()
        assert bool((ws[size:] == -7.0).all())
        y, x, depth = plan.get_tuning()
        assert y in (4, 8, 16) and x in (4, 8, 16) and depth in (8, 16, 32, 64) and nm % depth == 0
        for a, b in zip(ref, _run(plan, w)):
            assert torch.isfinite(a).all() and torch.equal(a, b)
