"""Column tiles of 4, 8 and 16 at the mesh lengths whose 16-wide (384) or 16- and 4-wide
(1024) tiles exchange real and imaginary parts in turn: the force of each width equals the
others' bit for bit, and the 384 one the oracle's."""
import numpy as np
import pytest
import torch

import paper_1301_0322_amd as cola
from gpu_util import announce
from oracle import pm as opm
from paper_1301_0322_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("np_side,nm", [(16, 384), (16, 1024)])
def test_column_widths_agree(np_side, nm):
    box = 50.0
    s = inputs.displacements(np_side, box, seed=nm, rms=2.0)
    with cola.Plan(cola.Config(np=np_side, nm=nm, box=box)) as plan:
        ws = plan.workspace()
        sd = torch.from_numpy(s).cuda()
        first = None
        for width in (0, 4, 8, 16):
            announce(f"column width {width} at {nm}")
            plan.set_fft_tile(0, width)
            acc = torch.full((3, np_side**3), float("nan"), device="cuda")
            plan.pm_force(sd, 0.5, acc, ws)
            first = acc if first is None else first
            assert torch.isfinite(acc).all() and torch.equal(acc, first), width
        got = first.cpu().numpy()
        del ws
        torch.cuda.empty_cache()
    if nm == 384:
        st = torch.from_numpy(s.astype(np.float64)).reshape(3, np_side, np_side, np_side)
        ref = opm.pm_force(st, 0.5, np_side, nm, box, 0.3).reshape(3, -1).numpy()
        # the bar of the repository's force tests
        assert np.linalg.norm(got - ref) <= 1e-5 * np.linalg.norm(ref)
