"""Shell statistics at mesh sizes whose half length is below a block's 16 reduced shells,
not a multiple of them, and larger (nm = 16, 24, 96, 256), with and without a second set
and with every column width of the x pass: mode counts exact, spectra at the bars of the
repository's cross-spectrum test (1e-5 of sqrt(P_aa P_bb) plus an FP32 floor)."""
import numpy as np
import pytest
import torch

import paper_1301_0322_amd as cola
from gpu_util import announce
from oracle import power
from oracle.pm import cic_deposit
from paper_1301_0322_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("np_side,nm", [(16, 16), (24, 24), (32, 96), (64, 256)])
def test_shell_statistics_match_oracle(np_side, nm):
    announce(f"shell statistics {np_side}/{nm}")
    box = 40.0
    sa = inputs.displacements(np_side, box, 31, rms=1.0)
    sb = (sa + inputs.displacements(np_side, box, 32, rms=0.4)).astype(np.float32)
    da, db = (cic_deposit(torch.from_numpy(s.astype(np.float64)).reshape(3, np_side, np_side, np_side), np_side, nm, box)
              - 1.0 for s in (sa, sb))
    pa, pb, px, cnt = (t[: nm // 2 - 1].numpy() for t in power.cross_power_from_delta(da, db, box))
    scale, floor = np.sqrt(pa * pb), 1e-7 * pa.max()
    with cola.Plan(cola.Config(np=np_side, nm=nm, box=box)) as plan:
        ws = plan.workspace()
        for width in (0, 4, 8):
            if width and (nm // 2) % width:
                continue
            plan.set_fft_tile(1, width)
            out = torch.full((6, nm // 2), float("nan"), dtype=torch.float64, device="cuda")
            ws.fill_(float("nan"))
            plan.cross_power(torch.from_numpy(sa).cuda(), torch.from_numpy(sb).cuda(), out, ws)
            got = out.cpu().numpy()
            assert np.array_equal(got[0, 1:], cnt) and not got[:, 0].any()
            for row, ref in ((1, pa), (2, pb), (3, px)):
                assert (np.abs(got[row, 1:] - ref) <= 1e-5 * scale + floor).all(), (row, width)
        auto = torch.full_like(out, float("nan"))
        plan.cross_power(torch.from_numpy(sa).cuda(), None, auto, ws)
        assert np.array_equal(auto[0].cpu().numpy(), got[0]) and not auto[2:].any()
        assert np.allclose(auto[1].cpu().numpy(), got[1], rtol=1e-12, atol=0)
