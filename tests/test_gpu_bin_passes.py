"""The binning passes with four particles per thread (2^20 particles and more) and with
one (below), with the empty blocks that round a grid up to a multiple of eight (24^3: 54
full blocks of 256, 56 launched; no supported size has a partial block): the density equals
the oracle's, and the mass deposit of both forms is exact in sum."""
import numpy as np
import pytest
import torch

import paper_1301_0322_amd as cola
from gpu_util import announce
from oracle.pm import cic_deposit
from paper_1301_0322_amd import inputs

pytestmark = pytest.mark.gpu


# 24^3 = 13.5 blocks of 1024 and 54 of 256; 96^3 just below 2^20, 128^3 above it
@pytest.mark.parametrize("np_side,nm", [(24, 48), (96, 96), (128, 128)])
def test_binning_matches_oracle(np_side, nm):
    announce(f"binning {np_side}/{nm}")
    box = 40.0
    s = inputs.displacements(np_side, box, 41, rms=3.0)
    ref = cic_deposit(torch.from_numpy(s.astype(np.float64)).reshape(3, np_side, np_side, np_side), np_side, nm,
                      box).reshape(-1).numpy()
    with cola.Plan(cola.Config(np=np_side, nm=nm, box=box)) as plan:
        ws = plan.workspace()
        ws.fill_(float("nan"))
        rho = torch.full((nm**3,), float("nan"), device="cuda")
        plan.density(torch.from_numpy(s).cuda(), rho, ws)
        got = rho.cpu().numpy().astype(np.float64)
    tmax = np.abs(s).max() * nm / box + 0.5
    assert (np.abs(got - ref) <= 1e-5 * ref + 8 * (nm / np_side) ** 3 * tmax * 2.0**-22).all()
    assert abs(got.sum() / nm**3 - 1.0) < 1e-6
