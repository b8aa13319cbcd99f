"""Shell sums of spectra with infinite modes, through the launcher that cola_cross_power
uses (densities are finite, so no public call reaches it with one): an infinite mode on an
axis or the diagonal, whose row the eight-fold symmetric sum loads twice and counts once,
makes its own shell infinite, never NaN, and leaves the other shells as they are."""
import ctypes

import numpy as np
import pytest
import torch

import paper_1301_0322_amd as cola
from gpu_util import announce

pytestmark = pytest.mark.gpu

_LAUNCH = "_ZN4cola18launch_shell_statsEiPK15HIP_vector_typeIfLj2EES3_PdldS4_P12ihipStream_t"


def _reference(n, fields):
    """Mode count and sums of |a|^2, |b|^2 and Re(a conj b) per shell in float64."""
    h = n // 2
    k = np.where(np.arange(n) <= h, np.arange(n), np.arange(n) - n)
    n2 = k[:, None, None] ** 2 + k[None, :, None] ** 2 + np.arange(h)[None, None, :] ** 2
    shell = np.rint(np.sqrt(n2)).astype(int)
    weight = np.broadcast_to(np.where(np.arange(h) > 0, 2.0, 1.0), n2.shape)
    a, b = (f.astype(np.float64) for f in fields)
    out = np.zeros((4, h))
    for r, v in enumerate((np.ones(n2.shape), (a * a).sum(-1), (b * b).sum(-1), (a * b).sum(-1))):
        for s in range(1, h):
            m = shell == s
            out[r, s] = (weight[m] * v[m]).sum()
    return out


@pytest.mark.parametrize("mode", [(0, 3, 2), (3, 0, 2), (4, 4, 1), (0, 0, 5), (-5, 0, 0), (2, -3, 1)])
@pytest.mark.parametrize("n", [16, 24])
def test_infinite_mode_stays_in_its_shell(n, mode):
    announce(f"infinite mode {mode} at n={n}")
    h = n // 2
    rng = np.random.default_rng(n)
    fields = [rng.standard_normal((n, n, h, 2)).astype(np.float32) for _ in range(2)]
    x, y, kz = mode
    fields[0][x % n, y % n, kz, 0] = np.inf
    fields[1][x % n, y % n, kz, 0] = 1.0
    fields[1][x % n, y % n, kz, 1] = 1.0
    ref = _reference(n, fields)
    lib = ctypes.CDLL(cola.LIB_PATH)
    launch = getattr(lib, _LAUNCH)
    launch.restype = ctypes.c_int
    launch.argtypes = [ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_long,
                       ctypes.c_double, ctypes.c_void_p, ctypes.c_void_p]
    a, b = (torch.from_numpy(f).cuda() for f in fields)
    part = torch.full((16 * 4 * h,), float("nan"), dtype=torch.float64, device="cuda")
    out = torch.full((6, h), float("nan"), dtype=torch.float64, device="cuda")
    assert launch(n, a.data_ptr(), b.data_ptr(), part.data_ptr(), part.numel(), 1.0, out.data_ptr(),
                  torch.cuda.current_stream().cuda_stream) == 0
    got = out.cpu().numpy()
    assert np.array_equal(got[0], ref[0])
    hit = np.isinf(ref[1])
    assert hit.sum() == 1
    count = np.maximum(ref[0], 1.0)
    for row in (1, 2, 3):
        want = ref[row] / count
        assert np.array_equal(np.isinf(got[row]), np.isinf(want)), row
        fin = np.isfinite(want)
        # FP64 sums in another order: some 1e3 terms
        assert np.allclose(got[row][fin], want[fin], rtol=1e-11, atol=1e-11), row
    assert got[1][hit] == np.inf
