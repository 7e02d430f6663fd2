"""Square grids: the energy's row and column blocks go in one launch, and from 1024^2 on the norm and the
check of a new state read eight points per thread at a time.  Against the FP64 oracle on the same rounded
state, at every square size with its own instantiation: both sides sum in fp64, so the energies agree to
1e-11 and the norms to 1e-12, relative, as for the rectangular grids; and a value that is not finite is
found wherever it stands."""
import os

import numpy as np
import pytest

from oracle import OracleGPE
from workloads import Params, gaussian_state, round_to_c64

pytestmark = pytest.mark.gpu

WORKERS = max(1, min(16, len(os.sched_getaffinity(0))))


@pytest.fixture(scope="module")
def sgpe():
    import paper_2010_15069_amd as m
    if m.device_count() <= 0:
        pytest.skip("no HIP device")
    return m


def _case(n, seed):
    p = Params(nx=n, ny=n, xmax=7.0, ymax=9.0, g_uu=5.0, g_dd=2.0, g_ud=3.0, k_l=1.1, omega=0.8,
               delta=-0.3, wx=1.2, wy=0.9)
    rng = np.random.default_rng(seed)
    noise = rng.standard_normal((2, 2, n, n))
    return p, gaussian_state(p, sigma=2.0, noise=0.0) * (1.0 + 0.2 * (noise[0] + 1j * noise[1]))


@pytest.mark.parametrize("precision", ["c64", "c128"])
@pytest.mark.parametrize("n", [16, 32, 64, 128, 512, 1024, 2048])
def test_square_energy_and_norm(sgpe, n, precision):
    p, psi = _case(n, n)
    if precision == "c64":
        psi = round_to_c64(psi)
    o = OracleGPE(p, workers=WORKERS)
    o.set_psi(psi)
    s = sgpe.Solver(p, precision=precision).set_psi(psi)
    e, eo = s.energy(), o.energy()
    assert abs(e - eo) <= 1e-11 * abs(eo), (e, eo)
    assert abs(s.norm() - o.norm()) <= 1e-12 * o.norm()
    s.close()


@pytest.mark.parametrize("n", [512, 1024])
@pytest.mark.parametrize("where", [0, 0.37, 1])
def test_a_value_that_is_not_finite_is_found(sgpe, n, where):
    torch = pytest.importorskip("torch")
    p, psi = _case(n, 7)
    t = np.ascontiguousarray(np.stack([psi[0].real, psi[0].imag, psi[1].real, psi[1].imag], axis=-1),
                             dtype=np.float32)
    s = sgpe.Solver(p).set_psi_device(torch.from_numpy(t).cuda())
    t.reshape(-1, 4)[int(where * (n * n - 1)), 3] = np.inf
    with pytest.raises(sgpe.SgpeError) as e:
        s.set_psi_device(torch.from_numpy(t).cuda())
    assert e.value.status == 4
    s.close()


@pytest.mark.parametrize("precision", ["c64", "c128"])
def test_square_energy_and_norm_256(sgpe, precision):
    # the square size between those above
    test_square_energy_and_norm(sgpe, 256, precision)
