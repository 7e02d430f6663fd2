"""The real-space exponential's small-angle and general forms in imaginary time: trap and coupling scales
that put every wave in the small form, every wave in the general one, and waves on both sides of the
limits (h V up to 0.1, 1 and 6; h |B| up to 0.02 and 0.4), in both precisions and for every real-space
form, against the oracle.

Tolerance: ten steps of at most 0.5e-6 (complex64) and 1e-14 (complex128) relative rounding each, which
imaginary time does not amplify over so few steps."""
import numpy as np
import pytest

from oracle import OracleGPE
from workloads import Params, gaussian_state

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def Solver():
    from paper_2010_15069_amd import Solver, device_count
    if device_count() <= 0:
        pytest.skip("no HIP device")
    return Solver


@pytest.mark.parametrize("trap", [0.1, 1.0, 6.0])
@pytest.mark.parametrize("form", ["diagonal", "nln_diagonal", "raman_small", "raman", "nln_raman"])
@pytest.mark.parametrize("precision", ["c64", "c128"])
def test_forms_agree_with_the_oracle(Solver, precision, form, trap):
    if precision == "c128" and form.startswith("nln"):
        pytest.skip("complex128 runs the default split")
    h = 5e-3
    w = np.sqrt(trap / h / 64.0)    # h V = trap at the corners of the box [-8, 8)^2
    omega = {"raman_small": 0.04 / h, "raman": 0.8 / h, "nln_raman": 0.8 / h}.get(form, 0.0)
    p = Params(nx=128, ny=64, xmax=8.0, ymax=8.0, g_uu=9.0, g_dd=7.0, g_ud=5.0, k_l=1.2, omega=0.5, delta=0.4, wx=w, wy=w,
               omega_r0=omega, omega_rw=2.0, dt=h)
    psi = gaussian_state(p, sigma=3.0, seed=3, noise=1e-2).astype(np.complex64).astype(complex)
    print(f"case: {precision} {form}, h V up to {trap}", flush=True)
    o = OracleGPE(p)
    s = Solver(p, precision=precision)
    if form.startswith("nln"):
        o.set_splitting("krk", "nln")
        s.set_splitting("krk", "nln")
    o.set_psi(psi)
    o.step_imag(10)
    g = s.set_psi(psi).step_imag(10).get_psi()
    err = np.linalg.norm(g - o.psi) / np.linalg.norm(o.psi)
    assert err <= (5e-6 if precision == "c64" else 1e-13), err
