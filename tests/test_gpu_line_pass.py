"""Real-time steps by line passes: one sweep per step, rows and columns in turn.  The oracle, for 1 to 3
steps (the pass after the leading one, an even and an odd number of alternations), at the shortest and
longest lines of either axis, in both precisions, for every real-space form and for R-K-R; and the bits
of a call that completes itself against one whose last half-step waits."""
import numpy as np
import pytest

from oracle import OracleGPE
from workloads import Params, gaussian_state

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    import paper_2010_15069_amd as m
    if m.device_count() <= 0 or not torch.cuda.is_available():
        pytest.skip("no HIP device")
    return torch, m


# a state of relative rounding 2^-24 (2^-53) per pass and about 20 roundings per transform level: a few
# steps stay well below 1e-6 (1e-13)
TOL = {"c64": 1e-6, "c128": 1e-13}
CASES = [(16, 16), (16, 64), (4096, 16), (16, 4096), (32, 2048), (1024, 32), (256, 512)]


@pytest.mark.parametrize("form", ["diagonal", "raman", "nln", "rkr", "rkr_nln"])
@pytest.mark.parametrize("nx,ny", CASES)
@pytest.mark.parametrize("precision", ["c64", "c128"])
def test_a_few_steps(env, precision, nx, ny, form):
    torch, m = env
    if precision == "c128" and form not in ("diagonal", "raman"):
        pytest.skip("complex128 runs the default split")
    p = Params(nx=nx, ny=ny, xmax=8.0, ymax=6.0, g_uu=30.0, g_dd=20.0, g_ud=10.0, k_l=1.3, omega=0.7, delta=0.2,
               wx=1.0, wy=1.4, omega_r0=0.0 if form == "diagonal" else 1.5, omega_rw=2.0, dt=2e-3)
    split = {"nln": ("krk", "nln"), "rkr": ("rkr", "frozen"), "rkr_nln": ("rkr", "nln")}.get(form, ("krk", "frozen"))
    psi = gaussian_state(p, sigma=1.5, seed=nx + 3 * ny, noise=1e-2).astype(np.complex64).astype(complex)
    ref = OracleGPE(p)
    ref.set_splitting(*split)
    dtype = torch.float64 if precision == "c128" else torch.float32
    for n in (1, 2, 3):
        print(f"case: {precision} {nx}x{ny} {form}, {n} real steps", flush=True)
        own = m.Solver(p, precision=precision)
        buf = torch.zeros((ny, nx, 4), dtype=dtype, device="cuda")
        torch.cuda.synchronize()
        lent = m.Solver(p, precision=precision, psi_dev=buf.data_ptr())
        if precision == "c64":
            own.set_splitting(*split)
            lent.set_splitting(*split)
        g = own.set_psi(psi).step_real(n).get_psi()
        ref.set_psi(psi)
        ref.step_real(n)
        err = np.linalg.norm(g - ref.psi) / np.linalg.norm(ref.psi)
        assert err <= TOL[precision], (n, err)
        assert np.array_equal(lent.set_psi(psi).step_real(n).get_psi(), g), n


@pytest.mark.parametrize("form", ["diagonal", "raman", "nln", "rkr", "rkr_nln"])
@pytest.mark.parametrize("precision,scale", [("c64", 1e18), ("c128", 1e152)])
def test_large_values_of_a_linear_problem(env, precision, scale, form):
    # without interactions a step is linear in the state, so it may be as large as its densities allow
    # (n = 1e36 in complex64, 1e304 in complex128): a pass must not form them of larger values than these
    torch, m = env
    if precision == "c128" and form not in ("diagonal", "raman"):
        pytest.skip("complex128 runs the default split")
    p = Params(nx=256, ny=256, xmax=8.0, ymax=6.0, g_uu=0.0, g_dd=0.0, g_ud=0.0, k_l=1.3, omega=0.7, delta=0.2,
               wx=1.0, wy=1.4, omega_r0=0.0 if form == "diagonal" else 1.5, omega_rw=2.0, dt=2e-3)
    split = {"nln": ("krk", "nln"), "rkr": ("rkr", "frozen"), "rkr_nln": ("rkr", "nln")}.get(form, ("krk", "frozen"))
    psi = gaussian_state(p, sigma=1.5, seed=5, noise=1e-2)
    psi = (psi / abs(psi).max()).astype(np.complex64).astype(complex)
    ref = OracleGPE(p)
    ref.set_splitting(*split)
    ref.set_psi(psi)
    ref.step_real(3)
    print(f"case: {precision} {form}, values up to {scale:g}", flush=True)
    s = m.Solver(p, precision=precision)
    if precision == "c64":
        s.set_splitting(*split)
    # the library's own rounding of scale psi: the scale is a power of two
    scale = 2.0 ** np.floor(np.log2(scale))
    g = s.set_psi(psi * scale).step_real(3).get_psi() / scale
    err = np.linalg.norm(g - ref.psi) / np.linalg.norm(ref.psi)
    assert err <= TOL[precision], err
