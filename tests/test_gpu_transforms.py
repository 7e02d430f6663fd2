"""The step kernels' transforms at every line length and number of points per lane (every sequence of
radices, rotated register orders included), along each axis: two real-time and two imaginary-time steps
of a rough state against the oracle.

Tolerance: a forward and inverse transform in fp32 return 1.4e-7 relative error at most (4096 points);
the calls hold about ten such pairs, whose roundings are independent: 1.4e-7 sqrt(10) = 4.5e-7 < 1e-6."""
import numpy as np
import pytest

from oracle import OracleGPE
from workloads import Params, gaussian_state

pytestmark = pytest.mark.gpu

CASES = [(n, p) for n in (16, 32, 64, 128, 256, 512, 1024, 2048, 4096) for p in (4, 8, 16) if p == 16 or n <= 1024]


@pytest.fixture(scope="module")
def Solver():
    from paper_2010_15069_amd import Solver, device_count
    if device_count() <= 0:
        pytest.skip("no HIP device")
    return Solver


@pytest.mark.parametrize("n,points", CASES)
@pytest.mark.parametrize("axis", ["x", "y"])
def test_every_length_and_points_per_lane(Solver, axis, n, points):
    nx, ny = (n, 32) if axis == "x" else (32, n)
    p = Params(nx=nx, ny=ny, xmax=8.0, ymax=7.0, g_uu=4.0, g_dd=3.0, g_ud=2.0, k_l=1.1, omega=0.6, delta=0.3, dt=1e-4)
    psi = gaussian_state(p, sigma=2.0, seed=n + points, noise=0.1).astype(np.complex64).astype(complex)
    s = Solver(p)
    s.set_schedule(**{f"{'row' if axis == 'x' else 'col'}_points": points}, col_tile=1)
    print(f"case: {nx}x{ny}, {points} points per lane along {axis}", flush=True)
    o = OracleGPE(p)
    o.set_psi(psi)
    o.step_real(2)
    o.step_imag(2)
    g = s.set_psi(psi).step_real(2).step_imag(2).get_psi()
    err = np.linalg.norm(g - o.psi) / np.linalg.norm(o.psi)
    assert err <= 1e-6, err


@pytest.mark.parametrize("nx,ny", [(1024, 2048), (512, 4096), (256, 2048)])
@pytest.mark.parametrize("raman", [0.0, 1.5])
def test_wide_column_workgroups(Solver, nx, ny, raman):
    # columns of 2048 and 4096 points on grids wide enough for two tiles per workgroup, and one that is
    # not; the same tolerance (a step of each kind)
    p = Params(nx=nx, ny=ny, xmax=8.0, ymax=7.0, g_uu=4.0, g_dd=3.0, g_ud=2.0, k_l=1.1, omega=0.6, delta=0.3,
               omega_r0=raman, omega_rw=2.0, dt=1e-4)
    psi = gaussian_state(p, sigma=2.0, seed=ny, noise=0.1).astype(np.complex64).astype(complex)
    print(f"case: {nx}x{ny}, raman {raman}", flush=True)
    o = OracleGPE(p, workers=8)
    o.set_psi(psi)
    o.step_real(1)
    o.step_imag(2)
    g = Solver(p).set_psi(psi).step_real(1).step_imag(2).get_psi()
    err = np.linalg.norm(g - o.psi) / np.linalg.norm(o.psi)
    assert err <= 1e-6, err


@pytest.mark.parametrize("nx,ny,tiles", [(1024, 2048, (1, 2, 4)), (512, 4096, (1, 2))])
@pytest.mark.parametrize("raman", [0.0, 1.5])
def test_an_explicit_column_tile_is_the_one_that_runs(Solver, nx, ny, tiles, raman):
    # the default's 1024-thread tile is a tile of the schedule: it is what get_schedule gives, a narrower
    # one can be had, and tiles do not change a point's arithmetic (imaginary time: the grouping of the
    # norm's fp64 partials, rel. 1e-6 as for the narrower grids)
    p = Params(nx=nx, ny=ny, xmax=8.0, ymax=7.0, g_uu=4.0, g_dd=3.0, g_ud=2.0, k_l=1.1, omega=0.6, delta=0.3,
               omega_r0=raman, omega_rw=2.0, dt=1e-4)
    psi = gaussian_state(p, sigma=2.0, seed=ny, noise=0.1).astype(np.complex64).astype(complex)
    d = Solver(p)
    assert d.get_schedule()["col_tile"] == tiles[-1]
    real = d.set_psi(psi).step_real(3).get_psi()
    imag = d.step_imag(2).get_psi()
    for tile in tiles:
        print(f"case: {nx}x{ny}, raman {raman}, column tile {tile}", flush=True)
        s = Solver(p)
        s.set_schedule(col_tile=tile)
        assert s.get_schedule()["col_tile"] == tile
        assert np.array_equal(s.set_psi(psi).step_real(3).get_psi(), real)
        g = s.step_imag(2).get_psi()
        assert np.linalg.norm(g - imag) <= 1e-6 * np.linalg.norm(imag)
        if tile == tiles[-1]:
            assert np.array_equal(g, imag)   # a saved default is the default
        s.close()
    with pytest.raises(Exception, match="SGPE_EINVAL"):
        d.set_schedule(col_tile=2 * tiles[-1])
    assert d.get_schedule()["col_tile"] == tiles[-1]


@pytest.mark.parametrize("nx,ny", [(1024, 2048), (512, 4096)])
@pytest.mark.parametrize("raman", [0.0, 1.5])
def test_wide_columns_with_the_full_op_on_both_sides(Solver, nx, ny, raman):
    # three steps (the third pass along columns, with K(dt) before and after R) and a call that continues
    # them; the tolerance of the pairs above for five steps: 1.4e-7 sqrt(22) = 6.6e-7 < 1e-6
    p = Params(nx=nx, ny=ny, xmax=8.0, ymax=7.0, g_uu=4.0, g_dd=3.0, g_ud=2.0, k_l=1.1, omega=0.6, delta=0.3,
               omega_r0=raman, omega_rw=2.0, dt=1e-4)
    psi = gaussian_state(p, sigma=2.0, seed=ny + 1, noise=0.1).astype(np.complex64).astype(complex)
    print(f"case: {nx}x{ny}, raman {raman}, 3 + 2 real steps", flush=True)
    o = OracleGPE(p, workers=8)
    o.set_psi(psi)
    o.step_real(5)
    s, one = Solver(p), Solver(p)
    g = s.set_psi(psi).step_real(3).step_real(2).get_psi()
    err = np.linalg.norm(g - o.psi) / np.linalg.norm(o.psi)
    assert err <= 1e-6, err
    assert np.array_equal(g, one.set_psi(psi).step_real(5).get_psi())
