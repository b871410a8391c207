"""States past positivity: a run goes on past cells of non-positive density or pressure (they are counted as
faults), so what such a cell does to its neighbours and to the time step is part of the results. Against the CPU
oracle, whose fast speed is NaN there and drops out of the signal speeds, with the bounds of the other stage tests."""
import numpy as np
import pytest

from paper_2501_06717_amd import workloads as wk

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-12


@pytest.fixture(scope="module")
def bd():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2501_06717_amd import binding
    binding.lib()
    return binding


def one_stage(bd, oracle_mod, wl, W, dt0, flux, **kw):
    """A single stage of given dt on the GPU and by the oracle: largest error per variable group."""
    g = bd.Grid.from_workload(wl).upload()
    U0 = g.set_state(torch.from_numpy(W).cuda())
    U1 = torch.zeros_like(U0)
    dt = torch.full((g.ns,), dt0, dtype=torch.float64, device="cuda")
    g.advance(U0, U1, dt, 1, flux=flux, recompute_dt=False, **kw)
    torch.cuda.synchronize()
    o = oracle_mod.Grid.from_workload(wl)
    R0 = o.set_state(W)
    R1 = np.zeros_like(R0)
    o.advance(R0, R1, [dt0], 1, flux=flux, recompute_dt=False)
    got = U1.cpu().numpy()
    assert np.isfinite(R1).all() and np.isfinite(got).all()
    return max(float(np.abs(got[v] - R1[v]).max() / np.abs(R1[v]).max()) for v in ([0], [1, 2, 3], [4, 5, 6], [7]))


@pytest.mark.parametrize("flux", ["rusanov", "hlle", "linde"])
@pytest.mark.parametrize("cell", [(3, 3, 3), (0, 0, 0), (7, 7, 7)])
@pytest.mark.parametrize("p", [0.5, -0.5])
def test_cell_of_negative_density(bd, oracle_mod, flux, cell, p):
    """One cell of negative density in a uniform state, inside a block and on both ends of one (its faces in the
    low, high and neighbour passes): the faces' fluxes stay finite, from the other side's signal speeds where
    its own has no real value (p > 0)."""
    wl = wk.uniform_state((2, 2, 2))
    W = wl.W.copy()
    i, j, k = cell
    W[:, 1, k, j, i] = (-0.01, 0.1, -0.2, 0.3, 0.5, -0.4, 0.3, p)
    print("negative density", flux, cell, p, flush=True)
    err = one_stage(bd, oracle_mod, wl, W, 0.05, flux)
    print("error", err, flush=True)
    assert err <= TOL, err


@pytest.mark.parametrize("flux", ["rusanov", "hlle", "linde"])
@pytest.mark.parametrize("e", [-258, 258])
def test_density_and_pressure_near_the_ends_of_the_range(bd, oracle_mod, flux, e):
    """Density and pressure in units of 2^(2 e), the field in units of 2^e: velocities and speeds are those of the
    ordinary state, and products of two pressures leave the range of doubles."""
    wl = wk.odd_box()
    W = wk.random_positive_state(wl, seed=3)
    for v, s in ((0, 2 * e), (4, e), (5, e), (6, e), (7, 2 * e)):
        W[v] = np.ldexp(W[v], s)
    for sim in wl.sims:                        # inflow states in the same units
        w = list(sim.inflow_W)
        sim.inflow_W = tuple(np.ldexp(w[v], 2 * e if v in (0, 7) else (e if v >= 4 else 0)) for v in range(8))
    dt = 0.05 * min(s.dx0 for s in wl.sims)
    print("units", flux, e, flush=True)
    err = one_stage(bd, oracle_mod, wl, W, dt, flux)
    print("error", err, flush=True)
    assert err <= TOL, err


@pytest.mark.parametrize("precision", ["fp64", "fp32_flux"])
@pytest.mark.parametrize("nroot", [(2, 2, 2), (8, 9, 8)])
def test_time_step_past_a_layer_of_negative_density(bd, nroot, precision):
    """A step that leaves two whole cell layers of some blocks at negative density (a thin layer that two streams
    leave, in one large step): the next step's dt comes from the other cells, as in the reduction of dt from the
    state, on a grid that is in flight at once and on a larger one."""
    wl = wk.uniform_state(nroot, W0=(1.0, 0.1, -0.2, 0.0, 0.5, 0.1, 0.1, 0.5))
    W = wl.W.copy()
    d = wl.ijk[:, 2, None] * 8 + np.arange(8) - 3
    W[3] = (np.sign(d) * np.exp(-np.abs(d) / 3.0))[:, :, None, None]
    W[0][d == 0] = 0.3
    g = bd.Grid.from_workload(wl).upload()
    kw = dict(flux="hlle", precision=precision, alpha=(0.0, 0.0), beta=(0.0, 8.0))
    A = g.set_state(torch.from_numpy(W).cuda()); A1 = torch.zeros_like(A)
    B = A.clone(); B1 = torch.zeros_like(B)
    dta = torch.zeros(1, dtype=torch.float64, device="cuda")
    dtb = torch.zeros_like(dta)
    print("layer of negative density", nroot, precision, flush=True)
    g.advance(B, B1, dtb, 2, **kw)
    first = dtb.item()
    below = (B[0] <= 0.0).flatten(2).all(2)        # layers, per block
    assert bool(below.any()) and not bool(below.all())
    dtb = g.reduce_dt(B, 0.8)
    g.advance(A, A1, dta, 4, **kw)
    torch.cuda.synchronize()
    print("dt", first, dta.item(), dtb.item(), flush=True)
    assert 0.0 < dtb.item() < float("inf")
    assert dta.item() == dtb.item()


@pytest.mark.parametrize("axis", [0, 1, 2])
def test_contact_without_pressure(bd, oracle_mod, axis):
    """A density jump where the pressure is exactly zero on both sides: the Linde-type flux has no sound speed to
    tell the entropy wave's part of the jump by, and takes none."""
    wl = wk.uniform_state((2, 2, 2), W0=(1.0, 0.5, -0.25, 0.5, 0.5, 0.25, 0.5, 0.0))
    W = wl.W.copy()
    W[0][wl.ijk[:, axis] == 1] = 0.25
    print("contact without pressure", axis, flush=True)
    err = one_stage(bd, oracle_mod, wl, W, 0.05, "linde")
    print("error", err, flush=True)
    assert err <= TOL, err


@pytest.mark.parametrize("precision", ["fp64", "fp32_flux"])
@pytest.mark.parametrize("flux", ["rusanov", "hlle", "linde"])
def test_flux_that_is_not_finite_stays_with_its_cells(bd, oracle_mod, flux, precision):
    """Negative density on both sides of a block's first x face in one row: that flux has no real value, and only the
    two cells it belongs to are lost, no cell of another row."""
    wl = wk.uniform_state((3, 1, 1))
    W = wl.W.copy()
    for j, k in ((1, 0), (2, 3), (5, 4), (7, 7)):
        for b, i in ((0, 7), (1, 0)):
            W[0, b, k, j, i] = -0.01
    print("flux that is not finite", flux, precision, flush=True)
    g = bd.Grid.from_workload(wl).upload()
    U0 = g.set_state(torch.from_numpy(W).cuda())
    U1 = torch.zeros_like(U0)
    dt = torch.full((1,), 0.05, dtype=torch.float64, device="cuda")
    g.advance(U0, U1, dt, 1, flux=flux, precision=precision, recompute_dt=False)
    torch.cuda.synchronize()
    o = oracle_mod.Grid.from_workload(wl)
    R0 = o.set_state(W)
    R1 = np.zeros_like(R0)
    o.advance(R0, R1, [0.05], 1, flux=flux, recompute_dt=False)
    fin = np.isfinite(R1)
    assert (~fin[0]).sum() == 8                # four faces, two cells each
    got = U1.cpu().numpy()
    assert np.array_equal(np.isfinite(got), fin)
    if precision == "fp64":
        assert np.abs(got[fin] - R1[fin]).max() <= TOL * np.abs(R1[fin]).max()
