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
