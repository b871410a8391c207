"""GPU parity: the HIP path (through the C ABI) against the CPU oracle on the same seeded inputs.

Bars: neighbour tables and ghost cells bit-exact (copy, restriction and prolongation are evaluated
without contraction on both sides); dt within 1e-14 relative; states after stages within 1e-12
relative per variable group (rho, momentum, B, energy: max abs difference over the group divided by
the group's max abs value); the FP32-flux form reported against the FP64 oracle.
"""
import math
import sys

import numpy as np
import pytest

from paper_2501_06717_amd import workloads as wk

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

GROUPS = {"rho": [0], "mom": [1, 2, 3], "B": [4, 5, 6], "e": [7]}
TOL = 1e-12


def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def bd():
    _need_gpu()
    from paper_2501_06717_amd import binding
    binding.lib()
    return binding


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def group_err(got, ref):
    out = {}
    for g, vs in GROUPS.items():
        scale = np.abs(ref[vs]).max()
        out[g] = float(np.abs(got[vs] - ref[vs]).max() / (scale if scale > 0 else 1.0))
    return out


def gpu_run(bd, wl, W, n_stages, dt0=None, **kw):
    g = bd.Grid.from_workload(wl).upload()
    U0 = g.set_state(dev(W))
    U1 = torch.zeros_like(U0)
    dt = dev(np.zeros(len(wl.sims)) if dt0 is None else np.asarray(dt0, np.float64))
    faults = torch.zeros(1, dtype=torch.int32, device="cuda")
    g.advance(U0, U1, dt, n_stages, faults=faults, **kw)
    torch.cuda.synchronize()
    return U0.cpu().numpy(), U1.cpu().numpy(), dt.cpu().numpy(), int(faults.item())


def oracle_run(oracle_mod, wl, W, n_stages, dt0=None, **kw):
    o = oracle_mod.Grid.from_workload(wl)
    U0 = o.set_state(W)
    U1 = np.zeros_like(U0)
    kw = {k: v for k, v in kw.items() if k in ("flux", "powell", "cfl", "recompute_dt", "alpha", "beta")}
    dt, faults = o.advance(U0, U1, np.zeros(len(wl.sims)) if dt0 is None else dt0, n_stages, **kw)
    return U0, U1, dt, faults


# ------------------------------------------------------------------------------------------------
# set_state, ghost fill, dt

@pytest.mark.parametrize("make", [lambda: wk.cp_alfven(16), lambda: wk.magnetosphere_cut(32), lambda: wk.two_level_box()])
def test_set_state(bd, oracle_mod, make):
    wl = make()
    say("set_state", wl.name)
    g = bd.Grid.from_workload(wl).upload()
    U = g.set_state(dev(wl.W)).cpu().numpy()
    ref = oracle_mod.Grid.from_workload(wl).set_state(wl.W)
    assert max(group_err(U, ref).values()) <= 1e-15


GHOST_CASES = {
    "periodic_1": lambda: wk.uniform_state((1, 1, 1)),
    "odd_box": lambda: wk.odd_box(),
    "two_level": lambda: wk.two_level_box(),
    "two_level_bc": lambda: wk.two_level_box(bc=(1, 2, 0, 0, 2, 1)),
    "two_level_48": lambda: wk.two_level_magnetosphere(48),
    "fast_wave_octant": lambda: wk.fast_wave((4, 2, 2), refine_octant=True),
}


@pytest.mark.parametrize("case", list(GHOST_CASES))
@pytest.mark.parametrize("field", ["unique_id", "random"])
def test_fill_ghosts_bit_exact(bd, oracle_mod, case, field):
    wl = GHOST_CASES[case]()
    say("fill_ghosts", case, field, wl.n_blocks)
    if field == "unique_id":
        U = wk.unique_id_field(wl)
    else:
        U = oracle_mod.Grid.from_workload(wl).set_state(wk.random_positive_state(wl, seed=9))
    g = bd.Grid.from_workload(wl).upload()
    view = g.fill_ghosts(dev(U)).cpu().numpy()
    ref = oracle_mod.Grid.from_workload(wl).fill_ghosts(U)
    bad = np.argwhere(view != ref)
    assert bad.shape[0] == 0, (bad[:5], view[tuple(bad[0])], ref[tuple(bad[0])])


@pytest.mark.parametrize("make", [lambda: wk.cp_alfven(32), lambda: wk.magnetosphere_cut(64), lambda: wk.two_level_box()])
def test_reduce_dt(bd, oracle_mod, make):
    wl = make()
    say("reduce_dt", wl.name)
    o = oracle_mod.Grid.from_workload(wl)
    U = o.set_state(wl.W)
    ref = o.dt(U, 0.8)
    g = bd.Grid.from_workload(wl).upload()
    dt = g.reduce_dt(dev(U), 0.8).cpu().numpy()
    assert np.all(np.abs(dt - ref) <= 1e-14 * ref), (dt, ref)


# ------------------------------------------------------------------------------------------------
# stages

STAGE_CASES = {
    "cp_alfven_32": (lambda: wk.cp_alfven(32), dict(flux="rusanov", powell=False)),
    "cp_alfven_32_hlle": (lambda: wk.cp_alfven(32), dict(flux="hlle", powell=True)),
    "odd_box": (lambda: wk.odd_box(), dict(flux="hlle", powell=True)),
    # one periodic block: every neighbour, across faces, edges and corners, is the block itself
    "periodic_1": (lambda: wk.with_state(wk.uniform_state((1, 1, 1)),
                                         wk.random_positive_state(wk.uniform_state((1, 1, 1)), seed=7)),
                   dict(flux="hlle", powell=True)),
    "magnetosphere_32": (lambda: wk.magnetosphere_cut(32), dict(flux="hlle", powell=True)),
    "two_level_box": (lambda: wk.two_level_box(), dict(flux="rusanov", powell=False)),
    "two_level_box_hlle": (lambda: wk.two_level_box(bc=(1, 2, 0, 0, 2, 1)), dict(flux="hlle", powell=True)),
    "two_level_48": (lambda: wk.two_level_magnetosphere(48), dict(flux="hlle", powell=True)),
    # a body cell on the coarse side of a level face: flux correction must leave it alone
    "two_level_box_body": (lambda: wk.two_level_box(body=True), dict(flux="hlle", powell=True)),
    # the Linde-type flux (contact anti-diffusion) on the paper's fast wave with a refined octant and on
    # the magnetosphere cut (body, inflow, outflow)
    "fast_wave_octant_linde": (lambda: wk.fast_wave((2, 2, 2), refine_octant=True), dict(flux="linde", powell=True)),
    "magnetosphere_32_linde": (lambda: wk.magnetosphere_cut(32), dict(flux="linde", powell=True)),
    "odd_box_linde": (lambda: wk.odd_box(), dict(flux="linde", powell=False)),
}


@pytest.mark.parametrize("scheme", ["face", "plane", "block"])
@pytest.mark.parametrize("case", list(STAGE_CASES))
@pytest.mark.parametrize("n_stages", [1, 2, 6])
def test_advance_parity(bd, oracle_mod, case, n_stages, scheme):
    make, kw = STAGE_CASES[case]
    wl = make()
    say("advance", case, n_stages, scheme, wl.n_blocks)
    U0, U1, dt, f = gpu_run(bd, wl, wl.W, n_stages, scheme=scheme, **kw)
    R0, R1, rdt, rf = oracle_run(oracle_mod, wl, wl.W, n_stages, **kw)
    assert f == 0 and rf == 0
    assert np.all(np.abs(dt - rdt) <= 1e-14 * rdt), (dt, rdt)
    got, ref = (U1, R1) if n_stages % 2 else (U0, R0)
    err = group_err(got, ref)
    say("  err", err)
    assert max(err.values()) <= TOL, err


@pytest.mark.parametrize("scheme", ["face", "plane"])
def test_slab_choice_is_bitwise_neutral(bd, scheme):
    wl = wk.magnetosphere_cut(32)
    a = gpu_run(bd, wl, wl.W, 4, flux="hlle", powell=True, slab=8, scheme=scheme)
    b = gpu_run(bd, wl, wl.W, 4, flux="hlle", powell=True, slab=4, scheme=scheme)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[2], b[2])


@pytest.mark.parametrize("slab,persist,scheme", [(4, 8, "face"), (4, 256, "face"), (8, 24, "face"), (4, 1024, "face"),
                                                 (4, 8, "plane"), (4, 256, "plane"), (8, 24, "plane")])
def test_persistent_form_is_bitwise_identical(bd, slab, persist, scheme):
    wl = wk.two_level_magnetosphere(48)
    kw = dict(flux="hlle", powell=True, scheme=scheme)
    a = gpu_run(bd, wl, wl.W, 4, slab=slab, persist_wgs=persist, **kw)
    b = gpu_run(bd, wl, wl.W, 4, slab=slab, **kw)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1]) and np.array_equal(a[2], b[2])


@pytest.mark.parametrize("precision", ["fp64", "fp32_flux"])
@pytest.mark.parametrize("slab", [4, 8])
def test_plane_scheme_matches_face_scheme(bd, precision, slab):
    """The two work splits evaluate the same face fluxes and sum them in the same order; they may differ
    only where the compiler contracts a multiply-add differently."""
    wl = wk.two_level_magnetosphere(48)
    kw = dict(flux="hlle", powell=True, precision=precision, slab=slab)
    a = gpu_run(bd, wl, wl.W, 4, scheme="plane", **kw)
    b = gpu_run(bd, wl, wl.W, 4, scheme="face", **kw)
    err = group_err(a[0], b[0])
    say("plane vs face", precision, slab, err)
    assert a[3] == 0 and b[3] == 0
    assert max(err.values()) <= (1e-13 if precision == "fp64" else 1e-5), err
    assert np.all(np.abs(a[2] - b[2]) <= 1e-14 * b[2])


@pytest.mark.parametrize("precision", ["fp64", "fp32_flux"])
@pytest.mark.parametrize("case", ["two_level_48", "magnetosphere_32", "periodic_1"])
def test_block_scheme_matches_plane_scheme(bd, precision, case):
    """The block form (blocks clear of a body; the others on the plane form) evaluates the same face
    fluxes as the plane form; the cell sums take each flux as its own multiply-add, so the two differ in
    the last places only."""
    make, kw = STAGE_CASES[case]
    wl = make()
    kw = dict(kw, precision=precision)
    a = gpu_run(bd, wl, wl.W, 4, scheme="block", **kw)
    b = gpu_run(bd, wl, wl.W, 4, scheme="plane", slab=4, **kw)
    err = group_err(a[0], b[0])
    say("block vs plane", case, precision, err)
    assert a[3] == 0 and b[3] == 0
    assert max(err.values()) <= (1e-13 if precision == "fp64" else 1e-5), err
    assert np.all(np.abs(a[2] - b[2]) <= 1e-14 * b[2])


def test_block_scheme_is_deterministic_and_graph_replays_match(bd):
    wl = wk.two_level_magnetosphere(48)
    kw = dict(flux="hlle", powell=True, scheme="block")
    a = gpu_run(bd, wl, wl.W, 6, **kw)
    b = gpu_run(bd, wl, wl.W, 6, **kw)
    c = gpu_run(bd, wl, wl.W, 6, use_graph=True, **kw)
    for x in (b, c):
        assert np.array_equal(a[0], x[0]) and np.array_equal(a[1], x[1]) and np.array_equal(a[2], x[2])


def test_cp_alfven_ten_steps(bd, oracle_mod):
    wl = wk.cp_alfven(32)
    say("cp_alfven 10 steps")
    U0, _, dt, _ = gpu_run(bd, wl, wl.W, 20, flux="rusanov")
    R0, _, rdt, _ = oracle_run(oracle_mod, wl, wl.W, 20, flux="rusanov")
    err = group_err(U0, R0)
    say("  err", err)
    assert max(err.values()) <= TOL


def test_fixed_dt_and_midpoint_table(bd, oracle_mod):
    wl = wk.odd_box()
    kw = dict(flux="rusanov", powell=True, recompute_dt=False, alpha=(0.0, 0.0), beta=(0.5, 1.0))
    U0, _, dt, _ = gpu_run(bd, wl, wl.W, 4, dt0=[0.05], **kw)
    R0, _, rdt, _ = oracle_run(oracle_mod, wl, wl.W, 4, dt0=[0.05], **kw)
    assert dt[0] == 0.05 and rdt[0] == 0.05
    assert max(group_err(U0, R0).values()) <= TOL


def test_deterministic_and_faults(bd):
    wl = wk.magnetosphere_cut(32)
    a = gpu_run(bd, wl, wl.W, 6, flux="hlle", powell=True)
    b = gpu_run(bd, wl, wl.W, 6, flux="hlle", powell=True)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
    # faults forced on the host: a pressure far below what one step of inflow can refill (a cell at
    # p = -1 next to p = 7500 gains about +50 in one step of 1e-5 and heals), and a negative density
    W = wl.W.copy()
    W[7, 5, 3, 3, 3] = -1e7
    W[0, 9, 4, 4, 4] = -1.0
    _, _, _, f = gpu_run(bd, wl, W, 2, flux="hlle", powell=True, recompute_dt=False, dt0=[1e-5])
    assert f >= 2


def test_fp32_flux_form_error(bd, oracle_mod):
    """FP32 reconstruction and flux with an FP64 update: report L1 and Linf against the FP64 oracle."""
    wl = wk.magnetosphere_cut(32)
    kw = dict(flux="hlle", powell=True)
    U0, _, _, f = gpu_run(bd, wl, wl.W, 10, precision="fp32_flux", **kw)
    R0, _, _, _ = oracle_run(oracle_mod, wl, wl.W, 10, **kw)
    assert f == 0 and np.all(np.isfinite(U0))
    err = group_err(U0, R0)
    l1 = {g: float(np.abs(U0[v] - R0[v]).mean() / np.abs(R0[v]).mean()) for g, v in GROUPS.items()}
    say("  fp32 Linf", err, "L1", l1)
    assert max(err.values()) < 1e-4


def test_two_level_conservation_gpu(bd, oracle_mod):
    """Periodic two-level grid, Powell off: the GPU keeps sum U dV to round-off (flux correction)."""
    wl = wk.two_level_box()
    W = wk.random_positive_state(wl, seed=11)
    U0, _, _, _ = gpu_run(bd, wl, W, 6, flux="hlle", powell=False)
    Ui = oracle_mod.Grid.from_workload(wl).set_state(W)
    vol = (1.0 / 2.0 ** wl.level) ** 3
    for v in range(8):
        t0 = math.fsum((Ui[v] * vol[:, None, None, None]).ravel())
        t1 = math.fsum((U0[v] * vol[:, None, None, None]).ravel())
        s = math.fsum((np.abs(Ui[v]) * vol[:, None, None, None]).ravel())
        assert abs(t1 - t0) <= 1e-14 * s


# ------------------------------------------------------------------------------------------------
# batched simulations, graph replay, autotuner

def small_batch():
    return wk.batched_waves(n_sims=5, seed=7, n_lo=8, n_hi=60)


def test_batched_parity_fp64(bd, oracle_mod):
    wl = small_batch()
    say("batched", wl.n_blocks, len(wl.sims))
    U0, _, dt, f = gpu_run(bd, wl, wl.W, 6, flux="rusanov")
    R0, _, rdt, rf = oracle_run(oracle_mod, wl, wl.W, 6, flux="rusanov")
    assert f == 0 and rf == 0
    assert np.all(np.abs(dt - rdt) <= 1e-14 * rdt)
    assert max(group_err(U0, R0).values()) <= TOL


def test_batched_member_equals_alone(bd):
    """Every simulation of a batch advances exactly as it does alone (its own dt, no coupling)."""
    import dataclasses
    wl = small_batch()
    U0, _, dt, _ = gpu_run(bd, wl, wl.W, 4, flux="rusanov", precision="fp32_flux")
    for s in (0, 3):
        sel = wl.sim == s
        alone = dataclasses.replace(wl, level=wl.level[sel], ijk=wl.ijk[sel], sim=np.zeros(sel.sum(), np.int32),
                                    sims=[wl.sims[s]], W=np.ascontiguousarray(wl.W[:, sel]))
        A0, _, adt, _ = gpu_run(bd, alone, alone.W, 4, flux="rusanov", precision="fp32_flux")
        assert adt[0] == dt[s]
        assert np.array_equal(A0, U0[:, sel])


@pytest.mark.parametrize("scheme", ["face", "plane"])
@pytest.mark.parametrize("precision", ["fp64", "fp32_flux"])
def test_graph_replay_matches_eager(bd, precision, scheme):
    """Graph replays interleaved with eager work and synchronisations, each checked bitwise."""
    wl = small_batch()
    g = bd.Grid.from_workload(wl).upload()
    kw = dict(flux="rusanov", precision=precision, persist_wgs=64, scheme=scheme)
    Ue = g.set_state(dev(wl.W)); U1e = torch.zeros_like(Ue); dte = torch.zeros(len(wl.sims), dtype=torch.float64, device="cuda")
    Ug = g.set_state(dev(wl.W)); U1g = torch.zeros_like(Ug); dtg = torch.zeros_like(dte)
    fe = torch.zeros(1, dtype=torch.int32, device="cuda"); fg = torch.zeros_like(fe)
    for rep in range(3):
        g.advance(Ue, U1e, dte, 8, faults=fe, **kw)
        torch.cuda.synchronize()
        g.advance(Ug, U1g, dtg, 8, faults=fg, use_graph=True, **kw)
        torch.cuda.synchronize()
        _ = (Ue * 2.0).sum().item()   # unrelated eager work between replays
        assert torch.equal(Ue, Ug) and torch.equal(U1e, U1g) and torch.equal(dte, dtg), rep
    assert fe.item() == 0 and fg.item() == 0


def test_autotune_picks_a_valid_shape(bd):
    wl = small_batch()
    g = bd.Grid.from_workload(wl).upload()
    U0 = g.set_state(dev(wl.W)); U1 = torch.zeros_like(U0)
    dt = torch.zeros(len(wl.sims), dtype=torch.float64, device="cuda")
    best, ms = g.autotune(U0, U1, dt, n_steps=2, flux="rusanov", precision="fp32_flux")
    say("autotune", ms, best.scheme, best.slab, best.persist_wgs)
    assert len(ms) == 13 and all(v > 0 for v in ms.values())
    assert best.scheme in (1, 2, 3) and best.slab in (4, 8) and best.persist_wgs >= 0
    assert all(v > 0 for v in ms.values())
    assert min(ms.values()) == pytest.approx(ms[min(ms, key=ms.get)])


def test_autotune_cache(bd, tmp_path, monkeypatch):
    """With BMHD_AUTOTUNE_CACHE set the autotuner stores its choice and a second call with the same
    device, grid and options returns it without timing; other options miss."""
    path = tmp_path / "tune.txt"
    monkeypatch.setenv("BMHD_AUTOTUNE_CACHE", str(path))
    wl = wk.two_level_box()
    g = bd.Grid.from_workload(wl).upload()
    U0 = g.set_state(dev(wl.W))
    U1 = torch.zeros_like(U0)
    dt = torch.zeros(1, dtype=torch.float64, device="cuda")
    kw = dict(flux="hlle", powell=True)
    b1, ms1 = g.autotune(U0.clone(), U1, dt, n_steps=1, **kw)
    assert all(v > 0 for v in ms1.values())
    assert len(path.read_text().splitlines()) == 1
    b2, ms2 = g.autotune(U0.clone(), U1, dt, n_steps=1, **kw)
    assert all(v == -1.0 for v in ms2.values())
    assert (b2.scheme, b2.slab, b2.persist_wgs) == (b1.scheme, b1.slab, b1.persist_wgs)
    _, ms3 = g.autotune(U0.clone(), U1, dt, n_steps=1, precision="fp32_flux", **kw)
    assert all(v > 0 for v in ms3.values())
    assert len(path.read_text().splitlines()) == 2


@pytest.mark.parametrize("n_steps", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("use_graph", [False, True])
@pytest.mark.parametrize("case", ["batch", "two_level_body"])
def test_time_step_of_every_step_in_a_call(bd, case, use_graph, n_steps):
    """dt of each step from the bound that the step before collected, in either of its two places and for
    every simulation, against dt reduced anew from the state (bmhd_reduce_dt) and one call per step: bit
    for bit, for pairs of steps replayed from a graph and the steps left over, and again in a second call."""
    wl = small_batch() if case == "batch" else wk.two_level_magnetosphere(48)
    kw = dict(flux="hlle", powell=case != "batch")
    g = bd.Grid.from_workload(wl).upload()
    A = g.set_state(dev(wl.W)); A1 = torch.zeros_like(A)
    B = g.set_state(dev(wl.W)); B1 = torch.zeros_like(B)
    dta = torch.zeros(g.ns, dtype=torch.float64, device="cuda")
    for rep in range(2):
        say("dt of every step", case, use_graph, n_steps, rep)
        g.advance(A, A1, dta, 2 * n_steps, cfl=0.8, use_graph=use_graph, **kw)
        for _ in range(n_steps):
            dtb = g.reduce_dt(B, 0.8)
            g.advance(B, B1, dtb, 2, recompute_dt=False, **kw)
        torch.cuda.synchronize()
        assert torch.equal(dta, dtb) and torch.equal(A, B) and torch.equal(A1, B1), rep


def test_graph_after_another_upload(bd):
    """A grid uploaded again has its tables and the bounds between steps in another workspace: steps replayed from a
    graph then equal the directly launched ones bit for bit, with the old workspace's memory in other use."""
    wl = small_batch()
    kw = dict(flux="hlle", powell=True)
    g = bd.Grid.from_workload(wl).upload()
    A = g.set_state(dev(wl.W)); A1 = torch.zeros_like(A)
    B = A.clone(); B1 = torch.zeros_like(B)
    dta = torch.zeros(g.ns, dtype=torch.float64, device="cuda")
    dtb = torch.zeros_like(dta)
    kept = []
    for rep in range(3):
        say("graph after upload", rep)
        g.advance(A, A1, dta, 12, use_graph=True, **kw)
        g.advance(B, B1, dtb, 12, **kw)
        torch.cuda.synchronize()
        assert torch.equal(A, B) and torch.equal(A1, B1) and torch.equal(dta, dtb), rep
        kept.append(g.work)                    # the next upload takes other memory
        g.upload()
        assert g.work.data_ptr() != kept[-1].data_ptr()
        kept[-1].zero_()                       # as another owner of it might


@pytest.mark.parametrize("shape,hit", [((3, 8, 0), True), ((2, 4, 2), True), ((1, 8, 0), True), ((3, 4, 0), False),
                                       ((3, 8, 2), False), ((4, 8, 0), False)])
def test_autotune_cache_takes_every_shape_it_writes(bd, tmp_path, monkeypatch, shape, hit):
    """A cached line of each scheme is returned without timing, whichever shape is the fastest here; one that no tuning
    writes is not."""
    path = tmp_path / "tune.txt"
    monkeypatch.setenv("BMHD_AUTOTUNE_CACHE", str(path))
    wl = wk.two_level_box()
    g = bd.Grid.from_workload(wl).upload()
    U0 = g.set_state(dev(wl.W))
    U1 = torch.zeros_like(U0)
    dt = torch.zeros(1, dtype=torch.float64, device="cuda")
    kw = dict(flux="hlle", powell=True)
    g.autotune(U0.clone(), U1, dt, n_steps=1, **kw)
    key = path.read_text().split()[0]
    path.write_text(f"{key} {shape[0]} {shape[1]} {shape[2]}\n")
    best, ms = g.autotune(U0.clone(), U1, dt, n_steps=1, **kw)
    say("autotune cache", shape, best.scheme, best.slab, best.persist_wgs)
    assert all((v == -1.0) == hit for v in ms.values())
    if hit:
        assert (best.scheme, best.slab) == shape[:2] and (best.persist_wgs > 0) == (shape[2] > 0)
        g.advance(U0, U1, dt, 2, slab=best.slab, scheme=best.scheme, persist_wgs=best.persist_wgs, **kw)
        torch.cuda.synchronize()
