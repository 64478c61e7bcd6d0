"""Batched launches: many uneven lattices stepped together match the oracle member by member."""
import numpy as np
import pytest

from paper_2603_24370_amd import inputs as I

pytestmark = pytest.mark.gpu

AH = "abelian_higgs"


@pytest.fixture(scope="module")
def ss():
    import torch
    assert torch.cuda.is_available()
    import paper_2603_24370_amd as m
    m.lib()
    return m


def _members(k0=0, n=6, sides=None):
    insts = []
    for b in range(k0, k0 + n):
        inst = I.gl_batch_instance(b)
        if sides is not None:
            side = sides[(b - k0) % len(sides)]
            L = 0.5 * 0.6 * side * inst.h
            inst = I.Instance(AH, side, side + 3 * (b % 3), inst.h, inst.params, I.uniform_centres(inst.seed,
                              len(inst.centres), L), inst.seed, kappa=inst.kappa)
        insts.append(inst)
    return insts


def _np(t):
    return t.detach().cpu().numpy().astype(np.float64)


# (plan, tile): the fused pass runs on tile 0 in FP32 and tile 1 in FP64
BATCH_PLANS = {"f32": [(0, 0), (1, 0), (1, 1)], "f64": [(0, 0), (1, 1)]}


@pytest.mark.parametrize("dtype,which", [("f64", 0), ("f64", 1), ("f32", 0), ("f32", 1), ("f32", 2)])
def test_batch_flow_matches_oracle_per_member(ss, orc, dtype, which):
    plan, tile = BATCH_PLANS[dtype][which]
    insts = _members(0, 6, sides=[40, 71, 96, 33, 128, 64])
    B = ss.Batch(AH, [(m.Nx, m.Ny, m.h, m.params) for m in insts], dtype=dtype)
    B.set_plan(plan)
    B.set_tile(tile)
    assert B.plan == plan
    fields = []
    for m, mem in zip(insts, B.members):
        f = m.field()
        if dtype == "f32":
            f = f.astype(np.float32).astype(np.float64)
        mem.set_field(f)
        fields.append(f)
    infos = B.flow_step(5)
    rel = 1e-11 if dtype == "f64" else 1e-5
    for k, (m, mem, f) in enumerate(zip(insts, B.members, fields)):
        phi_r, v_r, E_r, na = orc.flow(AH, f, np.zeros_like(f), m.h, m.params, 5)
        phi = _np(mem.get_field())
        assert np.abs(phi - phi_r).max() <= rel * np.abs(phi_r).max(), k
        assert infos[k]["step"] == 5 and infos[k]["n_arrests"] == na
        if dtype == "f64":
            assert infos[k]["energy"] == pytest.approx(E_r, rel=1e-12)
        else:
            # energy of the member's own field (FP64 reduction of the stored values)
            assert infos[k]["energy"] == pytest.approx(orc.energy(AH, phi, m.h, m.params), rel=1e-12)
    # observables of all members in one call: the oracle's on each member's own field,
    # and bit for bit what the single-context call gives
    obs = B.observables()
    assert len(obs) == len(insts)
    for k, (m, mem) in enumerate(zip(insts, B.members)):
        r = orc.observables(AH, _np(mem.get_field()), m.h, m.params)
        for k_gpu, k_ref in [("energy", "E"), ("flux", "flux"), ("n_rho", "N_rho"), ("bogo_r1", "R1"),
                             ("bogo_r2", "R2"), ("n_wind", "N_wind")]:
            assert obs[k][k_gpu] == pytest.approx(r[k_ref], rel=1e-11, abs=1e-11), (k, k_gpu)
        assert obs[k] == mem.observables(), k
    B.close()


@pytest.mark.parametrize("which", [0, 1])
def test_batch_minimise_stops_each_member_where_the_oracle_does(ss, orc, which):
    """FP64: each member stops at the oracle's step count even though members stop
    at different times and the work list is compacted between graph replays."""
    plan, tile = BATCH_PLANS["f64"][which]
    insts = _members(10, 5, sides=[32, 48, 40, 56, 36])
    B = ss.Batch(AH, [(m.Nx, m.Ny, m.h, m.params) for m in insts], dtype="f64")
    B.set_plan(plan)
    B.set_tile(tile)
    fields = [m.field() for m in insts]
    for f, mem in zip(fields, B.members):
        mem.set_field(f)
    rc, infos = B.minimise(grad_tol=2e-3, max_steps=3000, graph_steps=8)
    steps = set()
    for k, (m, f) in enumerate(zip(insts, fields)):
        phi_r, v_r, info_r = orc.minimise(AH, f, m.h, m.params, grad_tol=2e-3, max_steps=3000)
        assert infos[k]["step"] == info_r["steps"], k
        assert infos[k]["n_arrests"] == info_r["arrests"], k
        assert infos[k]["reason"] == {1: "grad", 2: "stall", 0: "max_steps"}[info_r["reason"]]
        phi = _np(B.members[k].get_field())
        assert np.abs(phi - phi_r).max() < 1e-9, k
        steps.add(info_r["steps"])
    assert len(steps) > 1  # members really stop at different times
    B.close()


def test_batch_tiles_and_autotune(ss, orc):
    insts = _members(20, 4, sides=[64, 100, 37, 80])
    B = ss.Batch(AH, [(m.Nx, m.Ny, m.h, m.params) for m in insts], dtype="f32")
    best, plan, ms = B.autotune(2)
    timed = [m for row in ms for m in row if m >= 0]
    assert 0 <= best < ss.ss_tile_count() and ms[plan][best] == min(timed)
    assert len(timed) == ss.ss_tile_count() + 2  # every tile for the stages plan, tiles 0 and 1 fused
    B.set_plan(0)
    for tile in range(ss.ss_tile_count()):
        B.set_tile(tile)
        fields = []
        for m, mem in zip(insts, B.members):
            f = m.field().astype(np.float32).astype(np.float64)
            mem.set_field(f)
            fields.append(f)
        B.flow_step(3)
        for m, mem, f in zip(insts, B.members, fields):
            phi_r, _, _, _ = orc.flow(AH, f, np.zeros_like(f), m.h, m.params, 3)
            assert np.abs(_np(mem.get_field()) - phi_r).max() <= 1e-5 * np.abs(phi_r).max(), tile
    B.close()


P_CM = [1.0, 1.0, 0.1, 0.6]


@pytest.mark.parametrize("dtype,plan,tile", [("f64", 0, 0), ("f64", 1, 1), ("f32", 0, 0), ("f32", 1, 0)])
def test_chiral_magnet_batch_matches_oracle_per_member(ss, orc, dtype, plan, tile):
    """Chiral-magnet members (3 components, projected flow) of uneven sizes stepped
    together: each member's field against the oracle, and the batch observables
    (energy, both charges) against the oracle's on the member's own field."""
    CM = "chiral_magnet"
    h = 0.2
    sides = [(40, 33), (71, 64), (96, 90), (33, 48)]
    fields = []
    for k, (Nx, Ny) in enumerate(sides):
        f = I.cm_skyrmion_ansatz(Nx, Ny, h, R=min(Nx, Ny) * h / 8)
        f = I.renormalise_interior(f + I.noise(30 + k, 3, Nx, Ny, 1e-3))
        if dtype == "f32":
            f = f.astype(np.float32).astype(np.float64)
        fields.append(f)
    B = ss.Batch(CM, [(Nx, Ny, h, P_CM) for Nx, Ny in sides], dtype=dtype)
    B.set_plan(plan)
    B.set_tile(tile)
    for f, mem in zip(fields, B.members):
        mem.set_field(f)
    print(f"[case] CM batch {dtype} plan {plan} tile {tile}", flush=True)
    infos = B.flow_step(5)
    rel = 1e-11 if dtype == "f64" else 1e-5
    obs = B.observables()
    for k, (f, mem) in enumerate(zip(fields, B.members)):
        phi_r, v_r, E_r, na = orc.flow(CM, f, np.zeros_like(f), h, P_CM, 5)
        phi = _np(mem.get_field())
        assert np.abs(phi - phi_r).max() <= rel * np.abs(phi_r).max(), k
        assert infos[k]["step"] == 5 and infos[k]["n_arrests"] == na
        nrm = np.sqrt((phi[:, 2:-2, 2:-2] ** 2).sum(0))
        assert np.abs(nrm - 1).max() < (1e-14 if dtype == "f64" else 1e-6)
        r = orc.observables(CM, phi, h, P_CM)
        assert obs[k]["energy"] == pytest.approx(r["E"], rel=1e-11)
        assert obs[k]["q_fd"] == pytest.approx(r["Q_fd"], rel=1e-11, abs=1e-12)
        assert obs[k]["q_bl"] == pytest.approx(r["Q_bl"], abs=1e-9)
    B.close()


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("scheme", ["vv", "gf"])
@pytest.mark.parametrize("tile", [0, 1])
def test_one_pass_batch_flow_matches_oracle_per_member(ss, orc, dtype, scheme, tile):
    """Velocity Verlet and gradient flow in batched launches (one pass per step for
    every member, after one prime pass): each member's trajectory is the oracle's."""
    insts = _members(20, 5, sides=[40, 71, 96, 33, 64])
    B = ss.Batch(AH, [(m.Nx, m.Ny, m.h, m.params) for m in insts], dtype=dtype)
    B.set_integrator(scheme)
    B.set_tile(tile)
    assert B.integrator == ss.INTEGRATORS[scheme]
    fields = []
    for m, mem in zip(insts, B.members):
        f = m.field()
        if dtype == "f32":
            f = f.astype(np.float32).astype(np.float64)
        mem.set_field(f)
        fields.append(f)
    n = 6
    infos = B.flow_step(n)
    rel = 1e-11 if dtype == "f64" else 1e-5
    for k, (m, mem, f) in enumerate(zip(insts, B.members, fields)):
        phi_r, v_r, E_r, na = orc.flow(AH, f, np.zeros_like(f), m.h, m.params, n, scheme=scheme)
        phi, vel = (_np(x) for x in mem.get_field(velocity=True))
        assert np.abs(phi - phi_r).max() <= rel * np.abs(phi_r).max(), k
        assert np.abs(vel - v_r).max() <= rel * max(np.abs(phi_r).max(), 1.0), k
        assert infos[k]["step"] == n and infos[k]["n_arrests"] == na, k
        if dtype == "f64":
            assert infos[k]["energy"] == pytest.approx(E_r, rel=1e-12)
    B.close()


@pytest.mark.parametrize("scheme,tol", [("vv", 2e-3), ("gf", 5e-2)])
def test_one_pass_batch_minimise_stops_each_member_where_the_oracle_does(ss, orc, scheme, tol):
    """FP64 velocity Verlet (half-step form) and gradient flow (the field only):
    every member stops at the oracle's step with its arrest count, across graph
    replays and work-list compaction."""
    insts = _members(30, 5, sides=[32, 48, 40, 56, 36])
    B = ss.Batch(AH, [(m.Nx, m.Ny, m.h, m.params) for m in insts], dtype="f64")
    B.set_integrator(scheme)
    fields = [m.field() for m in insts]
    for f, mem in zip(fields, B.members):
        mem.set_field(f)
    rc, infos = B.minimise(grad_tol=tol, max_steps=3000, graph_steps=8)
    steps = set()
    for k, (m, f) in enumerate(zip(insts, fields)):
        phi_r, v_r, info_r = orc.minimise(AH, f, m.h, m.params, grad_tol=tol, max_steps=3000, scheme=scheme)
        assert infos[k]["step"] == info_r["steps"], k
        assert infos[k]["n_arrests"] == info_r["arrests"], k
        assert infos[k]["reason"] == {1: "grad", 2: "stall", 0: "max_steps"}[info_r["reason"]]
        phi = _np(B.members[k].get_field())
        assert np.abs(phi - phi_r).max() < 1e-9, k
        steps.add(info_r["steps"])
    assert len(steps) > 1
    B.close()


@pytest.mark.parametrize("integ", ["vv", "gf", "rk4"])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("theory", ["abelian_higgs", "chiral_magnet"])
def test_default_tile_follows_the_integrator(ss, theory, dtype, integ):
    """Tile 0 of a batch stands for 64 x 16 or 64 x 8 sites by type and integrator:
    ragged members (a partial tile, a whole one, several), the integrator chosen
    after the batch is built and changed once, against single contexts (FP64
    1e-11, FP32 1e-5 of max|phi|: rounding order)."""
    params = [1.0] if theory == "abelian_higgs" else [1.0, 1.0, 0.1, 0.6]
    sizes, h, n = [(9, 65), (64, 64), (131, 37)], 0.17, 4
    print(f"[case] batch default tile {theory} {dtype} {integ}", flush=True)
    rel = 1e-11 if dtype == "f64" else 1e-5

    def start(s):
        if theory == "abelian_higgs":
            s.init_vortices([(0.0, 0.0)], seed=3, noise_amp=1e-3)
        else:
            s.init_skyrmion(R=0.4, seed=3, noise_amp=1e-3)

    B = ss.Batch(theory, [(nx, ny, h, params) for nx, ny in sizes], dtype=dtype)
    B.set_integrator("rk4" if integ != "rk4" else "vv")
    B.set_integrator(integ)
    for m in B.members:
        start(m)
    B.flow_step(n)
    for (nx, ny), m in zip(sizes, B.members):
        s = ss.Solver(theory, nx, ny, h, params, dtype=dtype)
        s.set_integrator(integ)
        start(s)
        s.flow_step(n)
        a, b = m.get_field().double(), s.get_field().double()
        assert (a - b).abs().max() <= rel * b.abs().max(), (nx, ny)
        s.close()
    B.close()


@pytest.mark.parametrize("n", [1, 2])
@pytest.mark.parametrize("integ", ["rk4", "vv", "gf"])
def test_step_information_is_each_members_own(ss, integ, n):
    """A lone member's is read without the launch that gathers several."""
    insts = _members(0, n, sides=[40, 71])
    B = ss.Batch(AH, [(m.Nx, m.Ny, m.h, m.params) for m in insts], dtype="f64")
    B.set_integrator(integ)
    for m, mem in zip(insts, B.members):
        mem.set_field(m.field())
    infos = B.flow_step(3)
    assert [i["step"] for i in infos] == [3] * n and infos == [mem.info() for mem in B.members]
    rc, infos = B.minimise(grad_tol=0.0, max_steps=9)
    for i, mem in zip(infos, B.members):
        assert i["reason"] == "max_steps" and {k: i[k] for k in mem.info()} == mem.info()
    B.close()
