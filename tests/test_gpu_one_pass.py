"""The one-pass integrators (velocity Verlet arrested Newton flow, gradient flow)
through the C ABI against the FP64 oracle's flows of the same scheme.

Tolerances as for the RK4 plans: FP64 fields to 1e-11 relative (rounding order
only), FP32 fields to 1e-5 relative (the FP32 tolerance of the flow), energies
of the device's own field to 1e-12 against the oracle, arrests and steps exact.
"""
import math

import numpy as np
import pytest

from paper_2603_24370_amd import inputs as I

pytestmark = pytest.mark.gpu

AH, CM = "abelian_higgs", "chiral_magnet"
P_CM = [1.0, 1.0, 0.1, 0.6]


@pytest.fixture(scope="module")
def ss():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_2603_24370_amd as m
    m.lib()
    return m


def _params(theory):
    return [1.0] if theory == AH else P_CM


def _field(theory, Nx, Ny, h, seed):
    if theory == AH:
        cen = I.uniform_centres(seed, 3, 0.3 * min(Nx, Ny) * h)
        return I.ah_vortex_ansatz(Nx, Ny, h, cen) + I.noise(seed, 4, Nx, Ny, 1e-3)
    f = I.cm_skyrmion_ansatz(Nx, Ny, h, R=min(Nx, Ny) * h / 8)
    return I.renormalise_interior(f + I.noise(seed, 3, Nx, Ny, 1e-3))


def _np(t):
    return t.detach().cpu().numpy().astype(np.float64)


# integrators under test: velocity Verlet in the form its context picks (the
# stored force on these small lattices), forced into the kick-drift-kick
# (half-step) form, and gradient flow; the oracle's scheme of each
INTEGS = ["vv", "vv_half", "gf"]


def _set_integ(s, integ):
    s.set_integrator("gf" if integ == "gf" else "vv")
    if integ == "vv_half":
        s.set_vv_form("half_step")
    elif integ == "vv_stored":
        s.set_vv_form("stored_force")


def _scheme(integ):
    return "gf" if integ == "gf" else "vv"


SHAPES = [(150, 37), (64, 16), (129, 70)]


@pytest.mark.parametrize("integ", INTEGS)
@pytest.mark.parametrize("theory", [AH, CM])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("shape", SHAPES)
def test_one_pass_flow_tracks_the_oracle(ss, orc, integ, theory, dtype, shape):
    Nx, Ny = shape
    h = 0.17
    print(f"[case] one-pass {integ} {theory} {dtype} {shape}", flush=True)
    f = _field(theory, Nx, Ny, h, seed=Nx + 5 * Ny)
    if dtype == "f32":
        f = f.astype(np.float32).astype(np.float64)
    s = ss.Solver(theory, Nx, Ny, h, _params(theory), dtype=dtype)
    _set_integ(s, integ)
    assert s.integrator == ss.INTEGRATORS[_scheme(integ)]
    if integ != "gf":
        assert s.vv_form == (ss.SS_VV_HALF_STEP if integ == "vv_half" else ss.SS_VV_STORED_FORCE)
    s.set_field(f)
    n = 6
    info = s.flow_step(n)
    phi, vel = s.get_field(velocity=True)
    phi, vel = _np(phi), _np(vel)
    phi_r, v_r, E_r, na_r = orc.flow(theory, f, np.zeros_like(f), h, _params(theory), n, scheme=_scheme(integ))
    rel = 1e-11 if dtype == "f64" else 1e-5
    assert np.abs(phi - phi_r).max() <= rel * np.abs(phi_r).max()
    assert np.abs(vel - v_r).max() <= rel * max(np.abs(phi_r).max(), 1.0)
    if integ == "gf":
        assert not vel.any() and na_r == 0
    assert info["step"] == n and info["n_arrests"] == na_r
    assert info["energy"] == pytest.approx(orc.energy(theory, phi, h, _params(theory)), rel=1e-12, abs=1e-12)
    if dtype == "f64":
        assert info["energy"] == pytest.approx(E_r, rel=1e-12)
    # max |G| reported is that of the final field
    a_ref = orc.acceleration(theory, phi, h, _params(theory))
    assert info["gnorm_inf"] == pytest.approx(np.abs(a_ref).max(), rel=1e-9 if dtype == "f64" else 1e-3)
    assert np.array_equal(phi[:, :2, :], f[:, :2, :]) and np.array_equal(phi[:, :, -2:], f[:, :, -2:])
    s.close()


@pytest.mark.parametrize("integ", INTEGS)
@pytest.mark.parametrize("theory", [AH, CM])
def test_one_pass_exact_gradient_tracks_the_oracle(ss, orc, integ, theory):
    """The one-pass passes also run with the exact gradient h^-2 dE_h/dphi."""
    Nx, Ny, h = 70, 45, 0.2
    print(f"[case] one-pass exact {integ} {theory}", flush=True)
    f = _field(theory, Nx, Ny, h, seed=11)
    s = ss.Solver(theory, Nx, Ny, h, _params(theory), dtype="f64", grad_mode=ss.SS_GRAD_EXACT)
    _set_integ(s, integ)
    s.set_field(f)
    info = s.flow_step(5)
    phi, vel = (_np(x) for x in s.get_field(velocity=True))
    phi_r, v_r, E_r, na_r = orc.flow(theory, f, np.zeros_like(f), h, _params(theory), 5, scheme=_scheme(integ),
                                     mode=orc.GRAD_EXACT)
    assert np.abs(phi - phi_r).max() <= 1e-11 * np.abs(phi_r).max()
    assert np.abs(vel - v_r).max() <= 1e-11 * max(np.abs(phi_r).max(), 1.0)
    assert info["n_arrests"] == na_r and info["energy"] == pytest.approx(E_r, rel=1e-12)
    s.close()


@pytest.mark.parametrize("integ", ["vv", "vv_half"])
def test_runs_compose_and_switch_integrators(ss, orc, integ):
    """Each run starts with a pass that tests the current field and stores its
    force, so with the stored force 3 + 4 steps equal 7 steps bit for bit; in
    the half-step form that pass forms u = v + dt/2 a and the run ends with
    v = u - dt/2 a, so they are equal up to the rounding of that round trip
    (the arrests are the same). A run of RK4 followed by velocity Verlet equals
    the oracle's RK4 then velocity Verlet."""
    Nx, Ny, h = 96, 40, 0.2
    f = _field(AH, Nx, Ny, h, seed=3)
    a = ss.Solver(AH, Nx, Ny, h, [1.0], dtype="f64")
    b = ss.Solver(AH, Nx, Ny, h, [1.0], dtype="f64")
    for s in (a, b):
        _set_integ(s, integ)
        s.set_field(f)
    a.flow_step(3)
    ia = a.flow_step(4)
    ib = b.flow_step(7)
    pa, pb = _np(a.get_field()), _np(b.get_field())
    if integ == "vv":
        assert np.array_equal(pa, pb) and ia["energy"] == ib["energy"]
    else:
        assert np.abs(pa - pb).max() <= 1e-14 * np.abs(pb).max()
        assert ia["energy"] == pytest.approx(ib["energy"], rel=1e-14)
    assert ia["n_arrests"] == ib["n_arrests"] and ia["step"] == 7
    a.set_integrator("rk4")
    a.set_field(f)
    a.flow_step(3)
    a.set_integrator("vv")
    info = a.flow_step(4)
    p1, v1, E1, n1 = orc.flow(AH, f, np.zeros_like(f), h, [1.0], 3)
    p2, v2, E2, n2 = orc.flow(AH, p1, v1, h, [1.0], 4, E_cur=E1, scheme="vv")
    assert np.abs(_np(a.get_field()) - p2).max() <= 1e-11 * np.abs(p2).max()
    assert info["n_arrests"] == n1 + n2 and info["step"] == 7
    a.close()
    b.close()


@pytest.mark.parametrize("integ", INTEGS)
def test_one_pass_arrests_and_stops_like_the_oracle(ss, orc, integ):
    """A long FP64 run: arrests fire at the oracle's steps, and the stall and
    gradient stop rules end the run at the oracle's step."""
    Nx, Ny, h = 48, 40, 0.25
    f = I.ah_vortex_ansatz(Nx, Ny, h, [(0.3, -0.2), (-1.1, 0.9)]) + I.noise(5, 4, Nx, Ny, 1e-3)
    s = ss.Solver(AH, Nx, Ny, h, [1.0], dtype="f64")
    _set_integ(s, integ)
    s.set_field(f)
    phi_r, v_r, E, total = f, np.zeros_like(f), None, 0
    for _ in range(4):
        info = s.flow_step(50)
        phi_r, v_r, E, na = orc.flow(AH, phi_r, v_r, h, [1.0], 50, E_cur=E, scheme=_scheme(integ))
        total += na
        assert info["n_arrests"] == total
    assert np.abs(_np(s.get_field()) - phi_r).max() <= 1e-10 * np.abs(phi_r).max()
    if integ != "gf":
        assert total > 0
    s.set_field(f)
    res = s.minimise(grad_tol=0.0, rel_e_tol=1e-4, window=20, max_steps=5000, graph_steps=8)
    _, _, ref = orc.minimise(AH, f, h, [1.0], grad_tol=0.0, rel_e_tol=1e-4, window=20, max_steps=5000,
                             scheme=_scheme(integ))
    assert res["reason"] == "stall" and ref["reason"] == 2
    assert res["step"] == ref["steps"] and res["n_arrests"] == ref["arrests"]
    assert res["energy"] == pytest.approx(ref["E"], rel=1e-12)
    s.set_field(f)
    res = s.minimise(grad_tol=2e-2, max_steps=5000, graph_steps=8)
    _, _, ref = orc.minimise(AH, f, h, [1.0], grad_tol=2e-2, max_steps=5000, scheme=_scheme(integ))
    assert res["reason"] == "grad" and ref["reason"] == 1 and res["step"] == ref["steps"]
    s.set_field(f)
    res = s.minimise(grad_tol=0.0, max_steps=37, graph_steps=8)
    assert res["reason"] == "max_steps" and res["step"] == 37
    s.close()


@pytest.mark.parametrize("tile", [0, 1])
@pytest.mark.parametrize("integ", ["vv", "vv_stored", "gf"])
def test_large_lattice_one_pass_step_sampled_parity(ss, orc, integ, tile):
    """One step of the 4096^2 GL workload with a one-pass integrator, as the
    benchmark times it (on 64 x 16 and on 64 x 8 tiles, the shapes its autotuner
    picks), on sampled windows: the oracle steps a window whose outer ring of
    M >= 4 sites (two radius-2 stencils per step) is held fixed."""
    N, h, M, S = 4096, 0.2, 6, 64
    print(f"[case] gl4096 one-pass {integ} tile {tile}", flush=True)
    inst = I.gl_large_instance(N, h)
    lam = I.gl_lambda_from_kappa(1.5)
    s = ss.Solver(AH, N, N, h, [lam], dtype="f32")
    s.set_tile(tile)
    assert ss.ss_get_tile(s.ctx) == tile
    _set_integ(s, integ)
    if integ == "vv":
        assert s.vv_form == ss.SS_VV_HALF_STEP  # the form a lattice of this size picks
    s.init_vortices(inst.centres, seed=4, noise_amp=1e-3)
    f0 = s.get_field().double().cpu().numpy()
    info = s.flow_step(1)
    assert info["step"] == 1 and info["nonfinite"] == 0
    f1, v1 = (x.double().cpu().numpy() for x in s.get_field(velocity=True))
    rng = np.random.default_rng(2)
    origins = [tuple(rng.integers(M, N - S - M, size=2)) for _ in range(5)] + [(0, 0), (N - S, N - S)]
    for j0, i0 in origins:
        ja, jb = max(j0 - M, 0), min(j0 + S + M, N)
        ia, ib = max(i0 - M, 0), min(i0 + S + M, N)
        win = np.ascontiguousarray(f0[:, ja:jb + 4, ia:ib + 4])
        w1, wv, _, _ = orc.flow(AH, win, np.zeros_like(win), h, [lam], 1, scheme=_scheme(integ))
        sl = (slice(None), slice(j0 - ja + 2, j0 - ja + S + 2), slice(i0 - ia + 2, i0 - ia + S + 2))
        got = (slice(None), slice(j0 + 2, j0 + S + 2), slice(i0 + 2, i0 + S + 2))
        assert np.abs(f1[got] - w1[sl]).max() <= 1e-5 * max(np.abs(w1[sl]).max(), 1.0), (j0, i0)
        assert np.abs(v1[got] - wv[sl]).max() <= 1e-5 * max(np.abs(w1[sl]).max(), 1.0), (j0, i0)
    s.close()


@pytest.mark.parametrize("integ,theory,dtype", [("vv", AH, "f32"), ("vv", AH, "f64"), ("gf", AH, "f32"),
                                                ("vv", CM, "f32"), ("gf", CM, "f64"), ("vv_stored", AH, "f32")])
def test_one_pass_units_of_several_tiles(ss, orc, integ, theory, dtype):
    """A ragged lattice with 6174 tiles of 64 x 8 (18 x 343), over three times the
    2048 workgroups of a stage launch, so each workgroup walks units of three
    tiles and the second and third take their top rows, and the velocity Verlet
    partial update of their first rows, from LDS: every site against the oracle
    after 3 steps."""
    Nx, Ny, h = 1100, 2740, 0.2
    print(f"[case] one-pass units {integ} {theory} {dtype}", flush=True)
    f = _field(theory, Nx, Ny, h, seed=23)
    if dtype == "f32":
        f = f.astype(np.float32).astype(np.float64)
    s = ss.Solver(theory, Nx, Ny, h, _params(theory), dtype=dtype)
    _set_integ(s, integ)
    s.set_tile(1)
    s.set_field(f)
    n = 3
    info = s.flow_step(n)
    phi, vel = (_np(x) for x in s.get_field(velocity=True))
    phi_r, v_r, E_r, na_r = orc.flow(theory, f, np.zeros_like(f), h, _params(theory), n, scheme=_scheme(integ))
    rel = 1e-11 if dtype == "f64" else 1e-5
    assert np.abs(phi - phi_r).max() <= rel * np.abs(phi_r).max()
    assert np.abs(vel - v_r).max() <= rel * max(np.abs(phi_r).max(), 1.0)
    assert info["step"] == n and info["n_arrests"] == na_r
    if dtype == "f64":
        assert info["energy"] == pytest.approx(E_r, rel=1e-12)
    s.close()


@pytest.mark.parametrize("integ", ["vv", "vv_half", "rk4"])
def test_split_runs_keep_the_oracle_arrests(ss, orc, integ):
    """A flow split into four runs of 50 steps on 64 x 8 tiles, where the passes
    around the half-step form's steps run on 64 x 16 tiles, and RK4's end-of-run
    check and first stage are different launches: each run's first test
    re-evaluates the field the last run ended on, possibly summed in another
    order, and takes no new arrest decision, so the arrests are those of the
    oracle's one continued flow."""
    Nx, Ny, h = 48, 40, 0.25
    print(f"[case] split runs {integ}", flush=True)
    f = I.ah_vortex_ansatz(Nx, Ny, h, [(0.3, -0.2), (-1.1, 0.9)]) + I.noise(5, 4, Nx, Ny, 1e-3)
    s = ss.Solver(AH, Nx, Ny, h, [1.0], dtype="f64")
    if integ == "rk4":
        s.set_integrator("rk4")
    else:
        _set_integ(s, integ)
    s.set_tile(1)
    s.set_field(f)
    scheme = "rk4" if integ == "rk4" else "vv"
    phi_r, v_r, E, total = f, np.zeros_like(f), None, 0
    for _ in range(4):
        info = s.flow_step(50)
        phi_r, v_r, E, na = orc.flow(AH, phi_r, v_r, h, [1.0], 50, E_cur=E, scheme=scheme)
        total += na
        assert info["n_arrests"] == total
    assert total > 0
    assert np.abs(_np(s.get_field()) - phi_r).max() <= 1e-10 * np.abs(phi_r).max()
    s.close()


# lattices on either side of each rule of the default tile's shape: 128 tiles of
# 64 x 16 sites (511 x 253), 135 (555 x 230), and 400000 sites (FP64) and 800000
# (FP32); odd sizes, so that the last tiles and the last units are partial
DEFAULT_TILE_SHAPES = [("f64", 511, 253), ("f32", 511, 253), ("f64", 555, 230), ("f32", 555, 230),
                       ("f64", 1291, 307), ("f64", 1291, 311), ("f32", 1291, 617), ("f32", 1291, 623)]


@pytest.mark.parametrize("theory,integ", [(AH, "vv"), (AH, "gf"), (AH, "rk4"), (CM, "vv"), (CM, "gf"), (CM, "rk4")])
@pytest.mark.parametrize("dtype,Nx,Ny", DEFAULT_TILE_SHAPES)
def test_default_tile_over_lattice_sizes(ss, orc, dtype, Nx, Ny, theory, integ):
    """The default tile's flow over the sizes where its compiled shape changes,
    every site against the oracle."""
    h, n = 0.2, 3
    print(f"[case] default tile {theory} {integ} {dtype} {Nx}x{Ny}", flush=True)
    f = _field(theory, Nx, Ny, h, seed=Nx + Ny)
    if dtype == "f32":
        f = f.astype(np.float32).astype(np.float64)
    s = ss.Solver(theory, Nx, Ny, h, _params(theory), dtype=dtype)
    s.set_integrator(integ)
    s.set_field(f)
    info = s.flow_step(n)
    phi, vel = (_np(x) for x in s.get_field(velocity=True))
    phi_r, v_r, _, na_r = orc.flow(theory, f, np.zeros_like(f), h, _params(theory), n, scheme=integ)
    rel = 1e-11 if dtype == "f64" else 1e-5
    assert np.abs(phi - phi_r).max() <= rel * np.abs(phi_r).max()
    assert np.abs(vel - v_r).max() <= rel * max(np.abs(phi_r).max(), 1.0)
    assert info["step"] == n and info["n_arrests"] == na_r
    assert info["energy"] == pytest.approx(orc.energy(theory, phi, h, _params(theory)), rel=1e-12, abs=1e-12)
    s.close()
