"""The shape that a context or a batch runs: a selected tile is the shape that it is reported as, at
every lattice size; while none is selected the default rule's applies (include/ss.h)."""
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


def _np(t):
    return t.double().cpu().numpy()


# lattices on which the default rule has 64 x 4, 64 x 8 and 64 x 16 sites
@pytest.mark.parametrize("dtype,Nx,Ny,default", [("f64", 150, 37, (64, 4, 1)), ("f32", 150, 37, (64, 8, 2)),
                                                 ("f64", 700, 573, (64, 8, 2)), ("f32", 555, 230, (64, 16, 2))])
@pytest.mark.parametrize("integ", ["vv", "rk4"])
def test_a_selected_tile_is_the_shape_that_runs(ss, orc, dtype, Nx, Ny, default, integ):
    h, n = 0.2, 2
    f = I.ah_vortex_ansatz(Nx, Ny, h, [(0.4, -0.3)]) + I.noise(7, 4, Nx, Ny, 1e-3)
    if dtype == "f32":
        f = f.astype(np.float32).astype(np.float64)
    phi_r = orc.flow(AH, f, np.zeros_like(f), h, [1.0], n, scheme=integ)[0]
    rel = 1e-11 if dtype == "f64" else 1e-5
    print(f"[case] selected tiles {dtype} {integ} {Nx}x{Ny}", flush=True)
    s = ss.Solver(AH, Nx, Ny, h, [1.0], dtype=dtype)
    s.set_integrator(integ)
    assert ss.ss_get_shape(s.ctx) == default and ss.ss_get_tile(s.ctx) == 0
    for tile in range(ss.ss_tile_count()):
        s.set_tile(tile)
        s.set_integrator(integ)  # a selected tile stays
        assert ss.ss_get_shape(s.ctx) == ss.ss_tile_shape(tile) and ss.ss_get_tile(s.ctx) == tile
        s.set_field(f)
        s.flow_step(n)
        assert np.abs(_np(s.get_field()) - phi_r).max() <= rel * np.abs(phi_r).max(), tile
    s.close()


def test_the_environment_selects_tile_zero_as_well(ss, monkeypatch):
    monkeypatch.setenv("SS_TILE", "0")
    s = ss.Solver(AH, 64, 64, 0.2, [1.0], dtype="f64")
    B = ss.Batch(AH, [(64, 64, 0.2, [1.0])], dtype="f64")
    assert ss.ss_get_shape(s.ctx) == ss.ss_batch_get_shape(B.batch) == ss.ss_tile_shape(0) == (64, 16, 2)
    B.close()
    s.close()


@pytest.mark.parametrize("dtype,integ,default", [("f64", "rk4", (64, 8, 2)), ("f32", "vv", (64, 8, 2)),
                                                 ("f32", "rk4", (64, 16, 2))])
def test_a_batch_runs_its_selected_tile(ss, orc, dtype, integ, default):
    sizes, h, n = [(9, 65), (131, 37)], 0.2, 2
    rel = 1e-11 if dtype == "f64" else 1e-5
    print(f"[case] batch selected tiles {dtype} {integ}", flush=True)
    fields = [I.ah_vortex_ansatz(nx, ny, h, [(0.1, -0.1)]) + I.noise(3, 4, nx, ny, 1e-3) for nx, ny in sizes]
    if dtype == "f32":
        fields = [f.astype(np.float32).astype(np.float64) for f in fields]
    refs = [orc.flow(AH, f, np.zeros_like(f), h, [1.0], n, scheme=integ)[0] for f in fields]
    B = ss.Batch(AH, [(nx, ny, h, [1.0]) for nx, ny in sizes], dtype=dtype)
    B.set_integrator(integ)
    assert ss.ss_batch_get_shape(B.batch) == default
    for tile in range(ss.ss_tile_count()):
        B.set_tile(tile)
        B.set_integrator(integ)
        assert ss.ss_batch_get_shape(B.batch) == ss.ss_tile_shape(tile)
        for m, f in zip(B.members, fields):
            m.set_field(f)
        B.flow_step(n)
        for m, r in zip(B.members, refs):
            assert np.abs(_np(m.get_field()) - r).max() <= rel * np.abs(r).max(), tile
    B.close()


def test_autotune_keeps_the_unselected_shape_where_it_is_the_fastest(ss, tmp_path, monkeypatch):
    """64 x 4 sites are none of the tiles: the tuner times them as well, and its file holds -1 for them."""
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("SS_AUTOTUNE_CACHE", str(cache))
    s = ss.Solver(AH, 128, 128, 0.1, [1.0], dtype="f64")
    s.set_integrator("vv")
    best, plan, ms = s.autotune(3)
    timed = [m for row in ms for m in row if m > 0]
    stored = int(cache.read_text().split()[-1])
    assert ms[plan][best] == min(timed) and len(timed) == 2 * ss.ss_tile_count()
    assert ss.ss_get_shape(s.ctx) == ((64, 4, 1) if stored == -1 else ss.ss_tile_shape(stored))
    assert ss.ss_get_tile(s.ctx) == best == max(stored, 0)
    s.close()
    key = cache.read_text().split()[:-1]
    for tile in (-1, 0):
        cache.write_text(" ".join(key + [str(tile)]) + "\n")
        s = ss.Solver(AH, 128, 128, 0.1, [1.0], dtype="f64")
        s.set_integrator("vv")
        s.set_tile(2)
        assert s.autotune(3)[0] == 0 == ss.ss_get_tile(s.ctx)
        assert ss.ss_get_shape(s.ctx) == ((64, 4, 1) if tile == -1 else (64, 16, 2))
        s.close()


# the chiral magnet's velocity Verlet in FP32: 64 x 16 below 4096 tiles of that shape
@pytest.mark.parametrize("dtype,integ,members,default", [("f32", "vv", 2, (64, 16, 2)), ("f32", "vv", 32, (64, 8, 2)),
                                                         ("f32", "vv", 31, (64, 16, 2)), ("f32", "gf", 2, (64, 8, 2)),
                                                         ("f64", "vv", 2, (64, 8, 2))])
def test_a_chiral_magnet_batch_runs_the_faster_shape(ss, orc, dtype, integ, members, default):
    h, n, par = 0.2, 2, [1.0, 1.0, 0.1, 0.6]
    sizes = [(131, 37)] + [(64, 2048)] * (members - 1) + [(64, 16 * (128 - 9))]  # 9 tiles, 128 each, 119
    rel = 1e-11 if dtype == "f64" else 1e-5
    print(f"[case] chiral magnet batch {dtype} {integ} {members}", flush=True)
    f = I.renormalise_interior(I.cm_skyrmion_ansatz(131, 37, h, R=1.0) + I.noise(3, 3, 131, 37, 1e-3))
    if dtype == "f32":
        f = f.astype(np.float32).astype(np.float64)
    ref = orc.flow("chiral_magnet", f, np.zeros_like(f), h, par, n, scheme=integ)[0]
    B = ss.Batch("chiral_magnet", [(nx, ny, h, par) for nx, ny in sizes], dtype=dtype)
    assert ss.ss_batch_get_shape(B.batch) == ((64, 16, 2) if dtype == "f32" else (64, 8, 2))  # RK4
    B.set_integrator(integ)
    assert ss.ss_batch_get_shape(B.batch) == default
    B.members[0].set_field(f)
    for m in B.members[1:]:
        m.init_skyrmion(R=1.0)
    B.flow_step(n)
    assert np.abs(_np(B.members[0].get_field()) - ref).max() <= rel * np.abs(ref).max()
    B.close()


# more tiles than the workgroups of an exact-gradient pass: 16 x 36 and 21 x 65 of 64 x 16 sites
@pytest.mark.parametrize("dtype,Nx,Ny", [("f64", 1021, 571), ("f32", 1291, 1033)])
@pytest.mark.parametrize("integ", ["rk4", "vv", "gf"])
@pytest.mark.parametrize("theory", [AH, "chiral_magnet"])
def test_exact_gradient_flow_of_several_tiles_per_workgroup(ss, orc, theory, integ, dtype, Nx, Ny):
    h, n = 0.17, 3
    par = [1.0] if theory == AH else [1.0, 1.0, 0.1, 0.6]
    print(f"[case] exact several tiles {theory} {integ} {dtype} {Nx}x{Ny}", flush=True)
    if theory == AH:
        f = I.ah_vortex_ansatz(Nx, Ny, h, [(3.4, -2.3)]) + I.noise(7, 4, Nx, Ny, 1e-3)
    else:
        f = I.renormalise_interior(I.cm_skyrmion_ansatz(Nx, Ny, h, R=4.0) + I.noise(7, 3, Nx, Ny, 1e-3))
    if dtype == "f32":
        f = f.astype(np.float32).astype(np.float64)
    phi_r, v_r, E_r, na_r = orc.flow(theory, f, np.zeros_like(f), h, par, n, scheme=integ, mode=orc.GRAD_EXACT)
    rel = 1e-11 if dtype == "f64" else 1e-5
    s = ss.Solver(theory, Nx, Ny, h, par, dtype=dtype, grad_mode=ss.SS_GRAD_EXACT)
    s.set_integrator(integ)
    s.set_field(f)
    info = s.flow_step(n)
    phi, vel = (_np(x) for x in s.get_field(velocity=True))
    assert np.abs(phi - phi_r).max() <= rel * np.abs(phi_r).max()
    assert np.abs(vel - v_r).max() <= rel * max(np.abs(phi_r).max(), 1.0)
    assert info["step"] == n and info["n_arrests"] == na_r
    assert info["energy"] == pytest.approx(orc.energy(theory, phi, h, par), rel=1e-12)
    # a relaxation that stops there leaves the field as its later passes found it
    s.set_field(f)
    s.minimise(grad_tol=0.0, max_steps=n)
    assert np.array_equal(_np(s.get_field()), phi)
    s.close()


@pytest.mark.parametrize("theory", [AH, "chiral_magnet"])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("integ,plan,tiles", [("vv", 1, (0, 1)), ("gf", 1, (0, 1, 2, 3)), ("rk4", 0, (0, 1, 2, 3))])
def test_a_member_and_a_lone_lattice_on_a_selected_tile_are_the_same_bits(ss, theory, dtype, integ, plan, tiles):
    """Stage passes and one-pass integrators (a batch runs velocity Verlet's half-step form)."""
    h, n, sizes = 0.2, 12, [(64, 64), (129, 70), (300, 260), (700, 400)]
    par = [1.3] if theory == AH else [1.0, 1.0, 0.1, 0.6]
    print(f"[case] member and lone lattice {theory} {dtype} {integ}", flush=True)

    def start(s, nx, ny):
        if theory == AH:
            s.init_vortices([(0.03 * nx, 0.1), (-0.03 * nx, -0.02 * ny)], seed=3, noise_amp=1e-3)
        else:
            s.init_skyrmion(R=min(nx, ny) * h / 8, seed=3, noise_amp=1e-3)

    B = ss.Batch(theory, [(nx, ny, h, par) for nx, ny in sizes], dtype=dtype)
    B.set_integrator(integ)
    B.set_plan(plan)
    for tile in tiles:
        B.set_tile(tile)
        for m, (nx, ny) in zip(B.members, sizes):
            start(m, nx, ny)
        B.flow_step(n)
        for m, (nx, ny) in zip(B.members, sizes):
            s = ss.Solver(theory, nx, ny, h, par, dtype=dtype)
            s.set_integrator(integ)
            s.set_plan(plan)
            s.set_vv_form("half_step")
            s.set_tile(tile)
            start(s, nx, ny)
            s.flow_step(n)
            for a, b in zip(m.get_field(velocity=True), s.get_field(velocity=True)):
                assert np.array_equal(_np(a), _np(b)), (tile, nx, ny)
            s.close()
    B.close()
