"""Kernels at the sizes where their paths change: edges of waves, rows shorter
and longer than a wave, single-node axes, walls and periodic faces."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2206_11634_amd import binding as B
from paper_2206_11634_amd import workloads as W

pytestmark = pytest.mark.gpu

NONE = W.make_particles([], np.zeros((0, 3)), np.zeros((0, 4)), 1.0)

# |f - w| stays below 0.03 and each of the 3 steps rounds about ten times at
# that size: 3 * 10 * 0.03 * 2^-24 for float, 3 * 0.03 * 2^-11 for half storage
BULK_TOL = {"f64": 1e-14, "f32": 6e-8, "f16": 5e-5}


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("lattice", [19, 15])
@pytest.mark.parametrize("dims", [(1, 1, 1), (2, 1, 3), (3, 70, 1), (63, 5, 4), (64, 4, 5),
                                  (65, 3, 7), (62, 6, 5), (130, 4, 6), (256, 3, 4), (20, 20, 4)])
def test_stream_collide_at_wave_and_row_edges(storage, lattice, dims):
    """Three steps of random populations against the oracle, for every set of
    periodic axes (waves off the faces, on them, and mixed; both pulls)."""
    rng = np.random.default_rng(5)
    for mask in range(8):
        per = tuple((mask >> a) & 1 for a in range(3))
        lat = W.LatticeSpec(*dims, periodic=per, tau=0.62, body_force=(2e-4, -1e-4, 3e-4))
        gpu, ora = B.Lattice(lat, storage=storage, lattice=lattice), O.Oracle(lat, Q=lattice)
        parts = B.DeviceParticles(NONE)
        ora.classify(NONE)
        _, w, _ = O.stencil(lattice)
        f = w[:, None] * (1.0 + 0.04 * rng.uniform(-1, 1, (lattice, lat.ncell)))
        if storage != "f64":   # values the storage holds
            cut, s = (np.float32, 1.0) if storage == "f32" else (np.float16, 1024.0)
            f = ((f - w[:, None]) * s).astype(cut).astype(np.float64) / s + w[:, None]
        gpu.set_populations(f)
        ora.f[:] = f
        for _ in range(3):
            gpu.step(parts)
            ora.step(NONE)
        assert np.abs(gpu.populations() - ora.f).max() <= BULK_TOL[storage], per
        gpu.close()


@pytest.mark.parametrize("storage,dims", [
    ("f32", (117, 117, 116)), ("f32", (117, 117, 117)), ("f32", (147, 147, 147)), ("f32", (148, 147, 147)),
    ("f64", (92, 92, 94)), ("f64", (93, 93, 93)), ("f16", (146, 147, 147)), ("f16", (148, 147, 147)),
    ("f16", (149, 147, 147))])
def test_stream_collide_at_the_cache_line_of_its_stores(storage, dims):
    """Two levels and the moments just below and just above 2^28 bytes, and for
    float 2^29 (where populations are stored past the cache), two steps of
    random populations against the oracle."""
    rng = np.random.default_rng(6)
    lat = W.LatticeSpec(*dims, periodic=(1, 0, 1), tau=0.62, body_force=(2e-4, -1e-4, 3e-4))
    gpu, ora = B.Lattice(lat, storage=storage), O.Oracle(lat)
    parts = B.DeviceParticles(NONE)
    ora.classify(NONE)
    _, w, _ = O.stencil(19)
    f = w[:, None] * (1.0 + 0.04 * rng.uniform(-1, 1, (19, lat.ncell)))
    if storage != "f64":
        cut, s = (np.float32, 1.0) if storage == "f32" else (np.float16, 1024.0)
        f = ((f - w[:, None]) * s).astype(cut).astype(np.float64) / s + w[:, None]
    gpu.set_populations(f)
    ora.f[:] = f
    for _ in range(2):
        gpu.step(parts)
        ora.step(NONE)
    assert np.abs(gpu.populations() - ora.f).max() <= BULK_TOL[storage]
    gpu.close()


@pytest.mark.parametrize("points", [1, 3, 6, 9])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 130])
def test_dem_paths_match_the_oracle(n, points):
    """dem_step around the particle count where a whole call moves from one
    workgroup to a launch per phase, with bodies of one control point, of three
    (both bodies' points in a group's registers), of six (64 bodies fill the
    workgroup's points) and of nine (neither), touching
    each other, the floor and each other across a periodic face: five calls of
    ten substeps against the oracle, within 1e-9."""
    rng = np.random.default_rng(100 * n + points)
    if points == 1:
        shape = W.sphere_shape(6.2, 0.2)
    else:
        pts = rng.uniform(-0.4, 0.4, (points, 3))
        shape = W.metaball_shape(pts, rng.uniform(0.7, 1.3, points) * 0.9 / points, 0.2, d_eq=6.4,
                                 samples_per_unit=2.0)
    per_row = 6
    rows = -(-n // per_row)
    k = np.arange(n)
    lat = W.LatticeSpec(36, max(6 * rows, 40), 30, (1, 0, 0))
    pos = np.stack([(k % per_row) * 6.0 + 3.0, (k // per_row) * 6.0 + 2.7, np.full(n, 2.5)], -1)
    pos += rng.uniform(-0.1, 0.1, (n, 3))
    quats = np.array([W.random_quaternion(rng) for _ in range(n)])
    ps = W.make_particles([shape] * n, pos, quats, 1.5, vel=rng.normal(size=(n, 3)) * 0.02,
                          omega=rng.normal(size=(n, 3)) * 0.004)
    kw = W.dem_defaults(ps, gravity=(0.0, 0.0, -2e-4))
    gpu, dem = B.Lattice.for_particles(lat, ps, storage="f32"), O.OracleDEM(ps, lat)
    parts, P = B.DeviceParticles(ps), ps.copy()
    zero = np.zeros((n, 3))
    for _ in range(5):
        gpu.dem(parts, 10, 0.1, B.DemParams.make(**kw))
        dem.step(P, zero, zero, O.DemParams(**kw), 10, 0.1)
    gpu.sync()
    G = parts.to_host(ps)
    gpu.close()
    if n > 1:
        assert np.abs(P.vel - ps.vel).max() > 1e-3   # contacts acted
    for key in ("pos", "vel", "omega", "quat", "world_pts"):
        a, b = getattr(G, key), getattr(P, key)
        assert np.abs(a - b).max() <= 1e-9 * max(1.0, np.abs(b).max()), key


@pytest.mark.parametrize("stated", ["none", "one", "all"])
@pytest.mark.parametrize("n,points", [(3, 6), (64, 7), (65, 1), (65, 6), (130, 9)])
def test_dem_of_contexts_that_do_not_state_their_control_points(n, points, stated):
    """dem_step goes by ctrl_off: with lbm_config.n_ctrl left at 0, or below the
    number of bodies, the bodies move as where it is stated, against the oracle
    within 1e-9 (above 64 bodies, and below with more points than a workgroup's
    call holds)."""
    rng = np.random.default_rng(10 * n + points)
    if points == 1:
        shape = W.sphere_shape(6.2, 0.2)
    else:
        pts = rng.uniform(-0.4, 0.4, (points, 3))
        shape = W.metaball_shape(pts, rng.uniform(0.7, 1.3, points) * 0.9 / points, 0.2, d_eq=6.4,
                                 samples_per_unit=2.0)
    k = np.arange(n)
    lat = W.LatticeSpec(36, max(6 * (-(-n // 6)), 40), 30, (1, 0, 0))
    pos = np.stack([(k % 6) * 6.0 + 3.0, (k // 6) * 6.0 + 2.7, np.full(n, 2.5)], -1)
    pos += rng.uniform(-0.1, 0.1, (n, 3))
    quats = np.array([W.random_quaternion(rng) for _ in range(n)])
    ps = W.make_particles([shape] * n, pos, quats, 1.5, vel=rng.normal(size=(n, 3)) * 0.02,
                          omega=rng.normal(size=(n, 3)) * 0.004)
    kw = W.dem_defaults(ps, gravity=(0.0, 0.0, -2e-4))
    n_ctrl = {"none": 0, "one": n - 1, "all": len(ps.K)}[stated]
    gpu = B.Lattice(lat, n_particles=n, n_ctrl=n_ctrl, box_half=ps.box_half(), storage="f32")
    dem, parts, P = O.OracleDEM(ps, lat), B.DeviceParticles(ps), ps.copy()
    zero = np.zeros((n, 3))
    for _ in range(2):
        gpu.dem(parts, 10, 0.1, B.DemParams.make(**kw))
        dem.step(P, zero, zero, O.DemParams(**kw), 10, 0.1)
    gpu.sync()
    G = parts.to_host(ps)
    gpu.close()
    for key in ("pos", "vel", "omega", "quat", "world_pts"):
        a, b = getattr(G, key), getattr(P, key)
        assert np.abs(a - b).max() <= 1e-9 * max(1.0, np.abs(b).max()), key


def test_dem_reports_more_control_points_than_stated():
    """64 bodies of seven points in a context that states 384 of the 448: the next
    synchronisation says so."""
    rng = np.random.default_rng(2)
    shape = W.metaball_shape(rng.uniform(-0.4, 0.4, (7, 3)), np.full(7, 0.13), 0.2, d_eq=6.4,
                             samples_per_unit=2.0)
    k = np.arange(64)
    lat = W.LatticeSpec(40, 40, 160, (0, 0, 0))
    pos = np.stack([(k % 4) * 9.0 + 5.0, (k // 4 % 4) * 9.0 + 5.0, (k // 16) * 30.0 + 20.0], -1)
    ps = W.make_particles([shape] * 64, pos, np.tile([1.0, 0, 0, 0], (64, 1)), 1.5)
    gpu = B.Lattice(lat, n_particles=64, n_ctrl=384, box_half=ps.box_half(), storage="f32")
    gpu.dem(B.DeviceParticles(ps), 2, 0.1, B.DemParams.make(**W.dem_defaults(ps)))
    with pytest.raises(B.LbmError) as e:
        gpu.sync()
    assert e.value.code == B.LBM_ECAPACITY
    gpu.close()


@pytest.mark.parametrize("n", [1, 70])
@pytest.mark.parametrize("tol", [1e-12, 1e-100, 1e-170, 1e-300, 0.0, -1.0])
def test_dem_newton_tolerances(n, tol):
    """Spheres bouncing straight off the floor, whose contact point the search has
    exactly from the start: any positive step tolerance finds it, also one whose
    square underflows, and none that is not positive (no contact then), as the
    oracle's search."""
    k = np.arange(n)
    lat = W.LatticeSpec(64, 80, 30, (0, 0, 0))
    pos = np.stack([(k % 7) * 8.0 + 8.0, (k // 7) * 7.0 + 5.0, np.full(n, 2.55)], -1)
    ps = W.make_particles([W.sphere_shape(6.0, 0.2)] * n, pos, np.tile([1.0, 0, 0, 0], (n, 1)), 1.5,
                          vel=np.tile([0.0, 0.0, -0.05], (n, 1)))
    kw = dict(W.dem_defaults(ps, gravity=(0.0, 0.0, -2e-4)), newton_tol=tol)
    gpu, dem = B.Lattice.for_particles(lat, ps, storage="f32"), O.OracleDEM(ps, lat)
    parts, P = B.DeviceParticles(ps), ps.copy()
    zero = np.zeros((n, 3))
    for _ in range(4):
        gpu.dem(parts, 10, 0.1, B.DemParams.make(**kw))
        dem.step(P, zero, zero, O.DemParams(**kw), 10, 0.1)
    gpu.sync()
    G = parts.to_host(ps)
    gpu.close()
    assert (P.vel[:, 2].min() > -0.045) == (tol > 0.0)   # the floor slowed them, or did not
    for key in ("pos", "vel", "omega"):
        assert np.abs(getattr(G, key) - getattr(P, key)).max() <= 1e-9 * max(1.0, np.abs(getattr(P, key)).max())


@pytest.mark.parametrize("n", [1, 70])
@pytest.mark.parametrize("mu", [-5.0, -0.2, 0.0, 0.3, float("inf")])
def test_dem_friction_coefficients(n, mu):
    """Spheres sliding over the floor: the Coulomb limit for friction coefficients
    of every kind acts as the oracle's."""
    k = np.arange(n)
    lat = W.LatticeSpec(64, 80, 30, (0, 0, 0))
    pos = np.stack([(k % 7) * 8.0 + 8.0, (k // 7) * 7.0 + 5.0, np.full(n, 2.48)], -1)
    ps = W.make_particles([W.sphere_shape(6.0, 0.2)] * n, pos, np.tile([1.0, 0, 0, 0], (n, 1)), 1.5,
                          vel=np.tile([0.02, -0.01, 0.0], (n, 1)))
    kw = dict(W.dem_defaults(ps, gravity=(0.0, 0.0, -2e-4)), mu_s=mu)
    gpu, dem = B.Lattice.for_particles(lat, ps, storage="f32"), O.OracleDEM(ps, lat)
    parts, P = B.DeviceParticles(ps), ps.copy()
    zero = np.zeros((n, 3))
    for _ in range(3):
        gpu.dem(parts, 10, 0.1, B.DemParams.make(**kw))
        dem.step(P, zero, zero, O.DemParams(**kw), 10, 0.1)
    gpu.sync()
    G = parts.to_host(ps)
    gpu.close()
    assert (np.abs(P.omega).max() > 1e-6) == (mu != 0.0)   # friction turned them
    for key in ("pos", "vel", "omega"):
        assert np.abs(getattr(G, key) - getattr(P, key)).max() <= 1e-9 * max(1.0, np.abs(getattr(P, key)).max())


@pytest.mark.parametrize("n,points", [(1, 1), (1, 64), (2, 20), (21, 6), (22, 6), (64, 1), (64, 6), (70, 6)])
def test_dem_wall_contacts_of_bodies_in_a_channel(n, points):
    """Bodies between two walls and on the floor, apart from each other, some next
    to the end walls: up to 64 of them give a workgroup's first wave less and more
    wall contacts than it has lanes.  Three calls of ten substeps against the
    oracle, within 1e-9."""
    rng = np.random.default_rng(n + points)
    d = 6.2
    if points == 1:
        shape = W.sphere_shape(d, 0.2)
    else:
        pts = rng.uniform(-0.3, 0.3, (points, 3))
        shape = W.metaball_shape(pts, rng.uniform(0.7, 1.3, points) * 0.9 / points, 0.2, d_eq=d,
                                 samples_per_unit=2.0)
    lat = W.LatticeSpec(max(9 * n, 20), 6, 30, (0, 0, 0))
    k = np.arange(n)
    pos = np.stack([np.where(k == 0, 2.5, 9.0 * k + 4.5), np.full(n, 2.5), np.full(n, 2.5)], -1)
    pos += rng.uniform(-0.02, 0.02, (n, 3))
    ps = W.make_particles([shape] * n, pos, np.array([W.random_quaternion(rng) for _ in range(n)]), 1.5,
                          vel=rng.normal(size=(n, 3)) * 0.01, omega=rng.normal(size=(n, 3)) * 0.004)
    kw = W.dem_defaults(ps, gravity=(0.0, 0.0, -2e-4))
    gpu = B.Lattice(lat, n_particles=n, n_ctrl=len(ps.K), box_half=ps.box_half(), storage="f32")
    dem, parts, P = O.OracleDEM(ps, lat), B.DeviceParticles(ps), ps.copy()
    zero = np.zeros((n, 3))
    for _ in range(3):
        gpu.dem(parts, 10, 0.1, B.DemParams.make(**kw))
        dem.step(P, zero, zero, O.DemParams(**kw), 10, 0.1)
    gpu.sync()
    G = parts.to_host(ps)
    gpu.close()
    assert (np.abs(P.vel - ps.vel)[:, 1:] > 1e-5).sum() >= n   # the walls acted
    for key in ("pos", "vel", "omega", "quat", "world_pts"):
        a, b = getattr(G, key), getattr(P, key)
        assert np.abs(a - b).max() <= 1e-9 * max(1.0, np.abs(b).max()), key


@pytest.mark.parametrize("n,spacing", [(2048, 3.0), (2050, 13.0), (16384, 3.0), (16385, 3.0)])
def test_dem_cell_grids_match_the_oracle(n, spacing):
    """dem_step on the cell grid where its making moves from one workgroup to a
    launch per phase, and on a sparse box with more room than cells: spheres
    next to each other in couples, on walls and across a periodic face, one call
    of two substeps against the oracle, within 1e-9."""
    rng = np.random.default_rng(n)
    m = int(np.ceil((n / 2) ** (1 / 3)))
    k = np.arange(n) // 2
    pitch = np.array([2 * spacing, spacing, spacing])
    pos = np.stack([k % m, k // m % m, k // (m * m)], -1) * pitch
    pos[:, 0] += np.where(np.arange(n) % 2, 2.9, 0.0)
    pos += 0.9 + rng.uniform(0, 0.2, (n, 3))
    dims = [int(np.ceil(2 * spacing * m)), int(np.ceil(spacing * m)), int(np.ceil(spacing * m)) + 2]
    lat = W.LatticeSpec(*dims, (1, 0, 0))
    ps = W.make_particles([W.sphere_shape(3.0, 0.2)] * n, pos, np.tile([1.0, 0, 0, 0], (n, 1)), 1.5,
                          vel=rng.normal(size=(n, 3)) * 0.02, omega=rng.normal(size=(n, 3)) * 0.004)
    kw = W.dem_defaults(ps, gravity=(0.0, 0.0, -2e-4))
    gpu, dem = B.Lattice.for_particles(lat, ps, storage="f16"), O.OracleDEM(ps, lat)
    parts, P = B.DeviceParticles(ps), ps.copy()
    gpu.dem(parts, 2, 0.25, B.DemParams.make(**kw))
    zero = np.zeros((n, 3))
    dem.step(P, zero, zero, O.DemParams(**kw), 2, 0.25)
    gpu.sync()
    G = parts.to_host(ps)
    gpu.close()
    assert np.count_nonzero(np.abs(P.vel - ps.vel).max(1) > 1e-4) > n // 4   # contacts acted
    for key in ("pos", "vel", "omega"):
        a, b = getattr(G, key), getattr(P, key)
        assert np.abs(a - b).max() <= 1e-9 * max(1.0, np.abs(b).max()), key


def test_link_adjoint_on_both_sides_of_the_wave_split():
    """The adjoint of the links of 40 spheres (a wave per 64 records) and of 530
    (a workgroup per 256-record chunk): the dot products of the larger set, and
    the derivatives of the 40 spheres, which the other 490, more than two nodes
    away, do not change beyond the order of the sums."""
    from test_gpu_adjoint_dot import _Replay, _near_equilibrium, _replay_case
    rng = np.random.default_rng(8)
    m, n = 40, 530
    k = np.arange(n)
    lat = W.LatticeSpec(60, 60, 40, (1, 1, 0), tau=0.62, body_force=(1e-5, 0.0, 2e-5))
    pos = np.stack([(k % 10) * 6.0 + 3.0, (k // 10 % 10) * 6.0 + 3.0, (k // 100) * 6.0 + 4.0], -1)
    pos += rng.uniform(-0.4, 0.4, (n, 3))

    def spheres(count):
        rng = np.random.default_rng(9)
        v, om = rng.normal(size=(n, 3)) * 0.02, rng.normal(size=(n, 3)) * 0.01
        return W.make_particles([W.sphere_shape(3.3, 0.2)] * count, pos[:count],
                                np.tile([1.0, 0, 0, 0], (count, 1)), 1.5, vel=v[:count],
                                omega=om[:count])
    f0 = _near_equilibrium(lat, rng)
    few, many = _Replay(lat, spheres(m), 3), _Replay(lat, spheres(n), 3)
    _replay_case(many, f0, 31, 1e-7)
    lam1 = rng.normal(size=f0.shape) * (many.owners(f0)[1] == 0)[None, :]
    w = rng.normal(size=(n, 6))
    lam_a, g_a, x_a = few.run(f0, lam1=lam1, w=w[:m], adjoint=True)
    lam_b, g_b, x_b = many.run(f0, lam1=lam1, w=w, adjoint=True)
    inner = lambda a: a.reshape(-1, 40, 60, 60)[:, :6, 5:20]   # nodes of the 40 spheres alone
    for a, b in ((inner(lam_a), inner(lam_b)), (g_a[4:], g_b[4:4 + 3 * m]), (x_a, x_b[:, :m])):
        assert np.abs(a).max() > 0.1
        assert np.abs(a - b).max() <= 1e-12 * np.abs(a).max()


@pytest.mark.parametrize("dims", [(84, 84, 83), (84, 84, 84), (133, 133, 133), (134, 133, 133)])
def test_node_adjoint_at_the_cache_line_of_its_stores(dims):
    """Two FP64 adjoint fields and a taped level just below and above 2^28 and
    2^30 bytes (between them the taped level and the whole planes go past the
    cache): the dot products of a step with two moving bodies and a refill, to
    the bound that the smaller lattices meet."""
    from test_gpu_adjoint_dot import _Replay, _near_equilibrium, _one_body, _replay_case
    _, ps = _one_body([[0.12, 0.03, -0.02], [-0.08, 0.05, 0.1]],
                      [[0.01, -0.02, 0.015], [0.0, 0.01, -0.02]])
    lat = W.LatticeSpec(*dims, (1, 0, 1), tau=0.6, body_force=(1e-5, 0.0, 0.0))
    f0 = _near_equilibrium(lat, np.random.default_rng(4))
    _replay_case(_Replay(lat, ps, 3), f0, 41, 1e-7)


# bodies, diameter, box, periodic axes: boxes below and above a wave of rows
# with few planes (a workgroup each) and with many (a wave each), planes of more
# segments and more candidates than are listed at a time, squares around the
# ball of 1, 2 and 3 tiles
@pytest.mark.parametrize("n,d,dims,per,lattice",
                         [(1, 6.0, (33, 40, 35), (1, 1, 1), 15), (2, 29.0, (70, 64, 66), (0, 0, 0), 19),
                          (1, 31.6, (130, 64, 66), (1, 0, 0), 19), (1, 150.0, (160, 158, 156), (0, 0, 0), 19),
                          (230, 7.0, (47, 60, 50), (1, 1, 0), 19), (60, 72.0, (84, 90, 88), (0, 0, 0), 15),
                          (60, 28.0, (131, 60, 62), (1, 0, 0), 19)])
def test_classification_at_plane_and_tile_edges(n, d, dims, per, lattice):
    """Owners, links with q and refills of overlapping spheres, moved once,
    against the oracle bit for bit."""
    from test_gpu_parity import _compare_geometry
    rng = np.random.default_rng(3 * n + lattice)
    lat = W.LatticeSpec(*dims, per)
    pos = np.array(dims) * 0.5 + (rng.uniform(-0.5, 0.5, (n, 3)) * (np.array(dims) - d * 0.9) if n > 1
                                  else rng.uniform(-1, 1, (n, 3)))
    pos = np.where(np.array(per, bool), np.mod(pos, dims), pos)
    ps = W.make_particles([W.sphere_shape(d, 0.2)] * n, pos, np.tile([1.0, 0, 0, 0], (n, 1)), 1.5)
    gpu, ora = (B.Lattice.for_particles(lat, ps, storage="f32", lattice=lattice, classify="balls"),
                O.Oracle(lat, Q=lattice))
    for _ in range(2):
        gpu.classify(B.DeviceParticles(ps))
        ora.classify(ps)
        _compare_geometry(gpu, ora, f"{n} of {d}")
        ps = ps.copy()
        ps.pos += rng.uniform(-0.4, 0.4, (n, 3))
        ps.pos = np.where(np.array(per, bool), np.mod(ps.pos, dims), ps.pos)
        ps.refresh_world()
    gpu.close()


@pytest.mark.parametrize("exact", [False, True])
def test_force_sums_and_counters_between_steps(exact):
    """Forces of steps with and without a classification before them, after a
    classification that failed, and of replayed captured steps with eager work
    between the replays: the sums start from zero each time, and the counters of
    one classification do not reach the next."""
    lat, ps = W.tiny_case(21, dims=(34, 30, 32), periodic=(1, 0, 1), n_particles=3,
                          diameter_range=(5.0, 8.0), speed=0.05, spin=0.004, u0=(0.02, 0.0, 0.01))
    import torch
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        gpu, ora = (B.Lattice.for_particles(lat, ps, storage="f64", exact_forces=exact),
                    O.Oracle(lat, Q=19))
        parts, bad = B.DeviceParticles(ps), B.DeviceParticles(ps)
        bad.t["pos"][1, 0] = float("nan")

        def same(what):
            Fo, To = ora.step(P)
            F, T = (t.cpu().numpy()[:ps.n] for t in gpu.forces())
            assert np.abs(F - Fo).max() <= 1e-10 * np.abs(Fo).max(), what
            assert np.abs(T - To).max() <= 1e-10 * np.abs(To).max(), what

        for n in range(4):
            P = W.prescribed_state(ps, lat, float(n))
            parts.set_state(P)
            if n == 2:
                with pytest.raises(B.LbmError):
                    gpu.classify(bad)
            c = gpu.classify(parts)
            ora.classify(P)
            assert c.n_links == len(ora.links) and (n == 0 or c.n_refill == len(ora.refill_nodes))
            for k in range(2):
                gpu.step(parts)
                same((n, k))
        gpu.sync()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            gpu.step(parts)
            gpu.step(parts)
        for n in range(3):
            graph.replay()
            ora.step(P)
            same(("replay", n))
            gpu.step(parts)      # eager steps between the replays
            same(("eager", n, 0))
            gpu.step(parts)
            same(("eager", n, 1))
        gpu.sync()
        gpu.close()


@pytest.mark.parametrize("n", [1, 32, 33, 700, 4100])
def test_counts_of_many_bodies_are_reported_and_latched(n):
    """Every particle's counts reach the host, whichever workgroup reports them
    (one wave for a few bodies, all of the refill's for many), on the first
    classification and the next; and an asynchronous classification in which the
    links of the first, a middle or the last body outgrow their list is latched."""
    m = int(np.ceil(n ** (1 / 3)))
    k = np.arange(n)
    pos = np.stack([k % m, k // m % m, k // (m * m)], -1) * 14.0 + 8.0
    pos += np.random.default_rng(n).uniform(-0.5, 0.5, (n, 3))
    lat = W.LatticeSpec(14 * m + 6, 14 * m + 6, 14 * m + 6, (0, 0, 0))
    big = W.make_particles([W.sphere_shape(11.6, 0.2)] * n, pos, np.tile([1.0, 0, 0, 0], (n, 1)), 1.5)
    ps = W.make_particles([W.sphere_shape(5.8, 0.2)] * n, pos, np.tile([1.0, 0, 0, 0], (n, 1)), 1.5)
    for j in sorted({0, n // 2, n - 1}):
        gpu = B.Lattice(lat, n_particles=n, n_ctrl=n, box_half=big.box_half(), storage="f16",
                        classify="balls")
        parts = B.DeviceParticles(ps)
        for _ in range(3):
            c = gpu.classify(parts)
            L = gpu.links()
            per_body = np.bincount(L["part"], minlength=n)
            assert c.n_links == len(L["node"]) and per_body.min() > 100
            alone = np.unique(np.stack([L["node"], L["d"]]), axis=1).shape[1]
            assert alone == len(L["node"])       # no record written over another
        gpu.classify(parts, sync=False)
        gpu.sync()
        parts.t["K"][j] *= (11.6 / 5.8) ** 2
        gpu.classify(parts, sync=False)
        with pytest.raises(B.LbmError) as e:
            gpu.sync()
        assert e.value.code == B.LBM_ECAPACITY
        gpu.close()


@pytest.mark.parametrize("n,points,width,mode", [(3, 64, 0.5, "balls"), (3, 64, 1.6, "sweep"), (70, 24, 0.9, "balls"),
                                                 (400, 12, 0.9, "balls"), (400, 40, 0.3, "sweep")])
def test_classification_of_many_point_bodies(n, points, width, mode):
    """Owners, links with q and refills of bodies whose control points lie close
    together or apart (few or many of the visited nodes interior), by four waves
    and by one wave a plane, moved once, against the oracle bit for bit."""
    from test_gpu_parity import _compare_geometry
    rng = np.random.default_rng(points)
    d, c0 = 10.0, 0.97
    pts = rng.uniform(-width / 2, width / 2, (points, 3)) * d
    pts -= pts.mean(0)
    K = rng.uniform(0.7, 1.3, points) / points * (0.4 * d) ** 2
    V = np.pi / 6 * d ** 3
    shape = W.Shape(pts=pts, K=K, c0=c0, rs=0.2, volume=V, inertia_unit=np.full(3, 0.1 * V * d * d),
                    radius=W.body_radius(pts, K, c0))
    m, k, pitch = int(np.ceil(n ** (1 / 3))), np.arange(n), 1.7 * shape.radius
    side = max(int(m * pitch) + 2, 2 * int(shape.radius) + 14)
    lat = W.LatticeSpec(side, side + 1, side + 3, (1, 0, 0))
    pos = np.stack([k % m, k // m % m, k // (m * m)], -1) * pitch + pitch / 2
    pos = np.mod(pos + rng.uniform(-0.5, 0.5, (n, 3)), side)
    ps = W.make_particles([shape] * n, pos, np.array([W.random_quaternion(rng) for _ in range(n)]), 1.5)
    gpu = B.Lattice.for_particles(lat, ps, storage="f32", classify=mode)
    ora = O.Oracle(lat)
    for _ in range(2):
        gpu.classify(B.DeviceParticles(ps))
        ora.classify(ps)
        _compare_geometry(gpu, ora, (n, points))
        ps = ps.copy()
        ps.pos = np.mod(ps.pos + rng.uniform(-0.4, 0.4, (n, 3)), side)
        ps.refresh_world()
    gpu.close()
