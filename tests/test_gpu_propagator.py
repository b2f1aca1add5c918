"""The mixed path's propagator over its plans and tile edges.

One step from random orthonormal orbitals against the oracle's exponential.
The ensemble's velocities run from rest to two hundred times thermal, so one
launch holds the plans of the interaction picture (one to three sub-intervals,
two to eight low-rank columns, one to many Taylor terms) and the trajectories
that take the Chebyshev series.

Tolerance, absolute on coefficients of modulus at most one: rounding the
orbitals to FP32 at the upload, the phases before and after each of up to three
sub-intervals (two roundings of 2^-24 each), the products' 2^-21 of ||M|| < 0.3
per sub-interval and the truncation of at most 2^-24: below 1e-6.  The
Chebyshev series rounds in each of its up to 60 terms: 4e-6.
"""
import numpy as np
import pytest

from oracle import dynamics as dyn, models
from test_gpu_parity import ensemble, gpu, make_cfg, random_states, upload  # noqa: F401

pytestmark = pytest.mark.gpu

FACTORS = np.array([0.0, 1e-3, 0.2, 0.7, 1.3, 2.5, 5.0, 9.0, 15.0, 30.0, 60.0, 200.0])


# row tiles 1, 2, 3, 6, 7, 8, 12, 13, 14, 17, 21 (full and one row over), odd
# and single orbital tiles, both baths, one and six coordinates, repeated levels
@pytest.mark.parametrize("name,M,N", [
    ("c1", 1, 1), ("c1", 15, 8), ("c2", 16, 9), ("c2gl", 46, 17), ("c2", 95, 48), ("c3", 96, 41),
    ("c2", 127, 20), ("c3", 190, 95), ("c2", 200, 100), ("c2gl", 208, 104), ("c2", 223, 30),
    ("c5", 256, 128), ("c5", 20, 7), ("c3", 320, 160), ("c1", 335, 168),
])
def test_mixed_step_over_plans_and_tiles(name, M, N):
    cfg = make_cfg(name, M=M, N=N)
    m = models.from_config(cfg, M=M)
    T = len(FACTORS)
    nd = m.n_dof
    rs = np.random.default_rng(M)
    xs = np.linspace(3.0, 9.0, T) if name == "c3" else np.linspace(-4.0, 10.0, T)
    vth = 2e-3 if name == "c3" else 7e-4
    states = random_states(m, N, T, seed=5 + M, xs=xs, v_scale=0.0)
    for t, s in enumerate(states):
        if nd > 1:
            dof = np.array(cfg["model"]["dof"])
            s.x = dof[:, 3] + 0.1 * rs.normal(size=nd)
            s.v = FACTORS[t] * vth * rs.normal(size=nd)
        else:
            s.v[0] = FACTORS[t] * vth * (1 if t % 2 else -1)
    ens = ensemble(cfg, T, precision="mixed")
    upload(ens, states)
    ens.step()
    x, v, Cf, occ = ens.get_state()
    status = ens.status()
    from paper_2212_00518_amd import unpack_C
    ok = 0
    for t in range(T):
        if status[t]:  # the series did not converge within its terms
            assert FACTORS[t] >= 30.0
            continue
        F = dyn.el.forces(m, states[t].x, states[t].s)
        ref = dyn.step(m, states[t], cfg["dt"], 2.0, F)[0]
        err = np.max(np.abs(unpack_C(Cf, t, m.n, N, ens.n_max, ens.N_max) - ref.C))
        print(f"{name} M={M} v x {FACTORS[t]}: |dC| {err:.2e}", flush=True)
        assert err <= (1e-6 if FACTORS[t] < 9.0 else 4e-6), (t, err)
        ok += 1
    assert ok >= 8
    ens.close()


def test_mixed_propagator_product_counts():
    """At rest one product per step is enough, a thermal trajectory takes two
    to four, and a fast one the Chebyshev series' (eight at M = 200)."""
    counts = {}
    for f in (0.0, 1.0, 60.0):
        cfg = make_cfg("c2", M=200, N=100)
        ens = ensemble(cfg, 1, precision="mixed")
        m = models.from_config(cfg, M=200)
        states = random_states(m, 100, 1, seed=3, xs=[1.0], v_scale=0.0)
        states[0].v[0] = f * 7e-4
        upload(ens, states)
        ens.timing(False)
        ens.run(1)
        counts[f] = ens.work()[0]
        ens.close()
    assert counts[0.0] <= 2 and 2 <= counts[1.0] <= 4 and counts[60.0] >= 8, counts


# rows of the coupling matrix dealt to 8, 4, 2 and 1 threads and two rows a
# thread; series of 1 to about 60 terms
@pytest.mark.parametrize("dt_factor", [1e-6, 0.3, 1.0, 8.0, 18.0])
@pytest.mark.parametrize("M,N", [(1, 1), (15, 8), (31, 9), (40, 20), (64, 20), (127, 40), (200, 20), (300, 12)])
def test_fp64_series_over_orders_and_terms(M, N, dt_factor):
    """One FP64 step against the oracle's exponential: the series' tail and
    the roundings of up to 63 terms, the roots' 3e-15 times the phase (18 at most)
    and the oracle's own rounding: below 1e-12."""
    cfg = make_cfg("c2", M=M, N=N)
    cfg["dt"] *= dt_factor
    m = models.from_config(cfg, M=M)
    states = random_states(m, N, 3, seed=77 + M, xs=[-2.0, 1.0, 6.0], v_scale=7e-4 / max(1.0, dt_factor))
    ens = ensemble(cfg, 3)
    upload(ens, states)
    ens.step()
    x, v, C, occ = ens.get_state()
    assert np.all(ens.status() == 0)
    from paper_2212_00518_amd import unpack_C
    for t in range(3):
        F = dyn.el.forces(m, states[t].x, states[t].s)
        ref = dyn.step(m, states[t], cfg["dt"], 2.0, F)[0]
        err = np.max(np.abs(unpack_C(C, t, m.n, N, ens.n_max, ens.N_max) - ref.C))
        print(f"M={M} dt x {dt_factor}: |dC| {err:.2e}", flush=True)
        assert err <= 1e-12
    ens.close()


# one, two and three row tiles to a wave, full and half last blocks of columns,
# odd orbital tiles, four and eight waves; 48 takes the FP64 instructions
@pytest.mark.parametrize("M,N", [(48, 9), (100, 8), (111, 41), (120, 60), (130, 20), (144, 24), (200, 100), (207, 17),
                                 (255, 33), (256, 128), (320, 160), (335, 7)])
@pytest.mark.parametrize("scale", [0.0, 2.0 ** -60, 2.0 ** 45])
def test_fp64_orbitals_keep_their_scale(M, N, scale):
    """The propagation is linear, and everything in it is scaled by powers of
    two: orbitals times 2^k give the result times 2^k to the bit, whatever the
    other orbitals' scales, and zero orbitals stay zero.  Against the oracle's
    exponential within 1e-12 of an orbital's norm."""
    cfg = make_cfg("c2", M=M, N=N)
    m = models.from_config(cfg, M=M)
    states = random_states(m, N, 2, seed=5 + M, xs=[-2.0, 3.0], v_scale=2e-3)
    ref = [dyn.step(m, s, cfg["dt"], 2.0, dyn.el.forces(m, s.x, s.s))[0].C for s in states]
    from paper_2212_00518_amd import unpack_C
    out = []
    for f in (1.0, scale):
        ens = ensemble(cfg, 2)
        for s in states:
            s.C = s.C.copy()
            s.C[:, ::3] *= f
        upload(ens, states)
        ens.step()
        C = ens.get_state()[2]
        out.append([unpack_C(C, t, m.n, N, ens.n_max, ens.N_max) for t in range(2)])
        ens.close()
    for t in range(2):
        assert np.max(np.abs(out[0][t] - ref[t])) <= 1e-12
        want = out[0][t].copy()
        want[:, ::3] *= scale
        assert np.array_equal(out[1][t], want)


@pytest.mark.parametrize("M,N", [(44, 25), (106, 53)])
def test_mixed_phases_round_independently(M, N):
    """Thermal orbitals on a Gauss-Legendre bath, whose levels crowd at the
    Fermi level, where the phase of a sub-step is small.  A propagation takes
    two rotations of at most two roundings each, and both parts of a number of
    modulus at most one round: were the roundings independent (uniform within
    2^-25), the error after n propagations would be sqrt(8 n) 2^-25 / sqrt(3).
    A rounding that repeats itself step after step exceeds that."""
    cfg = make_cfg("c2gl", M=M, N=N)
    T, steps, sub = 48, 99, 2
    rs = np.random.default_rng(M)
    mass, omega, kT = cfg["model"]["mass"], cfg["model"]["omega"], cfg["kT"]
    x = rs.normal(0.0, np.sqrt(kT / (mass * omega ** 2)), T)
    v = rs.normal(0.0, np.sqrt(kT / mass), T)
    out = []
    for precision in ("fp64", "mixed"):
        ens = ensemble(cfg, T, precision=precision, elec_substeps=sub, lowdin_every=0)
        ens.init_thermal(x, v)
        ens.run(steps)
        out.append(ens.get_state())
        ens.close()
    same = np.all(out[0][3] == out[1][3], axis=1) & (np.abs(out[0][0] - out[1][0]) < 1e-9)  # the same hops
    assert np.sum(same) >= 40
    C64, C32 = (o[2].reshape(T, -1)[same] for o in out)
    err = np.linalg.norm(C32 - C64, axis=1) / np.linalg.norm(C64, axis=1)
    rms = np.sqrt(np.mean(err ** 2))
    print(f"M={M}: rms relative error {rms:.2e}", flush=True)
    assert rms <= np.sqrt(8.0 * steps * sub) * 2.0 ** -25 / np.sqrt(3.0)


# half the 64 eV band times the step: 31.8, 36.5 and 47; the FP32 series has
# its 62 terms up to 35.9 and refuses a longer step
@pytest.mark.parametrize("M,N", [(40, 20), (160, 80)])
@pytest.mark.parametrize("dt,accepted", [(27.0, True), (31.0, False), (40.0, False)])
def test_steps_beyond_the_series_stay_refused(M, N, dt, accepted):
    """Trajectories at rest and slow ones, whose propagator the interaction
    picture needs no series for, are refused with the others."""
    from paper_2212_00518_amd import _lib
    cfg = make_cfg("c3", M=M, N=N)
    cfg["dt"] = dt
    m = models.from_config(cfg, M=M)
    T = 4
    states = random_states(m, N, T, seed=M, xs=np.linspace(4.0, 8.0, T), v_scale=0.0)
    for t, s in enumerate(states):
        s.v[0] = -1e-6 * t
    ens = ensemble(cfg, T, precision="mixed", lowdin_every=0)
    upload(ens, states)
    ens.step()
    status = ens.status()
    ens.close()
    assert np.all(status == (0 if accepted else _lib.TRAJ_NONCONV)), status


# more items than work-groups, in slabs of three tiles and of one, of the first
# and the second register tier, and fewer; the queue is filled anew by every
# sub-step
@pytest.mark.parametrize("precision,tol", [("mixed", 4e-6), ("fp64", 1e-12)])
@pytest.mark.parametrize("substeps", [1, 2])
@pytest.mark.parametrize("name,M,N,T", [("c3", 40, 20, 1500), ("c2", 100, 50, 300), ("c3", 160, 80, 160),
                                        ("c2", 260, 40, 320), ("c2", 100, 50, 24)])
def test_long_queues_of_the_series(name, M, N, T, substeps, precision, tol):
    """Ensembles of which two thirds are too fast for the interaction picture
    and for 8-bit digits, over three steps: a sample against the oracle (the
    series' bound for each of its up to six propagations), and all states bit
    by bit with and without the no-hop bound, which reads the row norms by
    slab."""
    cfg = make_cfg(name, M=M, N=N)
    m = models.from_config(cfg, M=M)
    steps = 3
    rs = np.random.default_rng(M + T)
    x = rs.uniform(4.0, 9.0, T)
    v = np.where(np.arange(T) % 3 == 0, 0.0, (0.1 if name == "c3" else 0.03) * rs.choice([-1.0, 1.0], T))
    C = np.stack([random_states(m, N, 1, seed=q, xs=[0.0], v_scale=0.0)[0].C for q in range(8)])
    states = [dyn.State([x[t]], [v[t]], C[t % 8], np.arange(N)) for t in range(T)]
    out = []
    for off in (0, 1):
        ens = ensemble(cfg, T, precision=precision, elec_substeps=substeps, lowdin_every=0, hop_filter_off=off)
        upload(ens, states)
        ens.run(steps)
        out.append(ens.get_state())
        assert np.all(ens.status() == 0)
        terms = ens.work()[0] / (T * steps * substeps)
        ens.close()
    assert all(np.array_equal(a, b) for a, b in zip(*out))
    print(f"products per propagation {terms:.1f}", flush=True)
    assert terms > 5.0  # a plan takes at most four at rest
    from paper_2212_00518_amd import unpack_C
    ok = 0
    for t in np.unique(np.linspace(0, T - 1, 12).astype(int)):
        ref, _, _ = dyn.run(m, states[t], cfg["dt"], steps, cfg["seed"], int(t), substeps=substeps)
        if not np.array_equal(out[0][3][t][:N], ref.s):
            continue  # another hop
        err = np.max(np.abs(unpack_C(out[0][2], t, m.n, N, m.n, N) - ref.C))
        assert err <= tol * steps * substeps, (t, err)
        ok += 1
    assert ok >= 6


@pytest.mark.parametrize("name,M,N,v,dt_factor", [("c2", 120, 60, 0.07, 8.0), ("c2", 200, 100, 0.07, 8.0),
                                                  ("c3", 160, 80, 0.3, 1.0), ("c3", 320, 160, 0.3, 1.0)])
def test_fast_fp64_steps_keep_orbitals_orthogonal(name, M, N, v, dt_factor):
    """One FP64 step of unit orbitals.  An FP64 series of K <= 62 terms rounds
    every element by at most K units of 2^-53 of itself, so the overlaps of
    different orbitals, 2 Re <C_j, dC_k> with C_j near a unit vector, stay
    within 2 K 2^-53 of the orbitals' other elements (rms over all pairs).
    Fixed-point products, whose error is relative to the largest element,
    exceed that on a fast step."""
    cfg = make_cfg(name, M=M, N=N)
    cfg["dt"] *= dt_factor
    m = models.from_config(cfg, M=M)
    T = 4
    xs = np.linspace(4.0, 4.3, T) if name == "c3" else np.linspace(0.0, 2.0, T)
    states = [dyn.State([xs[t]], [v], np.eye(m.n, N, dtype=np.complex128), np.arange(N)) for t in range(T)]
    ens = ensemble(cfg, T)
    upload(ens, states)
    ens.step()
    Cf = ens.get_state()[2]
    assert np.all(ens.status() == 0)
    ens.close()
    from paper_2212_00518_amd import unpack_C
    off = ~np.eye(N, dtype=bool)
    overlap, rest = [], []
    for t in range(T):
        C = unpack_C(Cf, t, m.n, N, m.n, N)
        re, im = C.real.astype(np.longdouble), C.imag.astype(np.longdouble)
        G = np.hypot(re.T @ re + im.T @ im, re.T @ im - im.T @ re)
        overlap.append(np.sqrt(np.mean(G[off] ** 2)))
        rest.append(np.sqrt(np.mean(np.abs(C - np.eye(m.n, N) * C) ** 2)))
    a, b = float(np.mean(overlap)), float(np.mean(rest))
    print(f"{name} M={M}: overlaps {a:.2e}, bound {2 * 62 * 2.0 ** -53 * b:.2e}", flush=True)
    assert a <= 2 * 62 * 2.0 ** -53 * b


@pytest.mark.parametrize("M,N", [(15, 8), (54, 23), (200, 100)])
@pytest.mark.parametrize("scale", [0.0, 2.0 ** -60, 2.0 ** 120, 2.0 ** -104])
def test_mixed_orbitals_keep_their_scale(M, N, scale):
    """The same of the mixed path, planned and queued trajectories, over the
    range of FP32: bit by bit, and at 2^-104, where the smallest elements leave
    the range, within 2^-45 of an orbital's norm and the tolerance of a step."""
    cfg = make_cfg("c2", M=M, N=N)
    m = models.from_config(cfg, M=M)
    states = random_states(m, N, 3, seed=5 + M, xs=[-2.0, 3.0, 1.0], v_scale=2e-3)
    states[2].v[0] = 0.05
    from paper_2212_00518_amd import unpack_C
    out = []
    for f in (1.0, scale):
        ens = ensemble(cfg, 3, precision="mixed", lowdin_every=0)
        for s in states:
            s.C = s.C.astype(np.complex64).astype(np.complex128)
            s.C[:, ::3] *= f
        upload(ens, states)
        ens.step()
        C = ens.get_state()[2]
        out.append([unpack_C(C, t, m.n, N, ens.n_max, ens.N_max) for t in range(3)])
        ens.close()
    for t in range(3):
        if scale == 2.0 ** -104:
            got = out[1][t].copy()
            got[:, ::3] /= scale
            assert np.max(np.abs(got - out[0][t])) <= (1e-6 if t < 2 else 4e-6)
        else:
            want = out[0][t].copy()
            want[:, ::3] *= scale
            assert np.array_equal(out[1][t], want)


# every shape of work-group, with an orbital tile that is partly empty
@pytest.mark.parametrize("M,N", [(111, 41), (130, 20), (200, 100), (320, 60)])
@pytest.mark.parametrize("scale", [2.0 ** 600, 2.0 ** -600])
def test_fp64_orbitals_whose_squares_leave_the_range(M, N, scale):
    """Scaled orbitals and the others beside them, within 1e-12 of their norm
    of the unscaled ones' result."""
    cfg = make_cfg("c2", M=M, N=N)
    m = models.from_config(cfg, M=M)
    states = random_states(m, N, 2, seed=5 + M, xs=[-2.0, 3.0], v_scale=2e-3)
    from paper_2212_00518_amd import unpack_C
    out = []
    for f in (1.0, scale):
        ens = ensemble(cfg, 2)
        for s in states:
            s.C[:, ::3] *= f
        upload(ens, states)
        ens.step()
        C = ens.get_state()[2]
        out.append([unpack_C(C, t, m.n, N, ens.n_max, ens.N_max) for t in range(2)])
        ens.close()
    for t in range(2):
        got = out[1][t].copy()
        got[:, ::3] /= scale
        assert np.max(np.abs(got - out[0][t])) <= 1e-12


@pytest.mark.parametrize("precision,M,N,tiles,groups", [
    ("mixed", 200, 100, 7, 2), ("mixed", 320, 160, 4, 5), ("mixed", 40, 20, 3, 1),
    ("fp64", 200, 100, 2, 7), ("fp64", 130, 20, 1, 3), ("fp64", 320, 160, 1, 20)])
def test_class_info_names_the_running_shape(precision, M, N, tiles, groups):
    """Work-groups of one trajectory's ceil(N / 8) orbital tiles: the
    interaction picture's waves with a tile each (at most 8, beyond 13 row
    tiles 4), the digit kernel's one or two tiles."""
    ens = ensemble(make_cfg("c2", M=M, N=N), 4, precision=precision)
    info = ens.class_info(0)
    ens.close()
    assert (info["tiles_per_group"], info["groups_per_traj"]) == (tiles, groups), info
