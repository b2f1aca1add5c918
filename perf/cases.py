"""The work users have this library do, as measurable cases.

Every case goes through the public Python entry points (``Ensemble`` and the
functions of the package): an ensemble is created once with its inputs on the
GPU (``prepare``), and a pass (``run``) advances it and reads back what such a
program reads: observable records, hop events, status words and, for small
ensembles, the whole state.  Sizes are those of the repository's workloads
(M = 20 parity ensemble, M = 200 ensembles, four bath classes of scattering,
two-lead junction, dense Hamiltonian, adjoint, batched eigen-solves) and odd
ones between them.

A mixed-precision ensemble holds its orbitals in 32 bits, so what depends on
them (orbitals, P_d^wf, hop probabilities) is returned in 32 bits there; the
nuclear coordinates and energies are 64-bit on both paths.
"""
from __future__ import annotations

import math

import numpy as np

import paper_2212_00518_amd as iesh
from paper_2212_00518_amd.adjoint import path_loss

EV = 1.0 / 27.211386245988
ANGSTROM = 1.0 / 0.529177210903
AMU = 1822.888486209

HARMONIC = dict(kind="harmonic", mass=2000.0, omega=2e-4, g=20.0, dG=-3.8e-3, Gamma=0.01, eps_d=0.0)
MORSE = dict(kind="morse_tanh", De=0.1, x0=1.78 * ANGSTROM, a=1.0, D1=4.52 * EV, D2=0.79 * EV,
             ap=1.379 / ANGSTROM, Vinf=-1.5 * EV, q=0.05, atil=0.5 * ANGSTROM, xtil=3.5 * ANGSTROM,
             mass=10.54 * AMU, c=-45.7e-3 * EV, Gamma=1.0 * EV, eps_d=0.0)
MULTI_DOF = dict(kind="multi_dof", Gamma=0.01, Delta=0.005, eps_d=0.0,
                 dof=[[2000.0, 0.10, 1.0, 3.0, -0.004, 3.0, 1.5], [2000.0, 0.15, 1.2, 2.0, 0.002, 2.0, 2.0],
                      [4000.0, 0.08, 0.8, 0.0, 0.001, 0.0, 2.5], [4000.0, 0.08, 0.8, 0.0, -0.001, 0.0, 2.5],
                      [8000.0, 0.05, 0.6, 0.0, 0.0005, 0.0, 3.0], [8000.0, 0.05, 0.6, 0.0, -0.0005, 0.0, 3.0]])
DENSE = dict(kind="dense", mass=2000.0, omega=2e-4, g=20.0, dG=-3.8e-3, Gamma=0.01, t_bath=2.0e-4,
             alpha=0.02, x_c=0.0)
MODELS = dict(harmonic=HARMONIC, morse_tanh=MORSE, multi_dof=MULTI_DOF, dense=DENSE)
KT = 9.5e-4
LOWDIN_EVERY = 100


def _dynamics(name, model, bath, M, N, T, precision, steps, record, dt, width, kT=KT, start="thermal", leads=1,
              bias=0.0, state=False, classes="", compact=0, substeps=1, dt_levels=0):
    case = dict(path="dynamics", model=model, bath=bath, M=M, N=N, T=T, precision=precision, steps=steps,
                record=record, dt=dt, width=width, kT=kT, start=start, leads=leads, bias=bias, state=state,
                classes=classes, compact=compact, substeps=substeps, dt_levels=dt_levels)
    return dict(case, name=name) if name else case


def listed():
    return [
        # One step of a handful of trajectories and the state read back: interactive use,
        # a coupling to another integrator.  Launches and host work only.
        _dynamics("single_step_tiny", "harmonic", "trapezoid", 20, 10, 4, "fp64", 1, 0, 50.0, 0.1, state=True),
        # The small parity ensemble in FP64 with its records, as a relaxation study runs it.
        _dynamics("small_fp64", "harmonic", "trapezoid", 20, 10, 128, "fp64", 200, 20, 50.0, 0.1, state=True),
        # An odd-sized ensemble: odd M, N and trajectory count, state read back for a checkpoint.
        _dynamics("ragged_mixed", "harmonic", "gauss_legendre", 54, 23, 333, "mixed", 40, 10, 20.0, 0.1,
                  start="mixed", state=True),
        # The M = 200 production ensemble on the mixed path: the throughput workload.
        _dynamics("ensemble_mixed", "harmonic", "trapezoid", 200, 100, 4096, "mixed", 20, 10, 20.0, 0.1),
        # The same physics in FP64 (reference runs), half as many trajectories.
        _dynamics("ensemble_fp64", "harmonic", "trapezoid", 200, 100, 2048, "fp64", 10, 5, 20.0, 0.1),
        # Gauss-Legendre bath with mixed orbitals from the start: the determinant ratios are
        # evaluated for most trajectories, as late in a run on this bath.
        _dynamics("gauss_legendre_mixed", "harmonic", "gauss_legendre", 200, 100, 768, "mixed", 20, 10, 20.0, 0.1,
                  start="mixed"),
        # Scattering off the surface: four bath sizes in one context, compaction on the device.
        _dynamics("scattering_mixed", "morse_tanh", "gauss_legendre", 320, 160, 2048, "mixed", 10, 10, 5.0,
                  64.0 * EV, kT=0.0, classes="40,80,160,320", compact=5),
        # Biased two-lead junction with six coordinates (n = 257).
        _dynamics("two_lead_mixed", "multi_dof", "trapezoid", 256, 128, 1536, "mixed", 20, 10, 20.0, 0.1, leads=2,
                  bias=0.01),
        # A one-electron Hamiltonian of general structure (n = 96).
        _dynamics("dense_mixed", "dense", "cells", 95, 48, 2048, "mixed", 20, 10, 20.0, 0.1),
        # Training through prescribed paths: losses and their gradient, FP64.
        dict(name="adjoint", path="adjoint", M=100, N=50, T=512, steps=40, ckpt=20, dt=20.0),
        # Batches of dense symmetric eigenproblems beyond the LDS-resident order.
        dict(name="eigh_batch", path="eigh", n=201, batch=128),
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["dynamics"] * 8 + ["adjoint", "eigh"])
    if kind == "eigh":
        n = size(4, 230)
        return dict(path="eigh", n=n, batch=max(1, min(size(1, 512), int(1.2e9 / n ** 3))))
    if kind == "adjoint":
        M = size(6, 120)
        N = max(1, int(M * rng.uniform(0.3, 0.6)))
        steps = rng.randint(3, 40)
        T = max(1, min(size(4, 512), int(4.0e9 / (steps * (M + 20) ** 2 * (N + 8)))))
        return dict(path="adjoint", M=M, N=N, T=T, steps=steps, ckpt=rng.randint(2, 25), dt=20.0)
    model = rng.choice(["harmonic", "harmonic", "morse_tanh", "multi_dof", "dense"])
    precision = rng.choice(["mixed", "mixed", "fp64"])
    leads = 2 if model == "multi_dof" and rng.random() < 0.5 else 1
    M = size(6, 94 if model == "dense" else 320)
    bath = "cells" if model == "dense" else rng.choice(["trapezoid", "gauss_legendre"])
    M += M % 2 if model != "dense" else 0
    M += 2 * (M % 4 != 0) if leads == 2 else 0
    N = max(1, min(168, int(M * rng.uniform(0.3, 0.6))))
    steps = rng.randint(2, 20)
    cost = steps * (M + 12) ** 2 * (N + 8) * (4.0 if precision == "fp64" else 1.0)
    T = max(1, min(size(2, 4096), int(2.0e11 / cost)))
    start = "mixed" if T * M * N < 3e6 and rng.random() < 0.5 else "thermal"
    wide = model == "morse_tanh"
    return _dynamics("", model, bath, M, N, T, precision, steps, max(1, steps // 2), 5.0 if wide else 20.0,
                     64.0 * EV if wide else 0.1, kT=0.0 if wide else KT, start=start, leads=leads,
                     bias=0.01 if leads == 2 and rng.random() < 0.5 else 0.0, state=T * M * N < 3e6,
                     compact=rng.choice([0, 0, 2]), substeps=rng.choice([1, 1, 1, 2]),
                     dt_levels=rng.choice([0, 0, 0, 3]))


# ------------------------------------------------------------------------------------ inputs
def _dense_matrices(M, width):
    m = DENSE
    eps = -0.5 * width + (np.arange(M) + 0.5) * (width / M)
    V = np.full(M, math.sqrt(m["Gamma"] * (width / M) / (2.0 * math.pi)))
    k = m["mass"] * m["omega"] ** 2
    H0 = np.zeros((M + 1, M + 1))
    H1 = np.zeros((M + 1, M + 1))
    H0[0, 0] = 0.5 * k * m["g"] ** 2 + m["dG"]
    H0[0, 1:] = H0[1:, 0] = V
    H0[1:, 1:] = np.diag(eps)
    i = np.arange(1, M)
    H0[i, i + 1] = H0[i + 1, i] = m["t_bath"]
    H1[0, 0] = -k * m["g"]
    H1[0, 1:] = H1[1:, 0] = m["alpha"] * V
    return H0, H1


def _nuclei(case, rng):
    """Positions and velocities of the case's trajectories."""
    T, model = case["T"], case["model"]
    if model == "multi_dof":
        dof = np.array(MULTI_DOF["dof"])
        mass, omega = dof[:, 0], dof[:, 2] * np.sqrt(2.0 * dof[:, 1] / dof[:, 0])
        x = dof[:, 3] + rng.normal(size=(T, len(dof))) * np.sqrt(KT / (mass * omega * omega))
        return x, rng.normal(size=(T, len(dof))) * np.sqrt(KT / mass)
    if model == "morse_tanh":  # on the way to the surface
        x = rng.uniform(3.0, 5.0 * ANGSTROM, size=T)
        return x, -np.sqrt(2.0 * rng.uniform(0.05 * EV, 1.0 * EV, size=T) / MORSE["mass"])
    m = MODELS[model]
    x = rng.normal(0.0, math.sqrt(KT / (m["mass"] * m["omega"] ** 2)), size=T)
    return x, rng.normal(0.0, math.sqrt(KT / m["mass"]), size=T)


def _mixed_orbitals(n, N, rng):
    """N orthonormal orbitals: unit vectors of the lowest states, some of them
    near the Fermi level rotated into states above it with random phases."""
    C = np.zeros((N, n), dtype=np.complex128)
    C[np.arange(N), np.arange(N)] = 1.0
    p = min(8, N, n - N)
    low = N - 1 - rng.permutation(p)
    high = N + rng.permutation(p)
    th, ph = rng.uniform(0.1, 0.7, size=p), rng.uniform(0.0, 2.0 * math.pi, size=p)
    C[low, low] = np.cos(th)
    C[low, high] = np.sin(th) * np.exp(1j * ph)
    return C


def _inputs(case, seed):
    rng = np.random.default_rng([seed, 7])
    x, v = _nuclei(case, rng)
    C = None
    if case["start"] == "mixed":
        C = np.stack([_mixed_orbitals(case["M"] + 1, case["N"], rng) for _ in range(case["T"])])
    cls = None
    if case["classes"]:
        cls = rng.integers(0, len(case["classes"].split(",")), size=case["T"]).astype(np.int32)
    return x, v, C, cls


def _class_sizes(case):
    if not case["classes"]:
        return [(case["M"], case["N"])]
    return [(int(m), int(m) // 2) for m in case["classes"].split(",")]


def _paths(case, seed):
    rng = np.random.default_rng([seed, 11])
    T, t = case["T"], np.arange(case["steps"] + 1) * case["dt"]
    x0, v0 = rng.normal(0.0, 3.0, T), 0.1 * rng.normal(0.0, 7e-4, T)
    amp, phi = rng.uniform(0.0, 3.0, T), rng.uniform(0.0, 2.0 * math.pi, T)
    return x0[:, None] + v0[:, None] * t + amp[:, None] * np.sin(HARMONIC["omega"] * t + phi[:, None])


TERMS = (1.0, 1.0, 1.0, 1.0)


def _theta(case):
    eps, w = iesh.discretize("trapezoid", case["M"], 0.1)
    m = HARMONIC
    return np.concatenate([[m["eps_d"], m["Gamma"]], eps, [m["omega"], m["g"], m["dG"]]]), w


def prepare(case, seed):
    if case["path"] == "eigh":
        rng = np.random.default_rng([seed, 3])
        a = rng.normal(size=(case["batch"], case["n"], case["n"]))
        return dict(case=case, H=0.5 * (a + a.transpose(0, 2, 1)))
    if case["path"] == "adjoint":
        import torch
        theta, w = _theta(case)
        return dict(case=case, theta=torch.tensor(theta, requires_grad=True), w=w, paths=_paths(case, seed))
    x, v, C, cls = _inputs(case, seed)
    descs = []
    for M, N in _class_sizes(case):
        if case["model"] == "dense":
            from paper_2212_00518_amd._lib import dense_model_desc
            H0, H1 = _dense_matrices(M, case["width"])
            descs.append(dense_model_desc(H0, H1, DENSE["mass"], DENSE["omega"], N, DENSE["x_c"]))
        else:
            b = dict(kind=case["bath"], W=case["width"], leads=case["leads"])
            eps, w, lead, _ = iesh.bath_levels(b, M)
            descs.append(iesh.model_desc(MODELS[case["model"]], eps, w, N, lead))
    mixed = case["precision"] == "mixed"
    run = dict(n_traj=case["T"], precision=case["precision"], dt=case["dt"], kT=case["kT"], seed=seed,
               bias=case["bias"], lowdin_every=LOWDIN_EVERY if mixed else 0, record_every=case["record"],
               compact_every=case["compact"], elec_substeps=case["substeps"], dt_levels=case["dt_levels"],
               hop_gmax=1e-3 if case["dt_levels"] else 0.0)
    if case["model"] == "morse_tanh":
        run.update(exit_enabled=1, exit_x=15.0, max_steps=20000)
    ens = iesh.Ensemble(descs, run, traj_model=cls)
    if C is None:
        ens.init_thermal(x, v)
    else:
        occ = np.tile(np.arange(case["N"], dtype=np.int32), (case["T"], 1))
        ens.set_state(x, v, C, occ)
    return dict(case=case, ens=ens)


# ---------------------------------------------------------------------------------- one pass
def _head(case):
    """Leading trajectories whose records are returned on their own (those
    that the plain 64-bit evaluation covers)."""
    n = max(m for m, _ in _class_sizes(case)) + 1
    cost = case["steps"] * (2 + case["substeps"]) * (2e-4 + 9e-10 * n ** 3 + 6e-7 * n ** 2)
    return max(1, min(case["T"], int(6.0 / cost), 128))


def run(state):
    case = state["case"]
    if case["path"] == "eigh":
        lam, Q, sweeps = iesh.eigh_batched(state["H"])
        return dict(lam=lam, Q=Q, sweeps=sweeps)
    if case["path"] == "adjoint":
        theta = state["theta"]
        theta.grad = None
        loss = path_loss(theta, state["paths"], state["w"], HARMONIC["mass"], case["N"], case["dt"], case["ckpt"],
                         TERMS)
        loss.sum().backward()
        return dict(loss=loss.detach(), grad=theta.grad.clone())
    ens, T, h = state["ens"], case["T"], _head(case)
    real, cplx = (np.float32, np.complex64) if case["precision"] == "mixed" else (np.float64, np.complex128)
    obs = ens.run(case["steps"], record=case["record"] > 0)
    events, _ = ens.events()
    ens.clear_events()
    hops = np.zeros((T, 5), dtype=np.int64)  # per trajectory: hop attempts, and the last one
    for e in events:
        hops[e["traj"]] = hops[e["traj"], 0] + 1, e["step"], e["a"], e["b"], e["accepted"]
    out = dict(status=ens.status(), hops=hops)
    if obs is not None:
        for part, o in (("head", obs[:, :h]), ("rest", obs[:, h:])):
            out["nuclear_" + part] = np.ascontiguousarray(o[..., [0, 2, 3, 4]])
            out["pd_wf_" + part] = o[..., 1].astype(real)
    if case["state"]:
        x, v, C, occ = ens.get_state()
        C = C.reshape(T, -1).astype(cplx)
        out.update(x_head=x[:h], v_head=v[:h], C_head=C[:h], occ=occ, x_rest=x[h:], v_rest=v[h:], C_rest=C[h:])
    return out


def work(case):
    if case["path"] == "eigh":  # matrices in, vectors out; reduction and back-transformation
        n, b = case["n"], case["batch"]
        return dict(bytes=8.0 * b * (2 * n * n + n), flops=9.0 * b * n ** 3)
    if case["path"] == "adjoint":  # forward, recomputed and reverse propagation, contraction
        n, N, ts = case["M"] + 1, case["N"], case["T"] * case["steps"]
        return dict(bytes=8.0 * (ts + case["T"]), flops=4.0 * 8.0 * ts * n * n * N)
    total_b = total_f = 0.0
    sizes = _class_sizes(case)
    ts = case["T"] * case["steps"] / len(sizes)
    size = 8 if case["precision"] == "mixed" else 16
    for M, N in sizes:
        n = M + 1
        # orbitals in and out, and an n x n propagator applied to them
        total_b += ts * 2.0 * size * n * N
        total_f += ts * (8.0 * n * n * N * case["substeps"] + (9.0 * 2 * n ** 3 if case["model"] == "dense" else 40.0 * n * n))
    return dict(bytes=total_b, flops=total_f)


# ------------------------------------------------------------- plain evaluation in 64 bits
def _bath_levels(kind, M, width, leads):
    G = M // leads
    if kind == "gauss_legendre":
        t, w = np.polynomial.legendre.leggauss(G // 2)
        half = width / 4.0
        eps = np.concatenate([half * t - half, half * t + half])
        w = np.concatenate([half * w, half * w])
    else:
        eps = -0.5 * width + np.arange(G) * (width / G)
        w = np.full(G, width / G)
    if leads == 2:
        return np.repeat(eps, 2), np.repeat(0.5 * w, 2), np.tile([0, 1], G)
    return eps, w, None


class _Model:
    """U0, its gradient, H and dH/dR of one model."""

    def __init__(self, case, M):
        self.kind, self.m = case["model"], MODELS[case["model"]]
        self.lead = None
        if self.kind == "dense":
            self.H0, self.H1 = _dense_matrices(M, case["width"])
        else:
            self.eps, w, self.lead = _bath_levels(case["bath"], M, case["width"], case["leads"])
            self.V = np.sqrt(self.m["Gamma"] * w / (2.0 * math.pi))
        self.dof = np.array(MULTI_DOF["dof"]).T if self.kind == "multi_dof" else None
        self.mass = self.dof[0] if self.dof is not None else np.array([self.m["mass"]])

    def _scalars(self, x):
        """U0, dU0, h, dh, f, df (gradients per coordinate)."""
        m = self.m
        if self.kind == "multi_dof":
            _, D, a, r, g, c, s = self.dof
            e = np.exp(-a * (x - r))
            f = math.exp(-np.sum((x - c) ** 2 / (4.0 * s * s)))
            return (np.sum(D * (1 - e) ** 2), 2 * D * a * e * (1 - e), m["Delta"] + m["eps_d"] + np.sum(g * (x - r)),
                    g, f, -f * (x - c) / (2 * s * s))
        if self.kind == "morse_tanh":
            e, e1 = np.exp(-m["a"] * (x - m["x0"])), np.exp(-m["ap"] * (x - m["x0"]))
            U0, dU0 = m["De"] * (e - 1) ** 2 + m["c"], -2 * m["De"] * m["a"] * e * (e - 1)
            U1 = m["D1"] * e1 * e1 - m["D2"] * e1 + m["Vinf"]
            dU1 = -2 * m["ap"] * m["D1"] * e1 * e1 + m["ap"] * m["D2"] * e1
            t = np.tanh((x - m["xtil"]) / m["atil"])
            f = 0.5 * (1 - m["q"]) * (1 - t) + m["q"]
            return U0[0], dU0, (U1 - U0)[0] + m["eps_d"], dU1 - dU0, f[0], -0.5 * (1 - m["q"]) * (1 - t * t) / m["atil"]
        k = m["mass"] * m["omega"] ** 2
        U0, dU0 = 0.5 * k * x[0] ** 2, k * x
        if self.kind == "dense":
            return U0, dU0, 0.0, np.zeros(1), 1.0, np.zeros(1)
        return U0, dU0, 0.5 * k * (x[0] - m["g"]) ** 2 + m["dG"] - U0 + m["eps_d"], np.array([-k * m["g"]]), 1.0, np.zeros(1)

    def at(self, x):
        """lam, q0, Q, U0, dU0, G_nu = Q^T dH_nu Q at x."""
        U0, dU0, h, dh, f, df = self._scalars(x)
        if self.kind == "dense":
            H = self.H0 + x[0] * self.H1
        else:
            H = np.diag(np.concatenate([[h], self.eps]))
            H[0, 1:] = H[1:, 0] = self.V * f
        lam, Q = np.linalg.eigh(H)
        first = np.argmax(np.abs(Q) > 0, axis=0)
        Q = Q * np.where(Q[first, np.arange(len(lam))] < 0, -1.0, 1.0)
        if self.kind == "dense":
            return lam, Q, U0, dU0, [Q.T @ self.H1 @ Q]
        z = self.V @ Q[1:]
        q = Q[0]
        return lam, Q, U0, dU0, [a * np.outer(q, q) + b * (np.outer(q, z) + np.outer(z, q)) for a, b in zip(dh, df)]


def _coupling(lam, Gs, v):
    gap = lam[None, :] - lam[:, None]
    off = np.abs(gap) > 1e-12 * np.max(np.abs(lam))
    G = sum(a * g for a, g in zip(v, Gs))
    return np.where(off, G / np.where(off, gap, 1.0), 0.0)


def _philox(counter, traj, stream, seed):
    """Uniforms in [0, 1) for an array of counters (Philox4x32-10)."""
    c = np.asarray(counter, dtype=np.uint64)
    m32, sh = np.uint64(0xFFFFFFFF), np.uint64(32)
    c0, c1 = c & m32, c >> sh
    c2, c3 = np.full_like(c, traj), np.full_like(c, stream)
    k0, k1 = seed & 0xFFFFFFFF, seed >> 32
    for r in range(10):
        if r:
            k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
        p0, p1 = np.uint64(0xD2511F53) * c0, np.uint64(0xCD9E8D57) * c2
        c0, c1, c2, c3 = (p1 >> sh) ^ c1 ^ np.uint64(k0), p1 & m32, (p0 >> sh) ^ c3 ^ np.uint64(k1), p0 & m32
    return (((c1 << sh) | c0) >> np.uint64(11)).astype(np.float64) / 9007199254740992.0


def _thermal(model, lam, Q, N, kT, bias, seed, traj):
    n = len(lam)
    if kT <= 0.0:
        return np.arange(N)

    def filling(mu):
        fermi = lambda s: 0.5 * (1.0 - np.tanh(0.5 * (lam - mu - s) / kT))  # noqa: E731
        if bias == 0.0:
            return fermi(0.0)
        q2, w0 = Q[0] ** 2, np.sum(Q[1:][model.lead == 0] ** 2, axis=0)
        return q2 * fermi(0.0) + w0 * fermi(0.5 * bias) + (1.0 - q2 - w0) * fermi(-0.5 * bias)

    lo, hi = lam[0] - 1.0 - 50 * kT - abs(bias), lam[-1] + 1.0 + 50 * kT + abs(bias)
    for _ in range(200):
        mu = 0.5 * (lo + hi)
        lo, hi = (lo, mu) if filling(mu).sum() > N else (mu, hi)
    p = filling(0.5 * (lo + hi))
    for t0 in range(0, 4096, 64):
        u = _philox(np.arange(t0 * n, (t0 + 64) * n), traj, 1, seed).reshape(64, n) < p
        hit = np.flatnonzero(u.sum(axis=1) == N)
        if len(hit):
            return np.flatnonzero(u[hit[0]])
    return np.arange(N)


def _select(g, xi):
    cum = 0.0
    for r, total in enumerate(np.cumsum(g, axis=1)[:, -1]):
        if cum + total > xi:
            inside = cum + np.cumsum(g[r])
            hit = np.flatnonzero((inside > xi) & (g[r] > 0))
            return r, int(hit[0]) if len(hit) else int(np.flatnonzero(g[r] > 0)[-1])
        cum += total
    return None


def _trajectory(case, model, N, x, v, C, traj, seed):
    """Records, final x, v, C (N x n) of one trajectory."""
    x, v, m, S = np.atleast_1d(x).copy(), np.atleast_1d(v).copy(), model.mass, case["substeps"]
    lam, Q, U0, dU0, G = model.at(x)
    if C is None:
        s = _thermal(model, lam, Q, N, case["kT"], case["bias"], seed, traj)
        C = np.zeros((len(lam), N), dtype=np.complex128)
        C[s, np.arange(N)] = 1.0
    else:
        s, C = np.arange(N), C.T.copy()
    dt, rec = case["dt"], []
    force = lambda: -np.asarray(dU0) - np.array([np.sum(np.diag(g)[s]) for g in G])  # noqa: E731
    F = force()
    for k in range(case["steps"]):
        vh = v + 0.5 * dt * F / m
        xn = x + dt * vh
        for j in range(S):
            lm, _, _, _, Gm = model.at(x + ((j + 0.5) / S) * (xn - x))
            mu, P = np.linalg.eigh(np.diag(lm) - 1j * _coupling(lm, Gm, vh))
            C = P @ (np.exp(-1j * mu * dt / S)[:, None] * (P.conj().T @ C))
        x = xn
        lam, Q, U0, dU0, G = model.at(x)
        F = force()
        v = vh + 0.5 * dt * F / m
        W = np.linalg.solve(C[s].T, C.T).T
        g = np.maximum(-2.0 * dt * _coupling(lam, G, v)[:, s] * W.real, 0.0).T
        g[:, s] = 0.0
        pick = _select(g, _philox([k], traj, 0, seed)[0])
        if pick is not None:
            a, b = s[pick[0]], pick[1]
            d = np.array([_coupling(lam, [gn], [1.0])[b, a] for gn in G])
            A, B, dE = np.sum(d * d / (2 * m)), np.sum(v * d), lam[b] - lam[a]
            disc = B * B - 4 * A * dE
            if A != 0.0 and disc >= 0.0:
                q = B + math.copysign(math.sqrt(disc), B)
                v = v - (2 * dE / q if q else 0.0) * d / m
                s = np.sort(np.append(np.delete(s, pick[0]), b))
                F = force()
        if case["dt_levels"]:
            total, now = g.sum(), dt
            dt = case["dt"]
            for _ in range(case["dt_levels"]):
                dt = 0.5 * dt if total * (dt / now) > 1e-3 else dt
        if case["record"] and (k + 1) % case["record"] == 0:
            kin, pot = 0.5 * np.sum(m * v * v), U0 + np.sum(lam[s])
            rec.append((np.sum(Q[0, s] ** 2), np.sum(np.abs(Q[0] @ C) ** 2), kin, pot, kin + pot))
    return np.array(rec), x, v, C.T


def _exact_adjoint(case, seed):
    import torch
    theta, w = _theta(case)
    n, N, T, dt = case["M"] + 1, case["N"], case["T"], case["dt"]
    if T * case["steps"] * n ** 3 > 4e8:
        return None
    th, w, path = torch.tensor(theta, requires_grad=True), torch.tensor(w), torch.tensor(_paths(case, seed))
    eps_d, Gamma, eps = th[0], th[1], th[2:1 + n]
    omega, g, dG = th[1 + n], th[2 + n], th[3 + n]
    k = HARMONIC["mass"] * omega ** 2
    V, hp, eye = torch.sqrt(Gamma * w / (2 * math.pi)), -k * g, torch.eye(n, dtype=torch.float64)

    def at(x):  # lam, q0 of a batch of positions
        h = 0.5 * k * (g * g - 2 * g * x) + dG + eps_d
        H = torch.diag(torch.cat([torch.zeros(1, dtype=torch.float64), eps])).repeat(T, 1, 1)
        e0 = torch.zeros(n, dtype=torch.float64)
        e0[0] = 1.0
        Vf = torch.cat([torch.zeros(1, dtype=torch.float64), V])
        H = H + h[:, None, None] * torch.outer(e0, e0) + torch.outer(e0, Vf) + torch.outer(Vf, e0)
        lam, Q = torch.linalg.eigh(H)
        return lam, Q[:, 0, :] * torch.sign(Q[:, 0, :]).detach()

    def coupling(lam, q):
        gap = lam[:, None, :] - lam[:, :, None] + eye
        return hp * q[:, :, None] * q[:, None, :] / gap * (1 - eye)

    steps = case["steps"]
    C = torch.eye(n, dtype=torch.complex128)[:, :N].repeat(T, 1, 1)
    loss = torch.zeros(T, dtype=torch.float64)
    for t in range(steps):
        v = (path[:, t + 1] - path[:, t]) / dt
        lam, q = at(0.5 * (path[:, t] + path[:, t + 1]))
        A = torch.diag_embed(lam) - 1j * v[:, None, None] * coupling(lam, q)
        C = torch.matrix_exp(-1j * dt * A) @ C
        x = path[:, t + 1]
        lam, q = at(x)
        P = torch.sum(torch.abs(torch.sum(q[:, :, None] * C, dim=1)) ** 2, dim=1)
        W = C[:, N:] @ torch.linalg.inv(C[:, :N])
        G = torch.clamp(-2 * dt * v[:, None, None] * coupling(lam, q)[:, N:, :N] * W.real, min=0.0).sum(dim=(1, 2))
        F = -k * x - hp * torch.sum(q[:, :N] ** 2, dim=1)
        loss = loss + (TERMS[0] * P + TERMS[2] * G + TERMS[3] * F) / steps
    rho = torch.sum(torch.abs(C) ** 2, dim=2)
    n0 = (torch.arange(n) < N).to(torch.float64)
    loss = loss + TERMS[1] * torch.sum(lam * (rho - n0), dim=1)
    loss.sum().backward()
    return dict(loss=loss.detach(), grad=th.grad)


def exact(case, seed):
    if case["path"] == "eigh":
        H = prepare(case, seed)["H"]
        lam, Q = np.linalg.eigh(H)
        big = np.abs(Q) > 1e-12 * np.max(np.abs(Q), axis=1, keepdims=True)
        first = np.take_along_axis(Q, np.argmax(big, axis=1)[:, None, :], axis=1)
        return dict(lam=lam, Q=Q * np.where(first < 0, -1.0, 1.0), sweeps=None)
    if case["path"] == "adjoint":
        return _exact_adjoint(case, seed)
    x, v, C, cls = _inputs(case, seed)
    sizes = _class_sizes(case)
    models = [_Model(case, M) for M, _ in sizes]
    n_max, N_max = max(M for M, _ in sizes) + 1, max(N for _, N in sizes)
    h = _head(case)
    rec, xs, vs, Cs = [], [], [], np.zeros((h, n_max * N_max), dtype=np.complex128)
    for t in range(h):
        k = 0 if cls is None else int(cls[t])
        r, xt, vt, Ct = _trajectory(case, models[k], sizes[k][1], x[t], v[t], None if C is None else C[t], t, seed)
        rec.append(r)
        xs.append(xt)
        vs.append(vt)
        Cs[t, :Ct.size] = Ct.reshape(-1)
    out = dict(status=None, hops=None)
    if case["record"]:
        rec = np.stack(rec, axis=1)
        out.update(nuclear_head=np.ascontiguousarray(rec[..., [0, 2, 3, 4]]), pd_wf_head=rec[..., 1])
    if case["state"]:
        nuc = (lambda a: np.array(a)) if case["model"] == "multi_dof" else (lambda a: np.array(a)[:, 0])
        out.update(x_head=nuc(xs), v_head=nuc(vs), C_head=Cs)
    return out
