"""The no-hop bound over its splits, with records.

A target's sum over the occupied states is split into one to eight parts by the
number of unoccupied states, which may also take two turns of the work-group.
The bound is exact: with it and with the ratios at every step the states and
the hop events are bit-identical.  Observables are sums of at most 336 FP64
terms in either kernel's own order: 336 x 2^-52 < 1e-13 of the largest term, and
the amplitudes' moduli are at most one.
"""
import numpy as np
import pytest

from oracle import dynamics as dyn, models
from test_gpu_parity import ensemble, gpu, make_cfg, random_states, upload  # noqa: F401

pytestmark = pytest.mark.gpu


# unoccupied states: 1, 8, 32 and 33, 64 and 65, 128 and 129, 257 and more
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("M,N", [(1, 1), (15, 8), (40, 9), (40, 8), (83, 20), (84, 20), (160, 33), (160, 32),
                                 (276, 20), (335, 12), (335, 168)])
def test_bound_and_ratios_agree_over_the_splits(M, N, precision):
    cfg = make_cfg("c2", M=M, N=N)
    m = models.from_config(cfg, M=M)
    T = 6
    states = random_states(m, N, T, seed=M + N, xs=np.linspace(-8.0, 24.0, T), v_scale=1e-2)
    for t in range(1, T, 2):  # the bound rules out most steps
        states[t] = dyn.State(states[t].x, states[t].v, np.eye(m.n, N, dtype=np.complex128), np.arange(N))
    out = []
    for off in (0, 1):
        ens = ensemble(cfg, T, precision=precision, hop_filter_off=off, record_every=3)
        upload(ens, states)
        obs = ens.run(10, record=True)
        out.append((ens.get_state(), [(e["step"], e["traj"], e["a"], e["b"], e["accepted"]) for e in ens.events()[0]],
                    ens.hop_evals(), obs))
        ens.close()
    (s0, e0, h0, o0), (s1, e1, h1, o1) = out
    assert all(np.array_equal(a, b) for a, b in zip(s0, s1)) and e0 == e1
    assert h0 < h1 == 10 * T
    assert o0.shape[0] == 3 and np.all(np.isfinite(o0))
    assert np.all(np.abs(o0 - o1) <= 1e-13 * max(1.0, np.abs(o1).max()))
