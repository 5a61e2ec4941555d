"""RK3 steps whose last sweep finishes the stage together with what else goes
into it: the viscous fluxes (added into the directions' sum in FP64 contexts,
a buffer of their own in mixed ones), the positivity blend, and both; over the
sets of active axes, with one and two species in mixed contexts (a stage kernel
of their own) and more (the sweep).  The oracle's steps are the reference.

Tolerances, per field of the larger of its largest value and dt times its flux
scale (convective or viscous): 1e-12 in FP64 and 1e-5 mixed, the bars of
tests/test_gpu_stage.py; with the blend at sharp interfaces, whose theta is
ill-conditioned, 20 times the change of the oracle's own result under a random
relative perturbation of the initial state by the rounding of the arithmetic
(1e-15, mixed 6e-8) where that is larger, and 1e-4 mixed at least, as
tests/test_gpu_positivity.py has it.  What the terms change is checked to be a
hundred times the tolerance; the blend moves a state by less than FP32 resolves,
so for mixed blended steps that is the whole step, whose sum of directions they
are about.
"""
import numpy as np
import pytest

import oracle as O
from conftest import oracle_objects
from paper_2403_05910_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
V = O.xf_viscous

MASSES = [2.0, 32.0, 18.0, 28.0, 40.0, 16.0, 17.0, 34.0, 33.0]
STEPS = 2


def smooth(n, ns):
    return W.random_smooth_state(W.sampled_table(MASSES[:ns], 1), n, seed=sum(n), jump=n[0] > 1, bc=(1, 1, 0, 0, 1, 1))


def slabs(n, ns):
    """wavy slabs of one gas each with sharp interfaces, advected through a
    periodic box (the flow of workloads.species_slab, with more gases)"""
    tab = W.perfect_gas_table([1.4, 1.667, 1.3, 1.4, 1.5][:ns], [28.96, 4.003, 44.0, 2.016, 18.0][:ns])
    X, Y, Z = np.meshgrid(*((np.arange(k) + 0.5) / k if k > 1 else np.zeros(1) for k in n), indexing="ij")
    axes = [a for a, k in zip((X, Y, Z), n) if k > 1]
    place = axes[0] + sum(w * np.sin(2 * np.pi * a) for w, a in zip((0.1, 0.07), axes[1:]))
    gas = (np.floor(ns * place) % ns).transpose(2, 1, 0)
    frac = np.stack([np.where(gas == s, 1.0, 0.0) for s in range(ns)])
    T = np.full(gas.shape, 1e-3)
    vel = np.stack([np.full(gas.shape, v if n[k] > 1 else 0.0) for k, v in enumerate((1.0, 0.5, 0.25))])
    interior = W.assemble(tab, 1.0 / (W.mixture_R(tab, frac) * T), vel, T, frac)
    U = np.zeros((ns + 4,) + tuple(k + 6 if k > 1 else 1 for k in n[::-1]))
    U[(slice(None),) + tuple(slice(3, -3) if k > 1 else slice(None) for k in n[::-1])] = interior
    return W.Case("slabs", n, tuple(1.0 / k for k in n), (0,) * 6, tab, U)


def transport(ns, boost):
    t = W.sampled_transport(ns, 0)
    mu, kappa, D = t.mu.copy(), t.kappa.copy(), t.D.copy()
    for c in (mu, kappa, D):
        c[..., 0] += np.log(boost)
    return W.TransportTable(mu, kappa, D, t.p_ref)


def oracle_steps(case, dt, pp, tab, perturb=0.0):
    th, g = oracle_objects(case)
    U = O.fill_ghosts(g, case.U)
    if perturb:
        U = O.fill_ghosts(g, U * (1.0 + perturb * np.random.default_rng(7).standard_normal(U.shape)))
    tr = None if tab is None else V.Transport(tab.mu, tab.kappa, tab.D, tab.p_ref)
    for _ in range(STEPS):
        U = O.rk3_step(th, g, U, dt, pp=pp, transport=tr)
    return U


def reference(case, precision, pp, viscous):
    """dt, transport table, state after the steps, tolerance per field, and the
    state without the terms (mixed and blended: without the steps)"""
    th, g = oracle_objects(case)
    U0 = O.fill_ghosts(g, case.U)
    dt = 0.4 * O.cfl_dt(th, g, U0, 0.5)
    nv = len(U0)
    _, aux = O.rhs(th, g, U0, return_aux=True)
    scale, tab = aux["scale_llf"], None
    if viscous:
        tab = transport(case.thermo.ns, 3e4)
        scale = np.maximum(scale, V.viscous_rhs(th, V.Transport(tab.mu, tab.kappa, tab.D, tab.p_ref), g, U0,
                                                return_aux=True)[1]["scale"])
    want = oracle_steps(case, dt, pp, tab)
    size = np.maximum(np.abs(want).reshape(nv, -1).max(axis=1), dt * scale)
    bar = 1e-12 if precision == "fp64" else 1e-4 if pp else 1e-5
    tol = np.full(nv, bar)
    if pp:
        moved = oracle_steps(case, dt, pp, tab, 1e-15 if precision == "fp64" else 6e-8)
        change = np.abs(moved - want).reshape(nv, -1).max(axis=1) / np.where(size > 0, size, 1.0)
        tol = np.maximum(tol, 20.0 * change.max())
    without = U0 if pp and precision == "mixed" else oracle_steps(case, dt, False, None)
    return dt, tab, want, tol * size, without


STEPS_OF = [
    # mixed, viscous: the separate stage (one and two species) and the sweep's
    ("mixed", smooth, (33, 6, 5), 2, False, True), ("mixed", smooth, (17, 9, 8), 5, False, True),
    ("mixed", smooth, (1, 33, 6), 1, False, True), ("mixed", smooth, (1, 9, 33), 4, False, True),
    ("mixed", smooth, (1, 1, 70), 3, False, True),
    # mixed, blended, x last and y or z last
    ("mixed", slabs, (48, 10, 1), 3, True, False), ("mixed", smooth, (24, 8, 6), 5, True, False),
    ("mixed", smooth, (1, 48, 7), 4, True, False), ("mixed", slabs, (1, 1, 60), 3, True, False),
    ("mixed", slabs, (1, 40, 5), 2, True, False),
    # FP64, viscous, one active axis: the sum starts from zero
    ("fp64", smooth, (70, 1, 1), 2, False, True), ("fp64", smooth, (1, 64, 1), 3, False, True),
    ("fp64", smooth, (1, 1, 33), 9, False, True), ("fp64", smooth, (1, 17, 6), 4, False, True),
    # FP64, blended
    ("fp64", slabs, (1, 1, 60), 3, True, False), ("fp64", slabs, (1, 36, 5), 5, True, False),
]


@pytest.mark.parametrize("precision,make,n,ns,pp,viscous", STEPS_OF)
def test_stage_with_its_terms_matches_oracle(precision, make, n, ns, pp, viscous):
    from paper_2403_05910_amd import xf
    case = make(n, ns)
    dt, tab, want, tol, without = reference(case, precision, pp, viscous)
    nv = len(want)
    assert np.any(np.abs(want - without).reshape(nv, -1).max(axis=1) > 100.0 * tol)
    ctx = xf.Context.from_case(case, precision).set_positivity(pp)
    if viscous:
        ctx.set_viscous(tab)
    U = ctx.state_from_numpy(case.U)
    for _ in range(STEPS):
        ctx.rk3_step(U, dt)
    # the FP32 blend's floor is -1e-6 rho, so a mixed blended step may flag mass
    # fractions below -1e-12
    assert ctx.status() & ~(O.FLAG_Y if pp and precision == "mixed" else 0) == 0
    got = U.cpu().numpy()
    ctx.close()
    err = np.abs(got - want).reshape(nv, -1).max(axis=1)
    assert np.all(err <= tol), err / np.maximum(tol, 1e-300)
