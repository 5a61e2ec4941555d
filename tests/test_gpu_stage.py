"""The RK3 stage as the last sweep finishes it, over every set of active axes:
x last, y or z last (no x axis), a lone sweep with no other direction to add,
at sizes around one wave, one tile and one x-sweep block, for species counts
with an even and an odd end of the species loop; with the fluxes exchanged
across lanes (WENO5) and held in LDS (CU6).

Tolerances: FP64, 1e-12 of a field's largest value or of dt times the flux
scale (the residual's bar), whichever is larger; mixed, the declared 1e-5 of a
field's largest value.
"""
import numpy as np
import pytest

import oracle as O
from conftest import oracle_objects
from paper_2403_05910_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

MASSES = [2.0, 32.0, 18.0, 28.0, 40.0, 16.0, 17.0, 34.0, 33.0]


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n,ns,recon", [
    ((64, 1, 1), 1, "WENO5"), ((513, 1, 1), 2, "WENO5"), ((1, 33, 1), 2, "WENO5"), ((1, 1, 62), 3, "WENO5"),
    ((1, 32, 5), 4, "WENO5"), ((9, 1, 31), 5, "WENO5"), ((65, 8, 1), 9, "WENO5"), ((3, 9, 7), 8, "WENO5"),
    ((17, 31, 4), 9, "WENO5"), ((1, 17, 6), 3, "CU6"), ((19, 5, 16), 2, "CU6")])
def test_stage_finish_matches_oracle(n, ns, recon, precision):
    from paper_2403_05910_amd import xf
    tab = W.sampled_table(MASSES[:ns], 1)
    case = W.random_smooth_state(tab, n, seed=sum(n), jump=n[0] > 1, bc=(1, 1, 0, 0, 1, 1))
    th, g = oracle_objects(case)
    U0 = O.fill_ghosts(g, case.U)
    dt = O.cfl_dt(th, g, U0, 0.4)
    ref = U0
    for _ in range(2):
        ref = O.rk3_step(th, g, ref, dt, recon=recon)
    _, aux = O.rhs(th, g, U0, return_aux=True, recon=recon)
    ctx = xf.Context.from_case(case, precision).set_reconstruction(recon)
    U = ctx.state_from_numpy(U0)
    for _ in range(2):
        ctx.rk3_step(U, dt)
    assert ctx.status() == 0
    got = U.cpu().numpy()
    ctx.close()
    nv = ref.shape[0]
    err = np.abs(got - ref).reshape(nv, -1).max(axis=1)
    size = np.abs(ref).reshape(nv, -1).max(axis=1)
    tol = 1e-12 * np.maximum(size, dt * aux["scale_llf"]) if precision == "fp64" else \
        1e-5 * np.maximum(size, dt * aux["scale_llf"])
    assert np.all(err <= tol), (err / np.maximum(tol, 1e-300))
