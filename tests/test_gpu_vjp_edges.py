"""The face VJP at the edges of its blocks: 64 faces a wave in x and runs of
several rows in one wave, eight faces a block and 16 columns in y and z, a lone
face past a block, odd and even species counts; FP64 against the oracle's
complex step (the bar of tests/test_gpu_vjp.py, 1e-12 of the sum of absolute
terms), mixed at its declared 2e-4, and values large enough to take the
reconstruction's guarded branch.
"""
import numpy as np
import pytest

import oracle as O
from conftest import oracle_objects
from paper_2403_05910_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

MASSES = [2.0, 32.0, 18.0, 28.0, 40.0, 16.0, 17.0, 34.0, 33.0]


def _rel(case, precision, recon, seed=5):
    from paper_2403_05910_amd import xf
    th, g = oracle_objects(case)
    rng = np.random.default_rng(seed)
    U0 = O.fill_ghosts(g, case.U)
    _, aux = O.rhs(th, g, U0, return_aux=True, recon=recon)
    sel = (slice(None),) + g.interior()
    rbar, w = np.zeros_like(U0), np.zeros_like(U0)
    sc = np.where(aux["scale_llf"] > 0, aux["scale_llf"], 1.0).reshape(-1, 1, 1, 1)
    fs = np.abs(U0[sel]).reshape(len(U0), -1).max(axis=1).reshape(-1, 1, 1, 1)
    rbar[sel] = rng.standard_normal(rbar[sel].shape) / sc
    w[sel] = rng.standard_normal(w[sel].shape) * fs
    rc = O.rhs(th, g, O.fill_ghosts(g, U0 + 1e-30j * w), recon=recon)
    terms = rbar * rc.imag / 1e-30
    ctx = xf.Context.from_case(case, precision).set_reconstruction(recon)
    U = ctx.state_from_numpy(U0)
    Ub = ctx.rhs_vjp(U, ctx.state_from_numpy(rbar))
    ctx.fill_ghosts_vjp(Ub)
    assert ctx.status() == 0
    got = float(np.sum(Ub.cpu().numpy() * w))
    ctx.close()
    return abs(got - terms.sum()) / np.abs(terms).sum()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n,ns,recon", [
    ((63, 1, 1), 1, "WENO5"), ((64, 1, 1), 2, "WENO5"), ((1, 7, 1), 3, "WENO5"), ((1, 1, 8), 4, "WENO5"),
    ((17, 16, 1), 9, "WENO5"), ((16, 9, 7), 8, "WENO5"), ((3, 3, 15), 5, "CU6"), ((3, 24, 3), 2, "CU6")])
def test_vjp_block_edges(n, ns, recon, precision):
    case = W.random_smooth_state(W.sampled_table(MASSES[:ns], 1), n, seed=sum(n), jump=n[0] > 1, bc=(1, 1, 0, 0, 1, 1))
    assert _rel(case, precision, recon) <= (1e-12 if precision == "fp64" else 2e-4)


def test_vjp_and_residual_of_huge_values():
    """densities of 1e18 kg/m^3 or so (momenta 1e20): the products of the
    weights' denominators leave the fast branch's range"""
    case = W.random_smooth_state(W.sampled_table(MASSES[:3], 1), (20, 6, 1), seed=2, p0=1e23, jump=True)
    assert _rel(case, "fp64", "WENO5") <= 1e-12
    from paper_2403_05910_amd import xf
    th, g = oracle_objects(case)
    U0 = O.fill_ghosts(g, case.U)
    r, aux = O.rhs(th, g, U0, return_aux=True)
    ctx = xf.Context.from_case(case)
    got = ctx.rhs(ctx.state_from_numpy(U0)).cpu().numpy()
    ctx.close()
    err = np.abs(got - r).reshape(len(r), -1).max(axis=1)
    assert np.all(err <= 1e-12 * aux["scale_llf"])
