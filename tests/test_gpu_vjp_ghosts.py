"""The adjoints in contexts with four ghost layers (which WENO5 and CU6 take
too): rows longer than a wave's 64 faces, several short rows in one wave, and
no x axis.

The faces, their stencils and the order of a cell's sums are those of three
layers, so the cotangents have to agree with the three-layer context's to the
rounding of the sums (1e-13 of a field's largest) in both precisions, and the
fourth layer has to stay zero; FP64 also against the oracle's complex step on
four layers (the bar of tests/test_gpu_vjp.py, 1e-12 of the sum of absolute
terms).
"""
import numpy as np
import pytest

import oracle as O
from conftest import oracle_objects
from paper_2403_05910_amd import workloads as W
from test_gpu_vjp import vjp_dot_check

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

MASSES = [2.0, 32.0, 18.0, 28.0, 40.0, 16.0, 17.0, 34.0, 33.0]
CASES = [((64, 1, 1), 1, "WENO5"), ((256, 4, 1), 2, "WENO5"), ((4, 9, 5), 9, "WENO5"), ((70, 5, 4), 3, "CU6"),
         ((13, 21, 1), 5, "CU6"), ((1, 9, 17), 4, "WENO5")]


def _case(n, ns):
    return W.random_smooth_state(W.sampled_table(MASSES[:ns], 1), n, seed=sum(n), jump=n[0] > 1, bc=(1, 1, 0, 0, 1, 1))


def _adjoints(case, precision, recon, seed):
    """(rhs_vjp, rk3_step_vjp) of cotangents drawn on the interior"""
    from paper_2403_05910_amd import xf
    th, g = oracle_objects(case)
    U0 = O.fill_ghosts(g, case.U)
    dt = 0.3 * O.cfl_dt(th, g, U0, 0.5)
    ctx = xf.Context.from_case(case, precision).set_reconstruction(recon)
    sel = ctx.interior
    bar = np.zeros_like(U0)
    size = np.abs(U0[sel]).reshape(len(U0), -1).max(axis=1).reshape(-1, 1, 1, 1)
    bar[sel] = np.random.default_rng(seed).standard_normal(bar[sel].shape) / np.where(size > 0, size, 1.0)
    U, rb = ctx.state_from_numpy(U0), ctx.state_from_numpy(bar)
    out = [ctx.rhs_vjp(U, rb).cpu().numpy(), ctx.rk3_step_vjp(U, dt, rb.clone()).cpu().numpy()]
    assert ctx.status() == 0
    ctx.close()
    return out


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n,ns,recon", CASES)
def test_four_layers_give_the_adjoints_of_three(n, ns, recon, precision):
    case = _case(n, ns)
    three, four = (_adjoints(c, precision, recon, sum(n)) for c in (case, case.with_ghosts(4)))
    inner = (slice(None),) + tuple(slice(1, -1) if k > 1 else slice(None) for k in n[::-1])
    for a, b in zip(three, four):
        size = np.abs(a).reshape(len(a), -1).max(axis=1).reshape(-1, 1, 1, 1)
        assert np.all(np.abs(b[inner] - a) <= 1e-13 * size)
        b[inner] = 0.0
        assert not b.any()


@pytest.mark.parametrize("n,ns,recon", CASES)
def test_four_layer_vjp_against_complex_step(n, ns, recon):
    got, ref, mag = vjp_dot_check(_case(n, ns).with_ghosts(4), "fp64", 3, recon=recon)
    assert abs(got - ref) <= 1e-12 * mag
