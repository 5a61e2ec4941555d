"""The CFL step of an RK3 step on either side of the size up to which the
primitive pass's last block divides (8192 padded cells), with one block, a
block and a cell, and 32 blocks, over steps on a changing state, and with the
GLF speeds in the same buffer: against the separate reduction (the same
maximum; 1e-14 for a division by a value that may round differently) and the
oracle's step (1e-12, the bar of the forward quantities).
"""
import pytest

import oracle as O
from conftest import oracle_objects
from paper_2403_05910_amd import workloads as W

pytestmark = pytest.mark.gpu
pytest.importorskip("torch")


@pytest.mark.parametrize("visc", ["LLF", "GLF"])
@pytest.mark.parametrize("n,precision", [
    ((250, 1, 1), "fp64"), ((251, 1, 1), "mixed"), ((8186, 1, 1), "fp64"), ((8187, 1, 1), "fp64"),
    ((90, 79, 1), "mixed"), ((13, 14, 15), "fp64")])
def test_step_size_of_a_cfl_step(n, precision, visc):
    from paper_2403_05910_amd import xf
    case = W.random_smooth_state(W.sampled_table([2.0, 32.0], 1), n, seed=sum(n), jump=True, bc=(1, 1, 0, 0, 1, 1))
    th, g = oracle_objects(case)
    U0 = O.fill_ghosts(g, case.U)
    ctx = xf.Context.from_case(case, precision).set_dissipation(visc)
    U = ctx.state_from_numpy(U0)
    ctx.fill_ghosts(U)
    for k in range(3):
        want = ctx.cfl_dt(U, 0.4).item()
        got = ctx.rk3_step_cfl(U, 0.4).item()
        assert abs(got - want) <= 1e-14 * want
        if k == 0:
            assert abs(got - O.cfl_dt(th, g, U0, 0.4)) <= 1e-12 * want
    assert ctx.status() == 0
    ctx.close()
