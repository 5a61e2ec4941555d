"""The step size of every CFL step against the oracle's on the state the step
starts from, over steps that change it: one to 32 blocks of the primitive pass
(whose last block divides), more (a launch divides), and a reacting context
(a pass of its own).  1e-12 relative, the bar of the forward quantities; mixed
contexts take the step size in FP64 from their own state.
"""
import numpy as np
import pytest

import oracle as O
from conftest import oracle_objects
from paper_2403_05910_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

MASSES = [2.0, 32.0, 18.0, 28.0, 40.0, 16.0, 17.0, 34.0, 33.0]


@pytest.mark.parametrize("n,ns,precision,visc", [
    ((250, 1, 1), 2, "fp64", "LLF"), ((251, 1, 1), 3, "mixed", "GLF"), ((8187, 1, 1), 1, "fp64", "GLF"),
    ((13, 14, 15), 9, "fp64", "LLF"), ((1, 90, 79), 4, "mixed", "LLF"), ((21, 1, 40), 5, "fp64", "ROE")])
def test_every_step_size_is_the_oracles(n, ns, precision, visc):
    from paper_2403_05910_amd import xf
    case = W.random_smooth_state(W.sampled_table(MASSES[:ns], 1), n, seed=sum(n), jump=n[0] > 1, bc=(1, 1, 0, 0, 1, 1))
    th, g = oracle_objects(case)
    ctx = xf.Context.from_case(case, precision).set_dissipation(visc)
    U = ctx.state_from_numpy(O.fill_ghosts(g, case.U))
    seen = []
    for _ in range(4):
        want = O.cfl_dt(th, g, U.cpu().numpy(), 0.45)
        got = ctx.rk3_step_cfl(U, 0.45).item()
        assert abs(got - want) <= 1e-12 * want
        seen.append(got)
    assert len(set(seen)) == 4 and ctx.status() == 0
    ctx.close()


def test_step_size_of_a_reacting_step():
    from paper_2403_05910_amd import xf
    tab = W.with_formation_enthalpies(W.sampled_table(W.W9, 0), 1)
    case = W.random_smooth_state(tab, (12, 10, 8), seed=3, T0=1500.0, bc=(1, 1, 0, 0, 0, 0))
    th, g = oracle_objects(case)
    ctx = xf.Context.from_case(case).set_reactions(W.synthetic_mechanism(W.W9, tab, 0, 12), 2)
    U = ctx.state_from_numpy(O.fill_ghosts(g, case.U))
    for _ in range(3):
        want = O.cfl_dt(th, g, U.cpu().numpy(), 0.3)
        assert abs(ctx.rk3_step_cfl(U, 0.3).item() - want) <= 1e-12 * want
    assert ctx.status() == 0
    ctx.close()
