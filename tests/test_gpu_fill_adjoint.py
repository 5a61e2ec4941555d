"""The adjoint of the ghost fill against the fill itself, entry by entry: the
oracle's fill of a field of cell numbers says which interior cell every ghost
copies, and each cell's cotangent is the sum over its copies.  Every mix of
periodic and outflow axes (z is folded by itself where two axes have outflow
sides), one to three active axes, three and four layers, axes as short as the
layers, more and fewer fields than a thread takes.

Tolerance: a cell adds at most 125 values, 1e-13 of the sum of their sizes.
"""
import itertools

import numpy as np
import pytest

import oracle as O
from conftest import oracle_objects
from paper_2403_05910_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

MASSES = [2.0, 32.0, 18.0, 28.0, 40.0, 16.0, 17.0, 34.0, 33.0]


@pytest.mark.parametrize("ng", [3, 4])
@pytest.mark.parametrize("n,ns", [((4, 5, 6), 1), ((9, 4, 7), 4), ((4, 70, 11), 9), ((13, 8, 1), 2), ((1, 4, 19), 3),
                                  ((1, 1, 5), 5)])
def test_fill_adjoint_entry_by_entry(n, ns, ng):
    from paper_2403_05910_amd import xf
    for kinds in itertools.product((0, 1), repeat=sum(k > 1 for k in n)):
        per_axis = iter(kinds)
        bc = sum(((b, b) for b in (next(per_axis) if k > 1 else 0 for k in n)), ())
        case = W.random_smooth_state(W.sampled_table(MASSES[:ns], 1), n, seed=1, bc=bc).with_ghosts(ng)
        _, g = oracle_objects(case)
        shape = case.U.shape
        number = np.arange(np.prod(shape[1:]), dtype=float).reshape((1,) + shape[1:])
        source = O.fill_ghosts(g, np.broadcast_to(number, shape).copy())[0].astype(int).ravel()
        bar = np.random.default_rng(sum(n)).standard_normal(shape)
        ctx = xf.Context.from_case(case)
        got = ctx.fill_ghosts_vjp(ctx.state_from_numpy(bar)).cpu().numpy()
        ctx.close()
        for q in range(shape[0]):
            want, size = np.zeros(source.size), np.zeros(source.size)
            np.add.at(want, source, bar[q].ravel())
            np.add.at(size, source, np.abs(bar[q]).ravel())
            assert np.all(np.abs(got[q].ravel() - want) <= 1e-13 * size), (bc, q)
