"""The viscous fluxes at the edges of their blocks, against the oracle within
tests/test_gpu_viscous.py's bar (1e-12 of each field's flux-divergence scale):
250 cells a block along linearised x rows, 26 cells and 16 columns a tile in y
and z, one more and one less; a single cell past a tile; odd and even species
counts, and one set of terms without the species' stage.
"""
import pytest

from paper_2403_05910_amd import workloads as W
from test_gpu_parity import field_err
from test_gpu_viscous import gpu_rhs, oracle_rhs, table

pytestmark = pytest.mark.gpu
pytest.importorskip("torch")

MASSES = [2.0, 32.0, 18.0, 28.0, 40.0, 16.0, 17.0, 34.0, 33.0]


@pytest.mark.parametrize("n,ns,terms", [
    ((250, 1, 1), 1, "all"), ((251, 1, 1), 9, "all"), ((3, 26, 1), 2, "all"), ((1, 27, 4), 3, "all"),
    ((16, 25, 26), 4, "all"), ((17, 4, 27), 9, "all"), ((5, 53, 3), 5, "all"), ((33, 6, 5), 6, "no_diffusion")])
def test_viscous_block_edges(n, ns, terms):
    import oracle as O
    V = O.xf_viscous
    case = W.random_smooth_state(W.sampled_table(MASSES[:ns], 1), n, seed=sum(n), jump=n[0] > 1, bc=(1, 1, 0, 0, 1, 1))
    tab = table(case, boost=1e7)
    some = terms != "all"
    got, flags = gpu_rhs(case, tab, ("stress", "heat") if some else ("stress", "heat", "diffusion"))
    assert flags == 0
    rc, rv, scale, _, _ = oracle_rhs(case, tab, V.STRESS | V.HEAT if some else V.ALL_TERMS)
    err = field_err(got, rc + rv, scale)
    assert err.max() <= 1e-12, err
