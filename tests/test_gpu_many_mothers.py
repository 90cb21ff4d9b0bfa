"""More copies of a mother than one launch of the list form takes (their scratch is bounded): copies
without kicks come out alike."""
import numpy as np
import pytest

import ttcf_inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    from paper_2312_02990_amd import ttcf
    ttcf.lib()
    return ttcf


def test_copies_over_several_launches(T):
    n, copies = 2048, 1030
    print(f"{copies} copies of n={n}", flush=True)
    edge = (n / 0.8442) ** (1.0 / 3.0)
    r = np.mod(I.fcc_lattice(8, edge) + np.random.Generator(np.random.PCG64(3)).uniform(-0.04, 0.04, (3, n)), edge)
    p = I.maxwell_boltzmann(n, 0.722, 4)
    with T.Context() as ctx:
        mid = ctx.ttcf_init_mother(T.make_system(n, edge, 0.722, 0.0025), r, p, n_equil=0)
        ctx.ttcf_sample_states_replicated(mid, copies, None, 0, 1, 5)
        gr, gp = ctx.ttcf_export_states(mid, copies)
    assert np.abs(gp[0] - p.ravel()).max() > 0.0
    np.testing.assert_array_equal(gr, np.broadcast_to(gr[0], gr.shape))
    np.testing.assert_array_equal(gp, np.broadcast_to(gp[0], gp.shape))
