"""Mothers of 513 to 1088 atoms with FP32 forces advanced by one step a call run in the cell form, whose
start costs less than the lists': the same bits as a system that asks for it, also for copies."""
import numpy as np
import pytest

import ttcf_inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    from paper_2312_02990_amd import ttcf
    ttcf.lib()
    return ttcf


@pytest.mark.parametrize("copies", [0, 3])
@pytest.mark.parametrize("n,threads", [(513, 576), (640, 640), (1025, 1024), (1088, 1024)])
def test_one_step_is_the_cell_forms(T, n, threads, copies):
    print(f"short mother n={n} copies={copies}", flush=True)
    edge = (n / 0.8442) ** (1.0 / 3.0)
    rng = np.random.Generator(np.random.PCG64(n))
    sites = I.fcc_lattice(int(np.ceil((n / 4.0) ** (1.0 / 3.0) - 1e-9)), edge)
    r = np.mod(sites[:, np.sort(rng.permutation(sites.shape[1])[:n])] + rng.uniform(-0.04, 0.04, (3, n)), edge)
    p = I.maxwell_boltzmann(n, 0.722, n + 1)
    out = []
    for t in (0, threads):
        with T.Context() as ctx:
            mid = ctx.ttcf_init_mother(T.make_system(n, edge, 0.722, 0.0025, block_threads=t), r, p, n_equil=0)
            for _ in range(4):
                if copies:
                    ctx.ttcf_sample_states_replicated(mid, copies, None, 0, 1, 1)
                else:
                    ctx.ttcf_sample_states(mid, 1, 1)
            out.append(np.concatenate(ctx.ttcf_export_states(mid, max(copies, 1))))
    np.testing.assert_array_equal(out[0], out[1])
