"""Pair-list daughters in a batch that leaves waves of the chip free (which share their force pass
and list build) and in one that fills it, where every wave owns atoms: the same bits, with the pair
words in LDS for all waves, for the owners' waves alone, and in global scratch."""
import numpy as np
import pytest

import ttcf_inputs as I

pytestmark = pytest.mark.gpu

DT, TEMP, STEPS = 0.0025, 0.722, 60


@pytest.fixture(scope="module")
def T():
    from paper_2312_02990_amd import ttcf
    ttcf.lib()
    return ttcf


@pytest.mark.parametrize("nh", [False, True])
@pytest.mark.parametrize("n,copies,shape", [
    (130, 520, None),                                   # one wave and three spare ones
    (300, 260, None),                                   # two and six
    (864, 130, None),                                   # four and four, which list nothing
    (600, 130, dict(variant=2, skin=0.2, kmax=64)),     # pair words in global scratch
])
def test_spare_waves_change_nothing(T, n, copies, shape, nh):
    print(f"spare waves n={n} copies={copies} nh={nh}", flush=True)
    m = int(np.ceil((n / 4.0) ** (1.0 / 3.0) - 1e-9))
    edge = (n / 0.8442) ** (1.0 / 3.0)
    rng = np.random.Generator(np.random.PCG64(n))
    sites = I.fcc_lattice(m, edge)
    r = np.mod(sites[:, np.sort(rng.permutation(4 * m ** 3)[:n])] + rng.uniform(-0.04, 0.04, (3, n)), edge)
    p = I.maxwell_boltzmann(n, TEMP, n + 1)
    sysd = T.make_system(n, edge, TEMP, DT, precision=T.TTCF_PREC_FP32_FORCES,
                         thermostat=T.TTCF_DAUGHTER_NH if nh else T.TTCF_DAUGHTER_GIK)
    out = []
    for count in (1, copies):
        with T.Context() as ctx:
            mid = ctx.ttcf_init_mother(sysd, r, p, n_equil=0)
            if shape:
                ctx.ttcf_set_step_shape(**shape)
            ctx.ttcf_import_states(mid, np.repeat(r.reshape(1, -1), count, 0),
                                   np.repeat(p.reshape(1, -1), count, 0))
            first = ctx.ttcf_spawn_daughters(mid, count, 0, 0.3, STEPS)
            ctx.ttcf_step(STEPS)
            out.append(ctx.ttcf_export_series(first, 4 * count, STEPS + 1))
            assert ctx.ttcf_accumulate() == count
    assert np.isfinite(out[0]).all()
    np.testing.assert_array_equal(out[1].reshape(copies, 4, -1),
                                  np.broadcast_to(out[0], (copies, 4, STEPS + 1)))
