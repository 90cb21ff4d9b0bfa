"""Exports of many rows in one call equal the same rows one at a time: whole series, prefixes of
them, ranges over two batches of different lengths and with a gap, extra observables, stored
states of the bulk and the channel."""
import numpy as np
import pytest

import ttcf_inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    from paper_2312_02990_amd import ttcf
    ttcf.lib()
    return ttcf


def liquid(s, count, seed):
    r = np.stack([I.perturbed_positions(s, seed + k, 0.05).ravel() for k in range(count)])
    p = np.stack([I.maxwell_boltzmann(s.n, s.temperature, seed + 50 + k).ravel() for k in range(count)])
    return r, p


def test_series_ranges_and_states(T):
    s = I.System(4)
    r, p = liquid(s, 3, 7)
    with T.Context() as ctx:
        mid = ctx.ttcf_init_mother(T.make_system(s.n, s.box, s.temperature, s.dt), r[0], p[0], n_equil=0)
        ctx.ttcf_import_states(mid, r, p)
        er, ep = ctx.ttcf_export_states(mid, 3)
        np.testing.assert_array_equal(er, r)
        np.testing.assert_array_equal(ep, p)
        np.testing.assert_array_equal(ctx.ttcf_export_states(mid, 1)[0], r[:1])
        ctx.ttcf_record_observables(True)
        first = ctx.ttcf_spawn_daughters(mid, 3, 0, 0.1, 6)
        ctx.ttcf_spawn_daughters(mid, 3, 0, 0.2, 9, mapping_mask=0b0101)  # 6 daughters
        ctx.ttcf_step(9)
        for lo, hi in ((0, 18), (0, 12), (12, 18), (5, 16), (11, 13)):
            for n_t in (1, 3, 7):
                one = [ctx.ttcf_export_series(first + d, 1, n_t)[0] for d in range(lo, hi)]
                np.testing.assert_array_equal(ctx.ttcf_export_series(first + lo, hi - lo, n_t), one)
                one = [ctx.ttcf_export_observables(first + d, 1, n_t)[0] for d in range(lo, hi)]
                np.testing.assert_array_equal(ctx.ttcf_export_observables(first + lo, hi - lo, n_t), one)
        for bad in ((first, 19, 3), (first - 1, 2, 3), (first, 18, 8)):
            with pytest.raises(T.TTCFError):
                ctx.ttcf_export_series(*bad)


def test_channel_rows(T):
    g = I.ChannelSystem(n_x=7, n_z=10, n_fluid=420)
    r0, p0, lat = I.channel_initial_state(g, 3)
    rng = np.random.Generator(np.random.PCG64(4))
    r = np.stack([r0.ravel()] * 3)
    p = p0.ravel() * rng.uniform(0.9, 1.1, (3, 1))
    z = np.array([0.1, -0.2, 0.3])
    with T.ChannelContext(T.make_channel(g), r0, p0, lat) as ctx:
        ctx.import_states(r, p, z)
        for got, want in zip(ctx.export_states(3), (r, p, z)):
            np.testing.assert_array_equal(got, want)
        first = ctx.spawn(3, 0.1, 4)
        ctx.spawn(2, 0.2, 6, mapping_mask=0b0010)
        ctx.step(6)
        for lo, hi in ((0, 14), (0, 12), (10, 13)):
            for n_t in (1, 5):
                obs, s0 = ctx.export_series(first + lo, hi - lo, n_t)
                one = [ctx.export_series(first + d, 1, n_t) for d in range(lo, hi)]
                np.testing.assert_array_equal(obs, [o[0][0] for o in one])
                np.testing.assert_array_equal(s0, [o[1][0] for o in one])
