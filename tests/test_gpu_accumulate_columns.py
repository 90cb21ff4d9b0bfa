"""Accumulation of the extra observables' columns (64 time points at a time) against the definition
on the GPU's own series, around one and two blocks of points: D(t), the mapping mean, and
D(0) - V gamma / T times the trapezoid integral of P_xy(0) B(s)."""
import numpy as np
import pytest

import ttcf_inputs as I

pytestmark = pytest.mark.gpu

DT, TEMP, RATE, N = 0.0025, 0.722, 0.02, 130


@pytest.fixture(scope="module")
def T():
    from paper_2312_02990_amd import ttcf
    ttcf.lib()
    return ttcf


@pytest.mark.parametrize("steps", [1, 62, 63, 64, 130])
def test_columns_match_the_definition(T, steps):
    print(f"accumulate columns, {steps} steps", flush=True)
    edge = (N / 0.8442) ** (1.0 / 3.0)
    rng = np.random.Generator(np.random.PCG64(5))
    sites = I.fcc_lattice(4, edge)
    r = np.stack([np.mod(sites[:, np.sort(rng.permutation(256)[:N])] + rng.uniform(-0.03, 0.03, (3, N)),
                         edge).ravel() for _ in range(3)])
    p = np.stack([I.maxwell_boltzmann(N, TEMP, 7 + k).ravel() for k in range(3)])
    with T.Context() as ctx:
        mid = ctx.ttcf_init_mother(T.make_system(N, edge, TEMP, DT, precision=T.TTCF_PREC_FP32_FORCES),
                                   r[0], p[0], n_equil=0)
        ctx.ttcf_import_states(mid, r, p)
        ctx.ttcf_record_observables(True)
        first = ctx.ttcf_spawn_daughters(mid, 3, 0, RATE, steps)
        ctx.ttcf_step(steps)
        ser = ctx.ttcf_export_series(first, 12, steps + 1)
        obs = ctx.ttcf_export_observables(first, 12, steps + 1)
        assert ctx.ttcf_accumulate() == 3
        got = {c: ctx.ttcf_response(steps + 1, RATE, observable=o)
               for c, o in ((0, T.TTCF_OBS_N1), (1, T.TTCF_OBS_N2), (2, T.TTCF_OBS_ENERGY))}
    pxy0 = ser[:, :1] / edge ** 3
    for c, (mean, _, direct, _, used) in got.items():
        b = obs[:, :, c]
        integral = np.concatenate([np.zeros((12, 1)),
                                   np.cumsum(0.5 * DT * pxy0 * (b[:, 1:] + b[:, :-1]), axis=1)], axis=1)
        want = b[:, :1] - edge ** 3 * RATE / TEMP * integral
        scale = np.abs(want).max()
        assert used == 3
        # sums of at most 131 terms in FP64
        assert np.abs(np.ravel(direct) - b.mean(axis=0)).max() <= 1e-13 * scale
        assert np.abs(np.ravel(mean) - want.mean(axis=0)).max() <= 1e-12 * scale
