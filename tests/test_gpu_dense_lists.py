"""Clustered systems in the list forms: a ball of atoms so dense that its middle has more partners than
any list holds (looked up in the grid) and its outer part more than a list has room for in LDS (the
rest in global memory), against the oracle. Lists are rebuilt several times over the run."""
import numpy as np
import pytest

import ttcf_inputs as I

pytestmark = pytest.mark.gpu

DT, TEMP, TAU, STEPS = 0.0025, 0.722, 0.25, 30
N, RC, DENSITY = 600, 2.5, 0.08


@pytest.fixture(scope="module")
def T():
    from paper_2312_02990_amd import ttcf
    ttcf.lib()
    return ttcf


def ball():
    """The N sites of an fcc lattice of spacing 1.4 nearest the box's corner, jittered: the stencils of
    its atoms wrap in every direction."""
    edge = (N / DENSITY) ** (1.0 / 3.0)
    sites = I.fcc_lattice(int(round(edge / 1.4)), edge)
    d = sites - edge * np.rint(sites / edge)
    keep = np.sort(np.argsort((d * d).sum(0), kind="stable")[:N])
    rng = np.random.Generator(np.random.PCG64(11))
    r = np.mod(sites[:, keep] + rng.uniform(-0.02, 0.02, (3, N)), edge)
    return np.ascontiguousarray(r), I.maxwell_boltzmann(N, TEMP, 12), edge


def neighbours(r, edge, reach):
    d = r[:, :, None] - r[:, None, :]
    d -= edge * np.rint(d / edge)
    return ((d * d).sum(0) < reach * reach).sum(0) - 1


def test_ball_has_lists_of_every_kind():
    r, _, edge = ball()
    near = neighbours(r, edge, 1.15 * RC)
    assert near.max() > 128 and ((near > 24) & (near <= 128)).sum() > 100
    assert 1.5 * 4.18879 * (1.15 * RC) ** 3 * DENSITY <= 24


@pytest.mark.parametrize("copies", [1, 70])  # one atom per thread, four
@pytest.mark.parametrize("nh", [False, True])
def test_shear_daughters(T, orc, nh, copies):
    print(f"dense ball, shear nh={nh} copies={copies}", flush=True)
    r, p, edge = ball()
    box = orc.make_box(N, edge, rc=RC)
    zeta0, nf = 0.4, 3 * N - 3
    q = orc.nh_q(nf, TEMP, TAU)
    one, maps, rate = np.zeros(4, np.int32), np.arange(4, dtype=np.int32), np.full(4, 0.6)
    sr, sp, sz = r.reshape(1, -1), p.reshape(1, -1), np.array([zeta0])
    if nh:
        want = orc.run_daughters_nh(box, sr, sp, sz, one, maps, rate, DT, TEMP, q, nf, STEPS, nthreads=4)[0]
    else:
        want = orc.run_daughters(box, sr, sp, one, maps, rate, DT, STEPS, nthreads=4)[0]
    sysd = T.make_system(N, edge, TEMP, DT, r_cut=RC, precision=T.TTCF_PREC_FP64, potential=T.TTCF_LJ,
                         thermostat=T.TTCF_DAUGHTER_NH if nh else T.TTCF_DAUGHTER_GIK)
    with T.Context() as ctx:
        mid = ctx.ttcf_init_mother(sysd, r, p, n_equil=0)
        ctx.ttcf_import_states(mid, np.repeat(sr, copies, 0), np.repeat(sp, copies, 0))
        ctx.ttcf_import_states_zeta(mid, np.full(copies, zeta0))
        first = ctx.ttcf_spawn_daughters(mid, copies, 0, 0.6, STEPS)
        ctx.ttcf_step(STEPS)
        got = ctx.ttcf_export_series(first, 4 * copies, STEPS + 1)
        assert ctx.ttcf_accumulate() == copies
    # FP64 on both sides: roundings of 1e-16 grow less than a thousandfold over 30 steps
    assert np.abs(got[:4] - want).max() <= 1e-9 * np.std(want)
    np.testing.assert_array_equal(got.reshape(copies, 4, -1), np.broadcast_to(got[:4], (copies, 4, STEPS + 1)))


@pytest.mark.parametrize("flow", ["elong", "mixed"])
def test_carried_flows_are_refused(T, flow):
    """More than 24 partners within the cutoff: carried-flow daughters fail their health check."""
    print(f"dense ball, {flow}", flush=True)
    r, p, edge = ball()
    sysd = T.make_system(N, edge, TEMP, DT, r_cut=RC, precision=T.TTCF_PREC_FP64, potential=T.TTCF_LJ)
    with T.Context() as ctx:
        mid = ctx.ttcf_init_mother(sysd, r, p, n_equil=0)
        ctx.ttcf_import_states(mid, r.reshape(1, -1), p.reshape(1, -1))
        if flow == "mixed":
            first = ctx.ttcf_spawn_mixed(mid, 1, 0, 0.05, 0.1, 5)
        else:
            first = ctx.ttcf_spawn_elongational(mid, 1, 0, 0.1, 5)
        ctx.ttcf_step(5)
        assert all(ctx.ttcf_daughter_health(first + d) != 0 for d in range(4))


@pytest.mark.parametrize("precision,tol", [(0, 1e-9), (1, 1e-4)])
def test_mother(T, orc, precision, tol):
    print(f"dense ball, mother precision={precision}", flush=True)
    r, p, edge = ball()
    with T.Context() as ctx:
        sysd = T.make_system(N, edge, TEMP, DT, r_cut=RC, precision=precision, nh_tau=TAU, potential=T.TTCF_LJ)
        mid = ctx.ttcf_init_mother(sysd, r, p, n_equil=7)
        ctx.ttcf_sample_states(mid, 2, 12)
        gr, gp = ctx.ttcf_export_states(mid, 2)
        gz = ctx.ttcf_export_states_zeta(mid, 2)
    nf = 3 * N - 3
    st = orc.NHState(r.ravel().copy(), p.ravel().copy())
    wr, wp, wz = orc.mother_sample(orc.make_box(N, edge, rc=RC), st, 7, 2, 12, TEMP, DT,
                                   orc.nh_q(nf, TEMP, TAU), nf, with_zeta=True)
    dr = gr - wr
    dr -= edge * np.rint(dr / edge)
    assert np.abs(dr).max() / edge <= tol
    assert np.abs(gp - wp).max() / np.sqrt(np.mean(wp ** 2)) <= tol
    np.testing.assert_allclose(gz, wz, rtol=100 * tol, atol=100 * tol)
