"""Pair-list daughters of several sizes in one call, with the extra observables or in the colour field,
where spare waves share the work of some and not of others: the same bits as in a batch that fills the
chip. The eight-atom builds (more than 2048 atoms) of either thermostat, with observables and in the
colour field against the oracle."""
import numpy as np
import pytest

import ttcf_inputs as I

pytestmark = pytest.mark.gpu

DT, TEMP, TAU, STEPS = 0.0025, 0.722, 0.25, 40


@pytest.fixture(scope="module")
def T():
    from paper_2312_02990_amd import ttcf
    ttcf.lib()
    return ttcf


def state(n, density=0.8442):
    m = int(np.ceil((n / 4.0) ** (1.0 / 3.0) - 1e-9))
    edge = (n / density) ** (1.0 / 3.0)
    rng = np.random.Generator(np.random.PCG64(n))
    sites = I.fcc_lattice(m, edge)
    r = np.mod(sites[:, np.sort(rng.permutation(4 * m ** 3)[:n])] + rng.uniform(-0.04, 0.04, (3, n)), edge)
    return np.ascontiguousarray(r), I.maxwell_boltzmann(n, TEMP, n + 1), edge


def system(T, n, edge, nh):
    return T.make_system(n, edge, TEMP, DT, precision=T.TTCF_PREC_FP32_FORCES, nh_tau=TAU,
                         thermostat=T.TTCF_DAUGHTER_NH if nh else T.TTCF_DAUGHTER_GIK)


@pytest.mark.parametrize("nh", [False, True])
@pytest.mark.parametrize("kind", ["plain", "observables", "colour"])
def test_sizes_in_one_call(T, kind, nh):
    print(f"pair batches {kind} nh={nh}", flush=True)
    sizes = (130, 300, 864)
    out = []
    for copies in (1, 200):
        with T.Context() as ctx:
            ctx_first = []
            mids = []
            for n in sizes:
                r, p, edge = state(n)
                mids.append(ctx.ttcf_init_mother(system(T, n, edge, nh), r, p, n_equil=0))
                ctx.ttcf_import_states(mids[-1], np.repeat(r.reshape(1, -1), copies, 0),
                                       np.repeat(p.reshape(1, -1), copies, 0))
            ctx.ttcf_record_observables(kind == "observables")
            for mid in mids:
                spawn = ctx.ttcf_spawn_colour if kind == "colour" else ctx.ttcf_spawn_daughters
                ctx_first.append(spawn(mid, copies, 0, 0.3, STEPS))
            ctx.ttcf_step(STEPS)
            got = [ctx.ttcf_export_series(f, 4, STEPS + 1) for f in ctx_first]
            if kind == "observables":
                got += [ctx.ttcf_export_observables(f, 4, STEPS + 1) for f in ctx_first]
            out.append(got)
    for a, b in zip(*out):
        assert np.isfinite(a).all()
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("nh", [False, True])
@pytest.mark.parametrize("kind", ["plain", "observables", "colour"])
def test_eight_atom_builds_match_oracle(T, orc, kind, nh):
    n, rate = 2050, 0.3  # (the colour field takes even numbers)
    print(f"eight atoms a thread {kind} nh={nh}", flush=True)
    r, p, edge = state(n)
    box, nf = orc.make_box(n, edge), 3 * n - 3
    q = orc.nh_q(nf, TEMP, TAU)
    sr, sp, sz = r.reshape(1, -1), p.reshape(1, -1), np.zeros(1)
    one, maps, four = np.zeros(4, np.int32), np.arange(4, dtype=np.int32), np.full(4, rate)
    if kind == "colour":
        want = orc.run_daughters_colour(box, sr, sp, one, maps, four, DT, STEPS, nthreads=4,
                                        states_zeta=sz if nh else None, temperature=TEMP, q=q, nf=nf)[0]
    elif nh:
        want = orc.run_daughters_nh(box, sr, sp, sz, one, maps, four, DT, TEMP, q, nf, STEPS, nthreads=4)[0]
    else:
        want = orc.run_daughters(box, sr, sp, one, maps, four, DT, STEPS, nthreads=4)[0]
    with T.Context() as ctx:
        mid = ctx.ttcf_init_mother(system(T, n, edge, nh), r, p, n_equil=0)
        ctx.ttcf_import_states(mid, sr, sp)
        ctx.ttcf_record_observables(kind == "observables")
        spawn = ctx.ttcf_spawn_colour if kind == "colour" else ctx.ttcf_spawn_daughters
        first = spawn(mid, 1, 0, rate, STEPS)
        ctx.ttcf_step(STEPS)
        got = ctx.ttcf_export_series(first, 4, STEPS + 1)
    # FP32 forces: 1e-4 of the spread over some tens of steps, as for the other sizes
    assert np.abs(got - want).max() <= 1e-4 * np.std(want)
