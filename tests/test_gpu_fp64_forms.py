"""FP64 shear daughters over neighbour lists and in the cell form in one call: the form of a daughter
follows from its own system. Daughters of two sizes, and of either thermostat, in one list launch
against the oracle."""
import numpy as np
import pytest

import ttcf_inputs as I

pytestmark = pytest.mark.gpu

DT, TEMP, TAU, STEPS = 0.0025, 0.722, 0.25, 30


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


def run(T, systems):
    """Series of the four mapped daughters of each (n, block_threads, thermostat), in one step call."""
    with T.Context() as ctx:
        ids = []
        for n, threads, thermostat in systems:
            r, p, edge = state(n)
            sysd = T.make_system(n, edge, TEMP, DT, precision=T.TTCF_PREC_FP64, block_threads=threads,
                                 nh_tau=TAU, thermostat=thermostat)
            ids.append((ctx.ttcf_init_mother(sysd, r, p, n_equil=0), r, p))
        first = []
        for mid, r, p in ids:
            ctx.ttcf_import_states(mid, r.reshape(1, -1), p.reshape(1, -1))
            first.append(ctx.ttcf_spawn_daughters(mid, 1, 0, 0.3, STEPS))
        ctx.ttcf_step(STEPS)
        return [ctx.ttcf_export_series(f, 4, STEPS + 1) for f in first]


@pytest.mark.parametrize("other", [(300, 320, 0), (2049, 0, 0)])  # a fixed workgroup size; too many atoms
def test_form_does_not_depend_on_the_neighbours(T, other):
    print(f"FP64 forms beside {other}", flush=True)
    alone = run(T, [(256, 0, 0)])[0]
    beside = run(T, [(256, 0, 0), other])
    np.testing.assert_array_equal(beside[0], alone)
    np.testing.assert_array_equal(beside[1], run(T, [other])[0])


def test_two_sizes_and_thermostats_in_one_call(T, orc):
    systems = [(256, 0, 0), (1100, 0, 0), (300, 0, 1), (130, 0, 1)]
    print("FP64 lists of several sizes in one call", flush=True)
    got = run(T, systems)
    one, maps, rate = np.zeros(4, np.int32), np.arange(4, dtype=np.int32), np.full(4, 0.3)
    for (n, _, nh), g in zip(systems, got):
        r, p, edge = state(n)
        box, nf = orc.make_box(n, edge), 3 * n - 3
        sr, sp = r.reshape(1, -1), p.reshape(1, -1)
        if nh:
            want = orc.run_daughters_nh(box, sr, sp, np.zeros(1), one, maps, rate, DT, TEMP,
                                        orc.nh_q(nf, TEMP, TAU), nf, STEPS, nthreads=4)[0]
        else:
            want = orc.run_daughters(box, sr, sp, one, maps, rate, DT, STEPS, nthreads=4)[0]
        # FP64 on both sides: roundings of 1e-16 grow less than a thousandfold over 30 steps
        assert np.abs(g - want).max() <= 1e-9 * np.std(want)


def test_autotune_reports_what_runs(T):
    """Where FP64 forces take lists there is one shape: tuned, set as returned, imported, default."""
    print("FP64 autotune", flush=True)
    n, out = 500, []
    r, p, edge = state(n)
    sysd = T.make_system(n, edge, TEMP, DT, precision=T.TTCF_PREC_FP64)
    text = None
    for how in ("tuned", "set", "imported", "default"):
        with T.Context() as ctx:
            mid = ctx.ttcf_init_mother(sysd, r, p, n_equil=0)
            ctx.ttcf_import_states(mid, r.reshape(1, -1), p.reshape(1, -1))
            first = ctx.ttcf_spawn_daughters(mid, 1, 0, 0.3, STEPS)
            if how == "tuned":
                shape = ctx.ttcf_autotune(mid, 0, 0.3, 10)
                text = ctx.ttcf_autotune_export()
                assert shape["variant"] == 0 and shape["candidates"] == 1 and shape["ms_per_step"] > 0.0
            elif how == "set":
                ctx.ttcf_set_step_shape(shape["variant"], shape["threads"], shape["skin"], shape["kmax"])
            elif how == "imported":
                ctx.ttcf_autotune_import(text)
                with pytest.raises(T.TTCFError):
                    ctx.ttcf_autotune_import(text.replace('"precision": 0', '"precision": 1'))
            ctx.ttcf_step(STEPS)
            out.append(ctx.ttcf_export_series(first, 4, STEPS + 1))
    for series in out[1:]:
        np.testing.assert_array_equal(series, out[0])


@pytest.mark.parametrize("n", [300, 1100])
@pytest.mark.parametrize("flow", ["shear", "elong", "mixed"])
def test_shapes_and_splits_agree_to_rounding(T, n, flow):
    """A start state alone (one or two atoms a thread), in a batch that fills the chip (four), and over
    two step calls: sums in other orders, lists rebuilt on other steps."""
    print(f"FP64 lists {flow} n={n} in several shapes", flush=True)
    r, p, edge = state(n)
    sysd = T.make_system(n, edge, TEMP, DT, precision=T.TTCF_PREC_FP64)
    out = []
    for copies, parts in ((1, (STEPS,)), (322, (STEPS,)), (1, (11, STEPS - 11))):
        with T.Context() as ctx:
            mid = ctx.ttcf_init_mother(sysd, r, p, n_equil=0)
            ctx.ttcf_import_states(mid, np.repeat(r.reshape(1, -1), copies, 0), np.repeat(p.reshape(1, -1), copies, 0))
            if flow == "mixed":
                first = ctx.ttcf_spawn_mixed(mid, copies, 0, 0.2, 0.3, STEPS)
            elif flow == "elong":
                first = ctx.ttcf_spawn_elongational(mid, copies, 0, 0.3, STEPS)
            else:
                first = ctx.ttcf_spawn_daughters(mid, copies, 0, 0.3, STEPS)
            for k in parts:
                ctx.ttcf_step(k)
            out.append(ctx.ttcf_export_series(first, 4, STEPS + 1))
    for series in out[1:]:
        # roundings of 1e-16 grow less than a thousandfold over 30 steps
        assert np.abs(series - out[0]).max() <= 1e-12 * np.abs(out[0]).max()
