"""Daughters with FP64 forces over neighbour lists (ttcf_flow64.hip) against the oracle: shear,
planar elongation and mixed flow where the launch changes shape (one, two and four atoms per
thread, chosen by the batch), at atom numbers just past a wave or a thread count, in a box of
three cells a side (no room for a list skin), and with lists that outgrow their capacity (built at
the cutoff every step instead). Copies of one start state in a batch come out bit for bit alike."""
import numpy as np
import pytest

import ttcf_inputs as I

pytestmark = pytest.mark.gpu

DT, TEMP, STEPS = 0.0025, 0.722, 30


@pytest.fixture(scope="module")
def T():
    from paper_2312_02990_amd import ttcf
    ttcf.lib()
    return ttcf


def state(n, density, seed, slab=False):
    """n atoms of a jittered fcc lattice, and their momenta at TEMP."""
    m = int(np.ceil((n / 4.0) ** (1.0 / 3.0) - 1e-9))
    box = (n / density) ** (1.0 / 3.0)
    rng = np.random.Generator(np.random.PCG64(seed))
    sites = I.fcc_lattice(8 if slab else m, box)
    # all sites' lowest layers of y, or n of the sites that just hold n
    keep = np.argsort(sites[1], kind="stable")[:n] if slab else np.sort(rng.permutation(4 * m ** 3)[:n])
    r = sites[:, keep] + rng.uniform(-0.04, 0.04, (3, n))
    return np.mod(r, box), I.maxwell_boltzmann(n, TEMP, seed + 1), box


# flow, atoms, start-state copies, cutoff, density
CASES = [
    ("shear", 109, 1, I.WCA_RC, 0.8442),     # one atom per thread, a wave and a half
    ("narrow", 108, 1, I.WCA_RC, 1.1),       # elongation of a box from 4.1 to 3.14 cutoffs
    ("mixed", 257, 1, I.WCA_RC, 0.8442),
    ("shear", 1025, 1, I.WCA_RC, 0.8442),    # two per thread, one atom past 1024
    ("mixed", 1025, 1, I.WCA_RC, 0.8442),
    ("shear", 301, 322, I.WCA_RC, 0.8442),   # four per thread: more daughters than the chip holds
    ("elong", 301, 322, I.WCA_RC, 0.8442),
    ("shear", 2048, 65, I.WCA_RC, 0.8442),   # the largest system, four per thread
    ("mixed", 2047, 65, I.WCA_RC, 0.8442),
    ("elong", 500, 1, 1.5, 1.05),            # lists beyond their capacity with a skin
    ("shear", 500, 1, 1.5, 1.05),            # too dense for lists: the cell form
    ("slab", 600, 1, 1.75, 0.45),            # dense layers: more neighbours than a list holds
]


@pytest.mark.parametrize("nh", [False, True])
@pytest.mark.parametrize("flow,n,copies,rc,density", CASES)
def test_matches_oracle(T, orc, flow, n, copies, rc, density, nh):
    print(f"flow64 {flow} n={n} copies={copies} rc={rc:.3f} nh={nh}", flush=True)
    r, p, edge = state(n, density, 5 * n, flow == "slab")
    box = orc.make_box(n, edge, rc=rc)
    rate, zeta0, nf = 3.6 if flow == "narrow" else 0.6, 0.4, 3 * n - 3
    flow = {"narrow": "elong", "slab": "shear"}.get(flow, flow)
    q = orc.nh_q(nf, TEMP, 0.25)
    one, maps, four = np.zeros(4, np.int32), np.arange(4, dtype=np.int32), np.full(4, rate)
    sr, sp, sz = r.reshape(1, -1), p.reshape(1, -1), np.array([zeta0])
    if flow == "mixed":
        extra = dict(states_zeta=sz, temperature=TEMP, q=q, nf=nf) if nh else {}
        want = orc.run_daughters_mix(box, sr, sp, one, maps, 0.5 * four, four, DT, STEPS, 4, **extra)[0]
    elif flow == "elong":
        extra = dict(states_zeta=sz, temperature=TEMP, q=q, nf=nf) if nh else {}
        want = orc.run_daughters_pef(box, sr, sp, one, maps, four, DT, STEPS, 4, **extra)[0]
    elif nh:
        want = orc.run_daughters_nh(box, sr, sp, sz, one, maps, four, DT, TEMP, q, nf, STEPS, nthreads=4)[0]
    else:
        want = orc.run_daughters(box, sr, sp, one, maps, four, DT, STEPS, nthreads=4)[0]
    sysd = T.make_system(n, edge, TEMP, DT, r_cut=rc, precision=T.TTCF_PREC_FP64,
                         potential=T.TTCF_WCA if rc == I.WCA_RC else T.TTCF_LJ,
                         thermostat=T.TTCF_DAUGHTER_NH if nh else T.TTCF_DAUGHTER_GIK)
    with T.Context() as ctx:
        mid = ctx.ttcf_init_mother(sysd, r, p, n_equil=0)
        ctx.ttcf_import_states(mid, np.repeat(sr, copies, 0), np.repeat(sp, copies, 0))
        ctx.ttcf_import_states_zeta(mid, np.full(copies, zeta0))
        if flow == "mixed":
            first = ctx.ttcf_spawn_mixed(mid, copies, 0, 0.5 * rate, rate, STEPS)
        elif flow == "elong":
            first = ctx.ttcf_spawn_elongational(mid, copies, 0, rate, STEPS)
        else:
            first = ctx.ttcf_spawn_daughters(mid, copies, 0, rate, STEPS)
        ctx.ttcf_step(STEPS)
        got = ctx.ttcf_export_series(first, 4 * copies, STEPS + 1)
        assert ctx.ttcf_accumulate() == copies
    # FP64 on both sides: roundings of 1e-16 grow less than a thousandfold over 30 steps
    assert np.abs(got[:4] - want).max() <= 1e-9 * np.std(want)
    np.testing.assert_array_equal(got.reshape(copies, 4, -1), np.broadcast_to(got[:4], (copies, 4, STEPS + 1)))
