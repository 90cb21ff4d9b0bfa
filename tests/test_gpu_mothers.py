"""Mothers over neighbour lists (k_mother_lists) against the oracle where the launch changes shape:
one and four atoms per thread, atom numbers just past a wave or a thread count, a box of three cells
a side, dense layers with more neighbours than a list holds, and the cell form beyond 2048 atoms.
The FP32 form takes an atom's partners in an order that only the current positions decide: a run
split over calls, with lists rebuilt on other steps, differs from the whole one by the FP64 sums of
p^2 alone."""
import numpy as np
import pytest

import ttcf_inputs as I

pytestmark = pytest.mark.gpu

DT, TEMP, TAU = 0.0025, 0.722, 0.25


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
    keep = np.argsort(sites[1], kind="stable")[:n] if slab else np.sort(rng.permutation(4 * m ** 3)[:n])
    r = np.mod(sites[:, keep] + rng.uniform(-0.04, 0.04, (3, n)), box)
    return np.ascontiguousarray(r), I.maxwell_boltzmann(n, TEMP, seed + 1), box


def system(T, n, box, rc, precision, threads=0):
    return T.make_system(n, box, TEMP, DT, r_cut=rc, precision=precision, nh_tau=TAU, block_threads=threads,
                         potential=T.TTCF_WCA if rc == I.WCA_RC else T.TTCF_LJ)


@pytest.mark.parametrize("precision,tol", [(0, 1e-9), (1, 1e-4)])
@pytest.mark.parametrize("n,rc,density,slab", [
    (108, I.WCA_RC, 1.1, False),       # three cells a side
    (109, I.WCA_RC, 0.8442, False),
    (1024, I.WCA_RC, 0.8442, False),   # the largest with one atom per thread
    (1025, I.WCA_RC, 0.8442, False),   # four per thread, all but the last waves empty of the fourth
    (2048, I.WCA_RC, 0.8442, False),
    (2049, I.WCA_RC, 0.8442, False),   # the cell form
    (600, 1.75, 0.45, True),           # dense layers
])
def test_matches_oracle(T, orc, n, rc, density, slab, precision, tol):
    print(f"mother n={n} rc={rc:.3f} precision={precision}", flush=True)
    r, p, edge = state(n, density, 3 * n, slab)
    equil, count, between = 7, 2, 12
    with T.Context() as ctx:
        mid = ctx.ttcf_init_mother(system(T, n, edge, rc, precision), r, p, n_equil=equil)
        ctx.ttcf_sample_states(mid, count, between)
        gr, gp = ctx.ttcf_export_states(mid, count)
        gz = ctx.ttcf_export_states_zeta(mid, count)
    nf = 3 * n - 3
    st = orc.NHState(r.ravel().copy(), p.ravel().copy())
    wr, wp, wz = orc.mother_sample(orc.make_box(n, edge, rc=rc), st, equil, count, between, TEMP, DT,
                                   orc.nh_q(nf, TEMP, TAU), nf, with_zeta=True)
    dr = gr - wr
    dr -= edge * np.rint(dr / edge)
    assert np.abs(dr).max() / edge <= tol
    assert np.abs(gp - wp).max() / np.sqrt(np.mean(wp ** 2)) <= tol
    np.testing.assert_allclose(gz, wz, rtol=100 * tol, atol=100 * tol)


@pytest.mark.parametrize("n", [500, 2048])
def test_fp32_sums_do_not_depend_on_the_lists(T, n):
    r, p, edge = state(n, 0.8442, n)
    out = []
    for parts in ((60,), (23, 37)):
        print(f"mother n={n} in {len(parts)} parts", flush=True)
        with T.Context() as ctx:
            mid = ctx.ttcf_init_mother(system(T, n, edge, I.WCA_RC, 1), r, p, n_equil=0)
            for k in parts:
                ctx.ttcf_sample_states(mid, 1, k)
            out.append(np.concatenate(ctx.ttcf_export_states(mid, 1)))
    # sums of p^2 in another order: 1e-16, grown less than a thousandfold; another order of an
    # FP32 force sum would show at 1e-7
    assert np.abs(out[0] - out[1]).max() <= 1e-12 * edge


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n,density,threads", [(108, 1.1, 128), (500, 0.8442, 512), (1025, 0.8442, 1024)])
def test_lists_and_cells_agree(T, n, density, threads, precision):
    """A system that fixes its workgroup size runs in the cell form: the same separations and the
    same order of every FP32 sum, so the same trajectory but for FP64 sums."""
    print(f"mother n={n} precision={precision} lists against cells", flush=True)
    r, p, edge = state(n, density, 7 * n)
    out = []
    for t in (0, threads):
        with T.Context() as ctx:
            mid = ctx.ttcf_init_mother(system(T, n, edge, I.WCA_RC, precision, t), r, p, n_equil=0)
            ctx.ttcf_sample_states(mid, 1, 40)
            out.append(np.concatenate(ctx.ttcf_export_states(mid, 1)))
    assert np.abs(out[0] - out[1]).max() <= 1e-12 * edge
