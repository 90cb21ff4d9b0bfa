"""List build and force pass of the channel kernel in both of their forms, through the LDS window
and gathering from global memory, against the FP64 oracle (runs on an MI355X).

The forms differ by geometry alone: grid layers that are too large for the window (a channel long
in x and three cells deep in z) take the gathering form. Bar per atom: the pair arithmetic is
FP32, r^2 is off by a few units in 2^-24 and the force goes with its seventh power, so 32 * 2^-23 of
the sum over partners of (48 r^-12 + 24 c r^-6) / r, and 2^-23 of the force for the last rounding.
Atoms with a partner within 2e-6 of the cutoff are left out: the force is cut there and the two
arithmetics may disagree about the pair.
"""
import numpy as np
import pytest
from scipy.spatial import cKDTree

import ttcf_inputs as I

pytestmark = pytest.mark.gpu

SKIN = 0.4


def _state(g, seed):
    r, _, rl = I.channel_initial_state(g, seed)
    rng = np.random.Generator(np.random.PCG64(seed))
    r = r + rng.normal(0.0, 0.03, r.shape)
    r[0] %= g.lx
    r[2] %= g.lz
    return np.ascontiguousarray(r), rl


def _pairs(g, r, radius):
    """(i, j, distance) of the listed kinds: periodic in x and z, no wall-wall pairs."""
    box = np.array([g.lx, 10.0 * g.y_extent, g.lz])
    t = cKDTree(r.T % box, boxsize=box)
    ij = t.query_pairs(radius, output_type="ndarray")
    ij = ij[(ij < g.n_fluid).any(axis=1)]
    d = r[:, ij[:, 0]] - r[:, ij[:, 1]]
    d[0] -= g.lx * np.rint(d[0] / g.lx)
    d[2] -= g.lz * np.rint(d[2] / g.lz)
    return ij, np.sqrt((d * d).sum(axis=0))


@pytest.mark.parametrize("n_x, n_z, n_fluid", [
    (8, 10, 420),       # three cells in x and z: every neighbour row wraps
    (9, 12, 1001),      # ragged
    (16, 20, 5120),     # several chunks, all layers in the window
    (25, 30, 12000),    # the window moves through the layers
    (76, 10, 12160),    # three layers of 6080 slots: gathering form
])
def test_forces_of_both_forms(n_x, n_z, n_fluid):
    from oracle import channel as CHO
    from paper_2312_02990_amd import ttcf as T
    g = I.ChannelSystem(n_x=n_x, n_z=n_z, n_fluid=n_fluid)
    r, rl = _state(g, 5)
    print(f"channel lists {n_x} x {n_z}, {g.n} atoms", flush=True)
    f, out = T.ttcf_channel_debug_forces(T.make_channel(g, skin=SKIN), r.ravel(), rl.ravel())
    fo, oo = CHO.forces(CHO.make_channel(g), r.ravel(), rl.ravel())
    ij, d = _pairs(g, r, g.rc + 0.01)
    edge = np.unique(ij[np.abs(d - g.rc) < 2e-6])
    use = np.ones(g.n, bool)
    use[edge] = False
    s6 = np.where(d < g.rc + 1e-6, d ** -6.0, 0.0)
    c = np.where((ij < g.n_fluid).all(axis=1), g.c_ff, g.c_wf)
    size = np.bincount(ij.ravel(), np.repeat((48 * s6 * s6 + 24 * c * s6) / d, 2), minlength=g.n)
    bar = 2.0 ** -23 * (32 * size + np.abs(fo.reshape(3, -1)).max(axis=0))
    err = np.abs(f - fo).reshape(3, -1).max(axis=0)
    assert use.sum() > 0.9 * g.n
    assert (err[use] <= bar[use]).all()
    assert out[3] == 0 and out[4] == 0
    assert out[2] == pytest.approx(oo[4], rel=1e-12, abs=1e-12)


@pytest.mark.parametrize("n_x, n_z, n_fluid", [(16, 20, 5120), (76, 10, 12160)])
def test_list_capacity_is_exact(n_x, n_z, n_fluid):
    """A capacity that the fullest list just fits is enough, whatever margin the window's coarser
    distances add; one less is an overflow."""
    from paper_2312_02990_amd import ttcf as T
    g = I.ChannelSystem(n_x=n_x, n_z=n_z, n_fluid=n_fluid)
    r, rl = _state(g, 6)
    ij, d = _pairs(g, r, g.rc + SKIN + 0.01)
    longest = [np.bincount(ij[d < (g.rc + SKIN) * (1 + s)].ravel()).max() for s in (-1e-6, 1e-6)]
    assert longest[0] == longest[1]
    k = int(longest[0])
    print(f"channel list capacity {k}", flush=True)
    full, fits = T.ttcf_channel_debug_forces(T.make_channel(g, skin=SKIN), r.ravel(), rl.ravel())
    tight, out = T.ttcf_channel_debug_forces(T.make_channel(g, skin=SKIN, kmax=k), r.ravel(), rl.ravel())
    assert fits[3] == 0 and out[3] == 0
    assert np.array_equal(full, tight)
    _, out = T.ttcf_channel_debug_forces(T.make_channel(g, skin=SKIN, kmax=k - 1), r.ravel(), rl.ravel())
    assert out[3] == 1
