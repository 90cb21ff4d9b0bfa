"""Exports and imports of rows that lie apart: through a buffer that the context keeps, so a repeated
call neither allocates nor frees (a free would come before its copies have run, and with the default
allocator wait for every stream of the device); more bytes than the buffer holds go in parts."""
import gc

import numpy as np
import pytest

import ttcf_inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    from paper_2312_02990_amd import ttcf
    ttcf.lib()
    return ttcf


@pytest.fixture
def calls(T):
    """The library's allocations and frees, counted."""
    import ctypes as C

    import torch
    held, seen = {}, []

    def alloc(nbytes, stream, user):
        block = torch.empty(int(nbytes), dtype=torch.uint8, device="cuda")
        held[block.data_ptr()] = block
        seen.append("alloc")
        return block.data_ptr()

    def free(ptr, user):
        seen.append("free")
        torch.cuda.synchronize()
        del held[ptr]

    gc.collect()
    a, f = T._ALLOC(alloc), T._FREE(free)
    assert T.lib().ttcf_set_allocator(a, f, None) == T.TTCF_OK
    yield seen
    gc.collect()
    assert T.lib().ttcf_set_allocator(C.cast(None, T._ALLOC), C.cast(None, T._FREE), None) == T.TTCF_OK
    assert not held


def test_repeated_calls_do_not_allocate(T, calls):
    s = I.System(4)
    count = 9
    r = np.stack([I.perturbed_positions(s, k, 0.05).ravel() for k in range(count)])
    p = np.stack([I.maxwell_boltzmann(s.n, s.temperature, 40 + k).ravel() for k in range(count)])
    with T.Context() as ctx:
        mid = ctx.ttcf_init_mother(T.make_system(s.n, s.box, s.temperature, s.dt), r[0], p[0], n_equil=0)
        ctx.ttcf_import_states(mid, r, p)
        first = ctx.ttcf_spawn_daughters(mid, count, 0, 0.1, 20)
        ctx.ttcf_step(20)

        def work():
            ctx.ttcf_import_states(mid, r, p)
            return (*ctx.ttcf_export_states(mid, count), ctx.ttcf_export_series(first, 4 * count, 7))

        once = work()
        del calls[:]
        again = work()
        assert calls == []
        for a, b in zip(once, again):
            np.testing.assert_array_equal(a, b)


def test_channel_calls_do_not_allocate(T, calls):
    g = I.ChannelSystem(n_x=7, n_z=10, n_fluid=420)
    r0, p0, lat = I.channel_initial_state(g, 3)
    r, p, z = np.stack([r0.ravel()] * 5), np.stack([p0.ravel()] * 5), np.linspace(-0.1, 0.1, 5)
    with T.ChannelContext(T.make_channel(g), r0, p0, lat) as ctx:
        ctx.import_states(r, p, z)
        ctx.export_states(5)
        del calls[:]
        ctx.import_states(r, p, z)
        for got, want in zip(ctx.export_states(5), (r, p, z)):
            np.testing.assert_array_equal(got, want)
        assert calls == []


def test_more_than_the_buffer_holds(T):
    s, count = I.System(4), 3001  # 18 MB of positions
    rng = np.random.Generator(np.random.PCG64(5))
    r = rng.uniform(0.0, s.box, (count, 3 * s.n))
    p = rng.standard_normal((count, 3 * s.n))
    r0 = I.perturbed_positions(s, 1, 0.05)
    with T.Context() as ctx:
        mid = ctx.ttcf_init_mother(T.make_system(s.n, s.box, s.temperature, s.dt), r0, p[0], n_equil=0)
        ctx.ttcf_import_states(mid, r, p)
        er, ep = ctx.ttcf_export_states(mid, count)
    np.testing.assert_array_equal(er, r)
    np.testing.assert_array_equal(ep, p)
