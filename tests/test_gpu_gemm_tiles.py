"""The network's products at the edges of their tiles: rows and outputs just past a tile, a K chunk
or the four values of a vector load, and enough rows for the larger tile, forward and gradient
against the bfloat16 oracle."""
import numpy as np
import pytest

import ttcf_inputs as I
from oracle import mlp as M

pytestmark = pytest.mark.gpu

N_IN, N_HID = 64, 256


@pytest.fixture(scope="module")
def ctx():
    from paper_2312_02990_amd import ttcf as T
    s = I.System(4)
    r, p = I.initial_state(s, 3)
    with T.Context() as c:
        c.ttcf_init_mother(T.make_system(s.n, s.box, s.temperature, s.dt), r, p, n_equil=0)
        yield c


@pytest.mark.parametrize("rows,n_out", [(1, 1), (31, 3), (33, 50), (64, 32), (257, 64), (1025, 201),
                                        (4200, 30)])
def test_forward_and_gradient(ctx, rows, n_out):
    print(f"network rows={rows} n_out={n_out}", flush=True)
    rng = np.random.Generator(np.random.PCG64(rows + n_out))
    w32 = M.init_weights(N_IN, N_HID, n_out, 5).flat().astype(np.float32)
    w32 += 0.02 * rng.standard_normal(w32.size).astype(np.float32)
    net = M.MLP.from_flat(w32.astype(np.float64), N_IN, N_HID, n_out)
    x = rng.standard_normal((rows, N_IN)).astype(np.float32)
    t = rng.standard_normal((rows, n_out)).astype(np.float32)
    ctx.ttcf_cv_init(n_out, w32)
    y, cache = M.forward(net, x.astype(np.float64), bf16=True)
    grad = M.backward(net, cache, y, t.astype(np.float64), bf16=True)
    # FP32 and FP64 sums round a few operands in a thousand to neighbouring bfloat16 values, 2^-8
    # apart, among 64 or more terms of a sum
    got = ctx.ttcf_mlp_forward(x)
    assert np.abs(got - y).max() <= 4e-3 * np.abs(y).max()
    g = M.MLP.from_flat(ctx.ttcf_mlp_gradient(x, t).astype(np.float64), N_IN, N_HID, n_out)
    for a, b in zip(g.params(), grad.params()):
        assert np.linalg.norm(a - b) <= 4e-3 * np.linalg.norm(b)
