"""SwiGLU of gates at the ends of the exponent's range, in every kernel that forms it: z / (1 + exp(-z)) of an infinite gate,
of gates whose exponential overflows or nearly does, and of ordinary ones, by the number of rows of the call."""
import numpy as np
import pytest

import pd_inputs as I
from gpu_util import GpuLayer, tile_plan

pytestmark = pytest.mark.gpu
GATES = [np.inf, 2.0 ** 127, 2.0 ** 60, 88.0, 4.0, 1.0, 0.0, -1.0, -4.0, -80.0, -86.0, -87.0, -88.0, -88.5, -89.0, -96.0, -1024.0, -2.0 ** 60, -2.0 ** 126,
         -2.0 ** 127, np.nan, -np.inf]


# a few rows: the skinny kernel; then the tile forms, with K split (the sum's launch) and without
@pytest.mark.parametrize("T,d,d_ff,form,first", [(16, 256, 256, None, 0), (16, 256, 256, None, 8), (22, 256, 256, "64", 0), (200, 256, 8192, "128x64", 0),
                                                 (300, 256, 256, "deep", 0), (300, 1024, 128, "deep/split", 0), (2200, 256, 1024, "pair", 0),
                                                 (3000, 256, 4096, "192", 0), (1600, 256, 8192, "256", 0)])
def test_gates(T, d, d_ff, form, first):
    """Row t is a unit vector: its normalised row is sqrt(d) in one place, which meets one weight in one row of the gate matrix, and
    the down projection adds the one product that is not 0 to every column.  An infinite gate is a sum that overflows, a gate that
    is not a number two of those of opposite sign.  Bound: the exponential's few ulp and two roundings to bf16, 2^-7."""
    cfg = I.small_config(dtype="bf16", d_model=d, n_q_heads=2, n_kv_heads=1, head_dim=128, d_ff=d_ff)
    scratch = 256 * (640 * 128 + 2 * max(512, 2 * d_ff, d))
    if form:
        assert tile_plan(T, d_ff, d, 2, 0, scratch) == form
    w = {k: np.zeros_like(v) for k, v in I.layer_weights(cfg).items()}
    w["g_attn"][:] = w["g_ffn"][:] = w["w_down"][:] = 1.0
    root = np.float32(np.sqrt(d))
    w["w_up"][:] = 1.0 / root
    gates = np.roll(np.array(GATES, np.float32), -first)
    x = np.zeros((T, d), np.float32)
    huge = np.float32(2.0 ** 127)
    for j, z in enumerate(gates):
        f, at = (37 * j + 3) % d_ff, (11 * j) % d
        if np.isfinite(z):
            w["w_gate"][f, at] = z / root
        elif not np.isnan(z):
            w["w_gate"][f, at] = np.sign(z) * huge
        x[j::len(gates), at] = 1.0
        if np.isnan(z):                                # two places of the row, each overflowing
            w["w_gate"][f, at], w["w_gate"][f, at + 1] = huge, -huge
            x[j::len(gates), at + 1] = 1.0
    gl = GpuLayer(cfg, w)
    got = gl.prefill(x, np.array([0, T], np.int32))
    gl.close()
    with np.errstate(over="ignore", invalid="ignore"):
        act = (gates.astype(np.float64) / (1.0 + np.exp(-gates.astype(np.float64)))).astype(np.float32)
        act[np.exp(-gates) == np.inf] = np.where(np.isinf(gates[np.exp(-gates) == np.inf]), np.nan, -0.0)   # the exponential is a float
    for t in range(T):
        a = act[t % len(gates)]
        want = x[t] + a
        if np.isnan(a):
            assert np.isnan(got[t]).all(), t
        elif np.isinf(a):
            assert (got[t] == a).all(), t
        else:
            assert (np.abs(got[t] - want) <= 2.0 ** -7 * np.abs(want)).all(), (t, gates[t % len(gates)], got[t][:4], want[:4])
