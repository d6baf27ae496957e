"""Mixture-of-experts products on the tiled kernel: a grouped launch holds a row tile per group more than its rows
may need, and the tiles in use are dealt over the chip whatever the loads of the experts are."""
import numpy as np
import pytest

import pd_inputs as I
from oracle import layer as O
from gpu_util import GpuLayer, TOL, relmax, tile_plan

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d_ff,form", [(12, 1024, None), (64, 2048, None), (700, 1024, None), (2500, 512, "pair"), (2500, 1024, "deep"),
                                         (1150, 4096, "192"), (1450, 4096, "256")])
@pytest.mark.parametrize("skew", ["even", "two", "ragged"])
def test_grouped_products_deal_the_tiles_in_use(T, d_ff, form, skew):
    """Expert loads from even to two experts with all rows: the tiles in use are from all to few of those launched.
    form: of the gate / up product, where an expert has more than 256 rows on the average (its loads are not known on
    the host, so the forms are the same for every skew)."""
    if form:
        assert tile_plan(2 * T, d_ff, 256, 2, 8) == form
    cfg = I.small_config(dtype="bf16", d_model=256, n_q_heads=4, n_kv_heads=2, head_dim=128, d_ff=d_ff, n_experts=8, top_k=2)
    w = I.layer_weights(cfg, std=0.05)
    ol, gl = O.Layer(cfg, w), GpuLayer(cfg, w)
    r = I.router_logits(T, 8, seed=T)
    if skew == "two":
        r[:, 1] += 9.0
        r[:, 6] += 8.0
    if skew == "ragged":
        r += np.linspace(0.0, 3.0, 8, dtype=r.dtype)
    n = T // 4
    cu = np.array([0, n, 2 * n, 3 * n, T], np.int32)
    x = I.hidden(T, cfg["d_model"], seed=8, dtype="bf16")
    ref, eref = O.prefill(ol, x, cu, router_logits=r, return_experts=True)
    got = gl.prefill(x, cu, router_logits=r)
    assert np.array_equal(gl.experts(T), eref)
    assert relmax(got, ref) <= TOL["bf16"]
    assert max(relmax(got[i], ref[i]) for i in range(T)) <= 2 * TOL["bf16"]
    gl.close()


@pytest.mark.parametrize("T,E,top_k", [(31, 8, 2), (32, 8, 2), (33, 8, 2), (512, 8, 2), (513, 8, 2), (200, 64, 5), (128, 64, 8), (157, 64, 6), (158, 64, 6), (1, 3, 1)])
def test_routing_in_one_launch(T, E, top_k):
    """Up to 1024 pairs and 10240 staged logits are sorted by one workgroup, more by the general kernels; the place of
    every pair shows in the rows' outputs, ties go to the lower expert."""
    cfg = I.small_config(dtype="bf16", d_model=128, n_q_heads=2, n_kv_heads=1, head_dim=128, d_ff=64, n_experts=E, top_k=top_k)
    w = I.layer_weights(cfg, std=0.05)
    ol, gl = O.Layer(cfg, w), GpuLayer(cfg, w)
    r = I.router_logits(T, E, seed=T + E)
    r[T // 2] = 0.25
    cu = np.array([0, T], np.int32)
    x = I.hidden(T, cfg["d_model"], seed=9, dtype="bf16")
    ref, eref = O.prefill(ol, x, cu, router_logits=r, return_experts=True)
    got = gl.prefill(x, cu, router_logits=r)
    assert np.array_equal(gl.experts(T), eref)
    assert max(relmax(got[i], ref[i]) for i in range(T)) <= 2 * TOL["bf16"]
    gl.close()
