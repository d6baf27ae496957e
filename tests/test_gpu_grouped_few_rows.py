"""Grouped products of up to 256 rows per group on the average, on both sides of each line between the tiles (64, 128, 256
rows and the forms of longer products), with experts that need one row tile, several, or none: launches of few workgroups,
which keep the lowest tile while even second row tiles find a CU of their own, and of many."""
import ctypes as C

import numpy as np
import pytest

import paper_2603_04716_amd as pd
import pd_inputs as I
from oracle import layer as O
from gpu_util import GpuLayer, TOL, relmax

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [32, 33, 107, 108, 160, 161, 256])
@pytest.mark.parametrize("skew", [0.0, 9.0])
def test_each_side_of_a_line(rows, skew):
    T = 4 * rows                                   # 8 experts, two of them per token
    cfg = I.small_config(dtype="bf16", d_model=256, n_q_heads=4, n_kv_heads=2, head_dim=128, d_ff=384, n_experts=8, top_k=2)
    w = I.layer_weights(cfg, std=0.05)
    ol, gl = O.Layer(cfg, w), GpuLayer(cfg, w)
    r = I.router_logits(T, 8, seed=T)
    r[:, 5] += skew                                # with skew, every token takes expert 5: 4 x the mean
    cu = np.array([0, T // 3, T], np.int32)
    x = I.hidden(T, cfg["d_model"], seed=8, dtype="bf16")
    ref, eref = O.prefill(ol, x, cu, router_logits=r, return_experts=True)
    got = gl.prefill(x, cu, router_logits=r)
    assert np.array_equal(gl.experts(T), eref)
    assert max(relmax(got[i], ref[i]) for i in range(T)) <= 2 * TOL["bf16"]
    gl.close()


def row_tile(M, N, K, epilogue, groups, scratch):
    return pd.lib.pd_internal_grouped_row_tile(M, N, K, epilogue, groups, C.c_longlong(scratch))


# 8 experts, two of them per token; gate/up of 8192 columns is 512 workgroups and more, of 1024 columns 64 and more
@pytest.mark.parametrize("rows,d_ff,tile", [(32, 4096, 64), (33, 4096, 128), (107, 4096, 128), (108, 4096, 256), (160, 4096, 256),
                                            (44, 2048, 64), (52, 2048, 128), (160, 512, 64), (160, 1024, 128), (160, 1536, 256)])
@pytest.mark.parametrize("skew", [0.0, 9.0])
def test_row_tile(rows, d_ff, tile, skew):
    T, d = 4 * rows, 128
    cfg = I.small_config(dtype="bf16", d_model=d, n_q_heads=2, n_kv_heads=1, head_dim=128, d_ff=d_ff, n_experts=8, top_k=2)
    assert row_tile(2 * T, d_ff, d, 2, 8, 256 * (640 * 128 + 2 * max(512, 2 * d_ff))) == tile
    w = I.layer_weights(cfg, std=0.05)
    ol, gl = O.Layer(cfg, w), GpuLayer(cfg, w)
    r = I.router_logits(T, 8, seed=T)
    r[:, 5] += skew
    cu = np.array([0, T // 3, T], np.int32)
    x = I.hidden(T, d, seed=8, dtype="bf16")
    ref, eref = O.prefill(ol, x, cu, router_logits=r, return_experts=True)
    got = gl.prefill(x, cu, router_logits=r)
    assert np.array_equal(gl.experts(T), eref)
    assert max(relmax(got[i], ref[i]) for i in range(T)) <= 2 * TOL["bf16"]
    gl.close()
