"""fp32 decode steps: the norms ride in the products, the rotary embedding and the cache append in the attention."""
import numpy as np
import pytest
import torch

import paper_2603_04716_amd as pd
import pd_inputs as I
from oracle import layer as O
from gpu_util import GpuLayer, TOL, relmax, to_dev

pytestmark = pytest.mark.gpu


def _layer(head_dim, n_q, n_kv, d=64, d_ff=132):
    cfg = I.small_config(d_model=d, n_q_heads=n_q, n_kv_heads=n_kv, head_dim=head_dim, d_ff=d_ff)
    w = I.layer_weights(cfg, std=0.05)
    rng = np.random.default_rng(head_dim)
    for g in ("g_attn", "g_ffn"):
        w[g] = (1.0 + 0.3 * rng.standard_normal(d)).astype(np.float32)
    return cfg, w


@pytest.mark.parametrize("head_dim,n_q,n_kv", [(32, 4, 4), (64, 4, 1), (64, 6, 2), (128, 2, 2), (256, 2, 1)])
def test_steps_at_chunk_edges(head_dim, n_q, n_kv):
    """Slots that hold nothing, one key, and keys up to each side of a wave's and a workgroup's 64-key chunks; two steps, and
    what they append is what a chunk of one token (its own rotation launch) appends, bit for bit."""
    cfg, w = _layer(head_dim, n_q, n_kv, d=100 if head_dim == 32 else 64)
    ol, gl = O.Layer(cfg, w), GpuLayer(cfg, w)
    lens = [0, 1, 62, 63, 64, 65, 254, 255, 256, 257, 319]
    n, cap = len(lens), 324
    oc, gc, other = O.KVCache(ol, n, cap), gl.cache(n, cap), gl.cache(n, cap)
    rng = np.random.default_rng(1)
    for s, m in enumerate(lens):
        k, v = (rng.standard_normal((n_kv, m, head_dim)).astype(np.float32) for _ in range(2))
        oc.set(s, k, v)
        for c in (gc, other):
            pd.pd_kv_cache_set(c, s, to_dev(k, "f32"), to_dev(v, "f32"))
    slots = list(rng.permutation(n))
    for step in range(2):
        x = I.hidden(n, cfg["d_model"], seed=step)
        got = gl.decode(x, slots, gc)
        assert relmax(got, O.decode_step(ol, x, slots, oc)) <= TOL["f32"]
        gl.prefill_chunk(x, np.arange(n + 1, dtype=np.int32), slots, other)
    for s, m in enumerate(lens):
        a, b = ([torch.empty((n_kv, m + 2, head_dim), device="cuda") for _ in range(2)] for _ in range(2))
        pd.pd_kv_cache_get(gc, s, *a)
        pd.pd_kv_cache_get(other, s, *b)
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    gl.close()


@pytest.mark.parametrize("rows,d,d_ff", [(1, 4, 4), (3, 20, 36), (17, 516, 260), (33, 1028, 68), (500, 256, 1024),
                                         (5, 512, 640), (18, 576, 1040), (3, 1020, 1536), (40, 1040, 2060)])
def test_norm_in_products(rows, d, d_ff):
    """Rows of one k-step and less, K on both sides of the eight-wave form and of its rounds of four and of eight k-steps (512, 1536,
    2060: four; 576, 640, 1020: eight; 1040: nine k-steps a wave, four); rows of very different sizes, one of zeros."""
    cfg, w = _layer(32, 2, 1, d=d, d_ff=d_ff)
    ol, gl = O.Layer(cfg, w), GpuLayer(cfg, w)
    x = I.hidden(rows, d, seed=rows) * np.logspace(-3, 3, rows, dtype=np.float32)[:, None]
    if rows > 1:
        x[rows // 2] = 0.0
    cu = np.array([0, rows], np.int32)
    got, ref = gl.prefill(x, cu), O.prefill(ol, x, cu)
    assert np.isfinite(got).all()
    assert max(relmax(got[i], ref[i]) for i in range(rows) if np.abs(ref[i]).max() > 0) <= 2 * TOL["f32"]
    gl.close()
