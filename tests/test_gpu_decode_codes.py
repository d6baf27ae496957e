"""Decode over an 8-bit cache whose scales are powers of two (codes from the hardware conversion) or not (from the
double-precision one), with bf16 and 8-bit activations (the fused and the separate append), and batches around the
limits of what one launch's arguments carry."""
import numpy as np
import pytest
import torch

import paper_2603_04716_amd as pd
import pd_inputs as I
from oracle import layer as O
from gpu_util import GpuLayer, TOL, relmax, to_dev, to_np

pytestmark = pytest.mark.gpu

CFG = I.small_config(dtype="bf16", d_model=256, n_q_heads=4, n_kv_heads=2, head_dim=128, d_ff=256)


@pytest.mark.parametrize("scales", [(0.5, 0.125), (0.3, 0.07), (2.0 ** -9, 4.0)])
@pytest.mark.parametrize("B", [1, 5, 66])
def test_new_token_codes(B, scales):
    """2^-9 saturates keys, 4.0 leaves values among the subnormal codes."""
    w = I.layer_weights(CFG, std=0.05)
    ol, gl = O.Layer(CFG, w), GpuLayer(CFG, w)
    lens = np.random.default_rng(B).integers(1, 200, B)
    cap = 256
    oc, gc = O.KVCache(ol, B, cap, fp8_scales=scales), gl.cache(B, cap, fp8_scales=scales)
    for i, n in enumerate(lens):
        k, v = I.kv_fill(2, int(n), 128, seed=500 + i, dtype="bf16")
        oc.set(i, k, v)
        pd.pd_kv_cache_set(gc, i, to_dev(k, "bf16"), to_dev(v, "bf16"))
    slots = list(range(B))[::-1]
    for step in range(2):
        x = I.hidden(B, CFG["d_model"], seed=31 + step, dtype="bf16")
        ref, got = O.decode_step(ol, x, slots, oc), gl.decode(x, slots, gc)
        assert max(relmax(got[i], ref[i]) for i in range(B)) <= 2 * TOL["bf16"]
    for i, n in enumerate(lens):
        k = torch.empty((2, n + 2, 128), dtype=torch.bfloat16, device="cuda")
        v = torch.empty_like(k)
        pd.pd_kv_cache_get(gc, i, k, v)
        torch.cuda.synchronize()
        for got, ref, scale in ((to_np(k)[:, n:], oc.k[i, :, n:n + 2], scales[0]), (to_np(v)[:, n:], oc.v[i, :, n:n + 2], scales[1])):
            # the projections' bf16 error, then the neighbouring code: one spacing; 2^-8 for the read-back's bf16
            mag = np.maximum(np.maximum(np.abs(ref), np.abs(got)) / scale, 2.0 ** -6)
            slack = TOL["bf16"] * np.max(np.abs(ref)) + scale * 2.0 ** (np.floor(np.log2(mag)) - 3) + 2.0 ** -8 * np.abs(ref)
            assert np.all(np.abs(got - ref) <= slack)
    gl.close()


@pytest.mark.parametrize("B,a8", [(256, True), (257, False), (257, True), (480, True), (481, False), (960, True), (961, False)])
def test_batches_at_the_limits_of_a_launch(B, a8):
    """Lengths set for all slots at once, then a step: every row reads its own slot at its own length.  8-bit activations
    (more than 256 rows): the bound derived for the layer, 6e-2."""
    scales = (0.5, 0.125)
    w = I.layer_weights(CFG, std=0.05)
    ol, gl = O.Layer(CFG, O.quantise_layer_weights(w) if a8 else w), GpuLayer(CFG, w, a8=a8)
    rng = np.random.default_rng(B)
    oc, gc = O.KVCache(ol, B, 8, fp8_scales=scales), gl.cache(B, 8, fp8_scales=scales)
    lens = rng.integers(0, 7, B).astype(np.int32)
    for i in range(B):
        k, v = I.kv_fill(2, 7, 128, seed=i, dtype="bf16")
        oc.set(i, k, v)
        pd.pd_kv_cache_set(gc, i, to_dev(k, "bf16"), to_dev(v, "bf16"))
        oc.lens[i] = lens[i]
    slots = rng.permutation(B)
    pd.pd_kv_cache_set_lens(gc, [int(s) for s in slots], [int(lens[s]) for s in slots])
    x = I.hidden(B, CFG["d_model"], seed=3, dtype="bf16")
    ref = O.decode_step(ol, x, [int(s) for s in slots], oc, act8=a8 and B > 256)
    got = gl.decode(x, [int(s) for s in slots], gc)
    assert max(relmax(got[i], ref[i]) for i in range(B)) <= (2 * 6e-2 if a8 else 2 * TOL["bf16"])
    gl.close()
