"""Skinny product with 8-bit weights: K that leaves a wave no pair of k-steps, less than a batch of them, whole
batches, or whole batches and a part (the part asks for its last pair again and multiplies it with zeros)."""
import pytest

import pd_inputs as I
from oracle import layer as O
from gpu_util import GpuLayer, TOL, relmax

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 8, 9, 16])
@pytest.mark.parametrize("d_model,d_ff", [(64, 64), (192, 320), (256, 2048), (256, 2112), (576, 3200), (256, 8192), (256, 8256), (192, 9024)])
def test_products(d_model, d_ff, B):
    """The down projection's K is d_ff (from 8192 on over eight waves), QKV's and gate / up's d_model."""
    cfg = I.small_config(dtype="bf16", d_model=d_model, n_q_heads=4, n_kv_heads=2, head_dim=128, d_ff=d_ff)
    w = I.layer_weights(cfg, std=0.05)
    ol, gl = O.Layer(cfg, O.quantise_layer_weights(w)), GpuLayer(cfg, w, w8=True)
    oc, gc = O.KVCache(ol, B, 8), gl.cache(B, 8)
    slots = list(range(B))
    for step in range(2):
        x = I.hidden(B, d_model, seed=21 + step, dtype="bf16")
        ref, got = O.decode_step(ol, x, slots, oc), gl.decode(x, slots, gc)
        assert max(relmax(got[i], ref[i]) for i in range(B)) <= 2 * TOL["bf16"]
    gl.close()
