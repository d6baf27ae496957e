"""Cache fill and read-back over the blocked layouts: whole and partial blocks, tensors that are and are not
16-byte aligned, and what a fill must leave alone."""
import pytest
import torch

import paper_2603_04716_amd as pd
import pd_inputs as I
from gpu_util import GpuLayer

pytestmark = pytest.mark.gpu

CFG = I.small_config(dtype="bf16", d_model=256, n_q_heads=4, n_kv_heads=2, head_dim=128, d_ff=512)


def _tensors(n, seed, shift):
    """Two [2, n, 128] bf16 tensors whose first element sits `shift` elements behind a 16-byte boundary."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    flat = torch.randn((2, 2 * n * 128 + 8), device="cuda", generator=gen).to(torch.bfloat16)
    return [f[shift:shift + 2 * n * 128].view(2, n, 128) for f in flat]


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("n", [1, 31, 32, 33, 63, 64, 65, 127, 200])
@pytest.mark.parametrize("shift", [0, 1])
def test_set_get_blocks(fp8, n, shift):
    gl = GpuLayer(CFG, I.layer_weights(CFG, std=0.05))
    cap = 203
    gc = gl.cache(3, cap, fp8_scales=(0.5, 0.125) if fp8 else None)
    full_k, full_v = _tensors(cap, 1, 0)
    for s in range(3):
        pd.pd_kv_cache_set(gc, s, full_k, full_v)
    k, v = _tensors(n, 2, shift)
    pd.pd_kv_cache_set(gc, 1, k, v)
    pd.pd_kv_cache_set_len(gc, 1, cap)           # positions behind the new ones must still be the old ones

    def stored(t, scale):
        if not fp8:
            return t
        return (t.float() / scale).clamp(-448, 448).to(torch.float8_e4m3fn).float().mul(scale).to(torch.bfloat16)

    for s in (0, 1, 2):
        want_k, want_v = stored(full_k, 0.5).clone(), stored(full_v, 0.125).clone()
        if s == 1:
            want_k[:, :n], want_v[:, :n] = stored(k, 0.5), stored(v, 0.125)
        for length in (cap, n):
            gk, gv = _tensors(length, 3, shift)
            pd.pd_kv_cache_get(gc, s, gk, gv)
            torch.cuda.synchronize()
            assert torch.equal(gk, want_k[:, :length]) and torch.equal(gv, want_v[:, :length])
    gl.close()


def test_more_heads_than_a_grid_dimension():
    h = 65537
    cfg = I.small_config(dtype="bf16", d_model=2, n_q_heads=h, n_kv_heads=h, head_dim=128, d_ff=2)
    zeros = lambda *s: torch.zeros(s, device="cuda", dtype=torch.bfloat16)
    layer = pd.pd_layer_create(cfg, {"g_attn": zeros(2), "w_q": zeros(h * 128, 2), "w_k": zeros(h * 128, 2), "w_v": zeros(h * 128, 2),
                                     "w_o": zeros(2, h * 128), "g_ffn": zeros(2), "w_gate": zeros(2, 2), "w_up": zeros(2, 2),
                                     "w_down": zeros(2, 2)})
    cache = pd.pd_kv_cache_create(layer, 1, 3)
    gen = torch.Generator(device="cuda").manual_seed(4)
    k, v = (torch.randn((h, 3, 128), device="cuda", generator=gen).to(torch.bfloat16) for _ in range(2))
    gk, gv = torch.empty_like(k), torch.empty_like(v)
    pd.pd_kv_cache_set(cache, 0, k, v)
    pd.pd_kv_cache_get(cache, 0, gk, gv)
    torch.cuda.synchronize()
    assert torch.equal(gk, k) and torch.equal(gv, v)
    pd.pd_kv_cache_destroy(cache)
    pd.pd_layer_destroy(layer)


@pytest.mark.parametrize("n,repeats", [(3, 5), (120, 4), (400, 3), (300, 1)])
def test_last_length_of_a_repeated_slot_holds(n, repeats):
    """Lengths set with every slot listed several times, in other orders: the device's lengths, seen in where a step
    appends, are the host's, the last ones listed."""
    gl = GpuLayer(CFG, I.layer_weights(CFG, std=0.05))
    gc = gl.cache(n, 64)
    rng = torch.Generator().manual_seed(n)
    slots = [int(s) for _ in range(repeats) for s in torch.randperm(n, generator=rng)]
    lens = [int(v) for v in torch.randint(0, 64, (len(slots),), generator=rng)]
    pd.pd_kv_cache_set_lens(gc, slots, lens)
    want = dict(zip(slots, lens))
    assert all(pd.pd_kv_cache_len(gc, s) == want[s] for s in range(n))
    x = torch.randn((n, CFG["d_model"]), device="cuda").to(torch.bfloat16)
    pd.pd_decode_step(gl.h, x, list(range(n)), gc, torch.empty_like(x))
    for s in range(n):
        k = torch.empty((2, 64, 128), dtype=torch.bfloat16, device="cuda")
        pd.pd_kv_cache_get(gc, s, k, torch.empty_like(k))
        filled = (k != 0).any(2).any(0).nonzero().flatten().tolist()        # a new cache is zero
        assert filled == [want[s]]
    gl.close()
