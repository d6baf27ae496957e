"""fp32 layers on the fp32 matrix instructions and the split attention: tile edges, K that is not a multiple of
the 16-wide k-step, both tile sizes, every head size with its own form, one and four waves per attention row.
Bound: the fp32 bound of the other parity tests, 1e-5 of the largest element."""
import ctypes as C

import numpy as np
import pytest
import torch

import paper_2603_04716_amd as pd
import pd_inputs as I
from oracle import layer as O
from gpu_util import GpuLayer, TOL, relmax, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [[1], [15], [17, 1], [33], [65, 64], [300, 401]])
@pytest.mark.parametrize("cfg", [
    I.small_config(d_model=100, d_ff=516),                                    # K = 100: a last k-step of 4
    I.small_config(d_model=516, n_q_heads=8, n_kv_heads=2, head_dim=64, d_ff=260),
    I.small_config(d_model=64, n_q_heads=2, n_kv_heads=1, head_dim=128, d_ff=64),
    I.small_config(d_model=64, n_q_heads=1, n_kv_heads=1, head_dim=256, d_ff=68),
    I.small_config(d_model=96, d_ff=132, n_experts=5, top_k=2),
], ids=["k100", "k516_hd64", "hd128", "hd256", "moe"])
def test_prefill_then_decode(cfg, rows):
    w = I.layer_weights(cfg, std=0.05)
    ol, gl = O.Layer(cfg, w), GpuLayer(cfg, w)
    cu = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    n, cap = len(rows), max(rows) + 2
    slots = list(range(n))
    oc, gc = O.KVCache(ol, n, cap), gl.cache(n, cap)
    rl = I.router_logits(int(cu[-1]), cfg["n_experts"], seed=5) if cfg["n_experts"] else None
    x = I.hidden(int(cu[-1]), cfg["d_model"], seed=21)
    assert relmax(gl.prefill(x, cu, gc, slots, rl), O.prefill(ol, x, cu, rl, cache=oc, slots=slots)) <= TOL["f32"]
    for step in range(2):
        xn = I.hidden(n, cfg["d_model"], seed=30 + step)
        rn = None if rl is None else I.router_logits(n, cfg["n_experts"], seed=40 + step)
        assert relmax(gl.decode(xn, slots, gc, rn), O.decode_step(ol, xn, slots, oc, rn)) <= TOL["f32"]
    gl.close()


@pytest.mark.parametrize("head_dim", [64, 128])
def test_unseen_keys_do_not_reach_a_query(head_dim):
    """A token that is not finite leaves every earlier row of its sequence, and every other sequence, as it was."""
    cfg = I.small_config(d_model=64, n_q_heads=2, n_kv_heads=1, head_dim=head_dim, d_ff=64)
    gl = GpuLayer(cfg, I.layer_weights(cfg, std=0.05))
    cu = np.array([0, 40, 60], np.int32)
    x = I.hidden(60, cfg["d_model"], seed=3)
    want = gl.prefill(x, cu)
    x[21] = np.inf
    got = gl.prefill(x, cu)
    clean = np.r_[0:21, 40:60]
    assert np.array_equal(got[clean], want[clean]) and not np.isfinite(got[21:40]).any()
    gl.close()


@pytest.mark.parametrize("head_dim", [32, 64, 128, 256])
@pytest.mark.parametrize("lost", [(0, 64), (64, 128), (192, 256), (64, 300)])
def test_decode_with_keys_of_score_minus_infinity(head_dim, lost):
    """Whole 64-key chunks whose scores are all -infinity (the first that a wave sees among them) have no weight."""
    cfg = I.small_config(d_model=64, n_q_heads=2, n_kv_heads=1, head_dim=head_dim, d_ff=64)
    w = I.layer_weights(cfg, std=0.05)
    w["w_q"] = np.abs(w["w_q"])                      # with inputs > 0 every query channel is positive, also once the
    x = np.abs(I.hidden(1, 64, seed=4)) + 0.1        # slowest pair (hd / 2 - 1 and hd - 1) is turned by under 0.06
    ol, gl = O.Layer(cfg, w), GpuLayer(cfg, w)
    k, v = I.kv_fill(1, 300, head_dim, seed=6)
    k[:, lost[0]:lost[1], head_dim // 2 - 1] = -np.inf
    oc, gc = O.KVCache(ol, 1, 301), gl.cache(1, 301)
    oc.set(0, k, v)
    pd.pd_kv_cache_set(gc, 0, to_dev(k, "f32"), to_dev(v, "f32"))
    assert relmax(gl.decode(x, [0], gc), O.decode_step(ol, x, [0], oc)) <= TOL["f32"]
    gl.close()


@pytest.mark.parametrize("head_dim", [64, 128, 256])
@pytest.mark.parametrize("lost", [(16, 32), (48, 64), (16, 80)])
def test_prefill_with_keys_of_score_minus_infinity(head_dim, lost):
    """The same for 16-key tiles: the lost tokens' keys overflow to -infinity in the slowest rotary pair."""
    cfg = I.small_config(d_model=64, n_q_heads=2, n_kv_heads=1, head_dim=head_dim, d_ff=64)
    w = I.layer_weights(cfg, std=0.05)
    w["w_q"] = np.abs(w["w_q"])
    w["w_k"][head_dim // 2 - 1, 0] = -3e38
    x = np.abs(I.hidden(100, 64, seed=4)) + 0.1
    x[:, 0] = 0.0
    x[lost[0]:lost[1], 0] = 4.0                      # more than 1.2 after the norm: the product leaves fp32
    ol, gl = O.Layer(cfg, w), GpuLayer(cfg, w)
    cu = np.array([0, 100], np.int32)
    assert relmax(gl.prefill(x, cu), O.prefill(ol, x, cu)) <= TOL["f32"]
    gl.close()


def test_product_of_more_rows_than_a_grid_holds_tiles():
    """2.1 million rows: more 32-row tiles than a grid dimension holds."""
    T, d, V = 65535 * 32 + 33, 4, 16
    gen = torch.Generator(device="cuda").manual_seed(1)
    x, w = torch.randn((T, d), device="cuda", generator=gen), torch.randn((V, d), device="cuda", generator=gen)
    g = torch.ones(d, device="cuda")
    head = pd.pd_head_create(d, V, 1e-6, "f32", g, w, None, T)
    got = torch.full((T, V), float("nan"), device="cuda")
    pd.pd_lm_head(head, x, got)
    xd = x.double()
    ref = (xd * torch.rsqrt(xd.square().mean(1, keepdim=True) + 1e-6)) @ w.double().T
    assert float((got - ref).abs().max() / ref.abs().max()) <= TOL["f32"]
    pd.pd_head_destroy(head)


def test_chunk_attention_of_more_items_than_workgroups_fit_a_launch():
    """4096 chunks of 65 rows with 64 heads: 17.0 million (row, head) items, more than 2^32 threads of a workgroup each.
    Single sequences of it, fed alone, take the other form."""
    n, L = 4096, 65
    cfg = I.small_config(d_model=4, n_q_heads=64, n_kv_heads=1, head_dim=32, d_ff=4)
    gl = GpuLayer(cfg, I.layer_weights(cfg, std=0.5))
    x = I.hidden(n * L, 4, seed=9)
    all_, alone = gl.cache(n, L), gl.cache(1, L)
    got = gl.prefill_chunk(x, np.arange(0, n * L + 1, L), list(range(n)), all_)
    for s in (0, 1, 2047, n - 1):
        rows = slice(s * L, (s + 1) * L)
        pd.pd_kv_cache_set_len(alone, 0, 0)
        assert relmax(got[rows], gl.prefill_chunk(x[rows], [0, L], [0], alone)) <= TOL["f32"]
    gl.close()


def _split(hd, rows, hq, hkv, mean, longest, share=0):
    return bool(pd.lib.pd_internal_attn_split_pays(hd, rows, hq, hkv, C.c_double(mean), longest, share))


def test_split_attention_where_it_pays():
    """Sizes on both sides, each measured with both forms: a wave per item for many items with few keys or shared ones."""
    assert _split(64, 4, 4, 4, 100, 100) and _split(64, 16, 4, 4, 200, 200) and _split(128, 256, 16, 4, 1000, 1000)
    assert _split(256, 256, 4, 4, 200, 200) and _split(32, 4096, 8, 2, 200, 200) and _split(64, 2048, 4, 4, 1024.5, 2048, 1)
    assert not _split(64, 4096, 4, 4, 6, 6) and not _split(128, 256, 16, 4, 31, 31) and not _split(256, 1024, 4, 1, 65, 65)
    assert not _split(128, 2048, 16, 4, 1024.5, 2048, 1) and not _split(32, 1024, 8, 2, 2, 2) and not _split(64, 1, 4, 4, 2, 2)


@pytest.mark.parametrize("head_dim", [32, 64, 128, 256])
@pytest.mark.parametrize("B,keys,split", [(1, 2, False), (1, 400, True), (700, 3, False), (40, 130, True)])
def test_decode_on_both_sides_of_the_choice(head_dim, B, keys, split):
    """Ragged lengths up to `keys`; sampled rows where there are many."""
    cfg = I.small_config(d_model=64, n_q_heads=4, n_kv_heads=2, head_dim=head_dim, d_ff=64)
    lens = np.random.default_rng(B).integers(max(1, keys // 2), keys, B)
    assert _split(head_dim, B, 4, 2, float(lens.mean()) + 1, int(lens.max()) + 1) == split
    w = I.layer_weights(cfg, std=0.05)
    ol, gl = O.Layer(cfg, w), GpuLayer(cfg, w)
    k, v = I.kv_fill(2, keys, head_dim, seed=7)
    kd, vd = to_dev(k, "f32"), to_dev(v, "f32")
    oc, gc = O.KVCache(ol, B, keys + 1), gl.cache(B, keys + 1)
    for s, n in enumerate(lens):
        oc.set(s, k[:, :n], v[:, :n])
        pd.pd_kv_cache_set(gc, s, kd[:, :n].contiguous(), vd[:, :n].contiguous())
    x = I.hidden(B, 64, seed=8)
    assert relmax(gl.decode(x, list(range(B)), gc), O.decode_step(ol, x, list(range(B)), oc)) <= TOL["f32"]
    gl.close()


def _tiles(hd, hq, lens):
    return bool(pd.lib.pd_internal_attn_tiles_pay(hd, hq, len(lens), (C.c_int32 * len(lens))(*lens)))


def test_tiled_attention_where_it_pays():
    """Sizes on both sides, each measured with both forms: a wave per item for short sequences, alone or by the thousand."""
    assert _tiles(64, 4, [96] * 4) and _tiles(128, 16, [16] * 1000) and _tiles(256, 4, [1500] * 2) and _tiles(128, 64, [2000] + [3] * 500)
    assert _tiles(64, 4, [40]) and _tiles(128, 16, [100]) and _tiles(128, 16, [30] * 256)
    assert not _tiles(64, 16, [1] * 4096) and not _tiles(128, 16, [3] * 1000) and not _tiles(256, 4, [10] * 1000)
    assert not _tiles(64, 4, [1]) and not _tiles(128, 64, [100] + [1] * 1000)


@pytest.mark.parametrize("head_dim", [64, 128, 256])
@pytest.mark.parametrize("lens,tiled", [([300] + [1, 0, 2] * 20, True), ([120, 3, 0, 40], True), ([2] * 300, False)])
def test_prefill_on_both_sides_of_the_choice(head_dim, lens, tiled):
    """Also tiles in an odd grid: 300 rows have 19, 120 rows 8, which become 9."""
    assert _tiles(head_dim, 4, lens) == tiled
    cfg = I.small_config(d_model=64, n_q_heads=4, n_kv_heads=2, head_dim=head_dim, d_ff=64)
    w = I.layer_weights(cfg, std=0.05)
    ol, gl = O.Layer(cfg, w), GpuLayer(cfg, w)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    x = I.hidden(int(cu[-1]), 64, seed=8)
    assert relmax(gl.prefill(x, cu), O.prefill(ol, x, cu)) <= TOL["f32"]
    gl.close()


def test_time_of_a_long_sequence_among_short_ones():
    """256 + 800 x 2 rows (16 tiles per head, all but one of a short sequence empty) against 272 + 800 x 2 (17 tiles): the
    tiles of the short sequences are spread over the chip in both."""
    cfg = I.small_config(d_model=64, n_q_heads=16, n_kv_heads=4, head_dim=128, d_ff=64)
    gl = GpuLayer(cfg, I.layer_weights(cfg, std=0.05))

    def ms(lens):
        cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
        x, best = torch.zeros((int(cu[-1]), 64), device="cuda"), 1e9
        y = torch.empty_like(x)
        for _ in range(5):
            pd.pd_profile_enable(gl.h, True)
            pd.pd_prefill(gl.h, x, cu, y)
            best = min(best, dict(pd.pd_profile_read(gl.h))["prefill_attention"])
        return best

    assert ms([256] + [2] * 800) <= 2 * ms([272] + [2] * 800)
    gl.close()


@pytest.mark.parametrize("T,d", [(2016, 64), (1984, 64), (2016, 68)])
def test_products_with_a_short_k(T, d):
    """Beside the line between the plain form (K up to 64, from 2048 tiles on) and the matrix form: 63 x 33 and 62 x 33 tiles."""
    V = 1050
    gen = torch.Generator(device="cuda").manual_seed(d)
    x, w = torch.randn((T, d), device="cuda", generator=gen), torch.randn((V, d), device="cuda", generator=gen)
    head = pd.pd_head_create(d, V, 1e-6, "f32", torch.ones(d, device="cuda"), w, None, T)
    got = torch.full((T, V), float("nan"), device="cuda")
    pd.pd_lm_head(head, x, got)
    xd = x.double()
    ref = (xd * torch.rsqrt(xd.square().mean(1, keepdim=True) + 1e-6)) @ w.double().T
    assert float((got - ref).abs().max() / ref.abs().max()) <= TOL["f32"]
    pd.pd_head_destroy(head)
