"""Tiled rotary embedding + cache write of a prefill: sequences that end on, before and behind a 64-position tile,
chunks that start anywhere in one, every cache form (blocked, 8-bit with power-of-two and other scales, plain, none),
positions past the rotary table.  Outputs, stored keys and values against the oracle."""
import numpy as np
import pytest
import torch

import paper_2603_04716_amd as pd
import pd_inputs as I
from oracle import layer as O
from gpu_util import GpuLayer, TOL, relmax, to_dev, to_np

pytestmark = pytest.mark.gpu

CFG = I.small_config(dtype="bf16", d_model=128, n_q_heads=4, n_kv_heads=2, head_dim=128, d_ff=128)
PLAIN = I.small_config(dtype="bf16", d_model=128, n_q_heads=20, n_kv_heads=1, head_dim=128, d_ff=128)


def _check_cache(gl, gc, oc, slots, scales):
    for s in slots:
        n = pd.pd_kv_cache_len(gc, s)
        k = torch.empty((oc.k.shape[1], n, 128), dtype=torch.bfloat16, device="cuda")
        v = torch.empty_like(k)
        pd.pd_kv_cache_get(gc, s, k, v)
        torch.cuda.synchronize()
        for got, ref, scale in ((to_np(k), oc.k[s, :, :n], 0), (to_np(v), oc.v[s, :, :n], 1)):
            slack = TOL["bf16"] * np.max(np.abs(ref))
            if scales:                               # the neighbouring code: one spacing
                mag = np.maximum(np.maximum(np.abs(ref), np.abs(got)) / scales[scale], 2.0 ** -6)
                slack = slack + scales[scale] * 2.0 ** (np.floor(np.log2(mag)) - 3)
            assert np.all(np.abs(got - ref) <= slack)


@pytest.mark.parametrize("form", ["bf16", "fp8", "fp8_odd", "plain", "none"])
@pytest.mark.parametrize("lens", [[1], [7, 64, 9], [63, 65], [200, 1, 130]])
def test_prefill(form, lens):
    cfg = PLAIN if form == "plain" else CFG
    w = I.layer_weights(cfg, std=0.05)
    ol, gl = O.Layer(cfg, w), GpuLayer(cfg, w)
    scales = {"fp8": (0.5, 0.125), "fp8_odd": (0.3, 0.07)}.get(form)
    n = len(lens)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    slots = list(range(n))[::-1]
    x = I.hidden(int(cu[-1]), cfg["d_model"], seed=5, dtype="bf16")
    if form == "none":
        assert relmax(gl.prefill(x, cu), O.prefill(ol, x, cu)) <= TOL["bf16"]
    else:
        oc, gc = O.KVCache(ol, n, 260, fp8_scales=scales), gl.cache(n, 260, fp8_scales=scales)
        assert relmax(gl.prefill(x, cu, gc, slots), O.prefill(ol, x, cu, cache=oc, slots=slots)) <= TOL["bf16"]
        _check_cache(gl, gc, oc, slots, scales)
    gl.close()


@pytest.mark.parametrize("form", ["bf16", "fp8", "plain"])
@pytest.mark.parametrize("prefix,lens", [([0, 5], [20, 9]), ([63, 64], [66, 70]), ([100, 33], [9, 150]), ([3, 70], [40, 24]),
                                         ([3, 70], [40, 25]), ([1, 60], [200, 56]), ([1, 60], [200, 57])])
def test_chunk(form, prefix, lens):
    """What the slots hold behind a chunk's start stays as it was, except for the chunk's own positions.  Up to 64 rows
    (8-bit cache: 256) are rotated row by row, more by tiles."""
    cfg = PLAIN if form == "plain" else CFG
    w = I.layer_weights(cfg, std=0.05)
    ol, gl = O.Layer(cfg, w), GpuLayer(cfg, w)
    scales = (0.5, 0.125) if form == "fp8" else None
    cap = 300
    oc, gc = O.KVCache(ol, 2, cap, fp8_scales=scales), gl.cache(2, cap, fp8_scales=scales)
    for s in range(2):
        k, v = I.kv_fill(cfg["n_kv_heads"], cap, 128, seed=s, dtype="bf16")
        oc.set(s, k, v)
        pd.pd_kv_cache_set(gc, s, to_dev(k, "bf16"), to_dev(v, "bf16"))
        oc.lens[s] = prefix[s]
        pd.pd_kv_cache_set_len(gc, s, prefix[s])
    cu = np.array([0, lens[0], sum(lens)], np.int32)
    x = I.hidden(int(cu[-1]), cfg["d_model"], seed=6, dtype="bf16")
    assert relmax(gl.prefill_chunk(x, cu, [0, 1], gc), O.prefill_chunk(ol, x, cu, [0, 1], oc)) <= TOL["bf16"]
    for s in range(2):
        pd.pd_kv_cache_set_len(gc, s, cap)
    _check_cache(gl, gc, oc, [0, 1], scales)
    gl.close()


def test_chunk_past_the_rotary_table():
    ol, gl = (lambda w: (O.Layer(CFG, w), GpuLayer(CFG, w)))(I.layer_weights(CFG, std=0.05))
    n, rows = 32760, 20                              # positions 32760 .. 32779; the table ends at 32767
    oc, gc = O.KVCache(ol, 1, n + rows), gl.cache(1, n + rows)
    k, v = I.kv_fill(2, n, 128, seed=9, dtype="bf16")
    oc.set(0, k, v)
    pd.pd_kv_cache_set(gc, 0, to_dev(k, "bf16"), to_dev(v, "bf16"))
    x = I.hidden(rows, CFG["d_model"], seed=7, dtype="bf16")
    cu = np.array([0, rows], np.int32)
    assert relmax(gl.prefill_chunk(x, cu, [0], gc), O.prefill_chunk(ol, x, cu, [0], oc)) <= TOL["bf16"]
    _check_cache(gl, gc, oc, [0], None)
    gl.close()


def _stored_keys(gc, slots, n_kv_heads, n):
    k = torch.empty((len(slots), n_kv_heads, n, 128), dtype=torch.bfloat16, device="cuda")
    for i, s in enumerate(slots):
        pd.pd_kv_cache_get(gc, s, k[i], torch.empty_like(k[i]))
    torch.cuda.synchronize()
    return k.view(torch.int16)


def test_a_key_has_the_same_bits_whichever_call_brings_it():
    """The same rows (so the same projections: neither product depends on how rows are grouped into sequences) at the
    same positions, rotated by tiles (prefill, longer chunks), row by row (chunks of a few tokens) and in the append
    of a decode step: every stored key is the same bit pattern, 131072 and 32768 pairs of channels."""
    cfg = I.small_config(dtype="bf16", d_model=128, n_q_heads=32, n_kv_heads=32, head_dim=128, d_ff=128)
    gl = GpuLayer(cfg, I.layer_weights(cfg, std=0.05))
    n, L = 8, 8
    x = I.hidden(n * L, cfg["d_model"], seed=3, dtype="bf16")
    cu, slots = np.arange(0, n * L + 1, L).astype(np.int32), list(range(n))
    tiled, rows = gl.cache(n, 64), gl.cache(n, 64)
    gl.prefill(x, cu, tiled, slots)
    gl.prefill_chunk(x, cu, slots, rows)
    assert torch.equal(_stored_keys(tiled, slots, 32, L), _stored_keys(rows, slots, 32, L))

    p = 50                                           # a chunk of 16 rows at positions 50 .. 65 and 16 slots of one row each
    x = x[:16]
    chunk, steps = gl.cache(1, 128), gl.cache(16, 128)
    for s in range(16):
        pd.pd_kv_cache_set_len(steps, s, p + s)
    pd.pd_kv_cache_set_len(chunk, 0, p)
    gl.prefill_chunk(x, np.array([0, 16], np.int32), [0], chunk)
    gl.decode(x, list(range(16)), steps)
    want, got = _stored_keys(chunk, [0], 32, p + 16)[0], _stored_keys(steps, list(range(16)), 32, p + 16)
    for s in range(16):
        assert torch.equal(got[s, :, p + s], want[:, p + s])
    gl.close()


def _many(n, long, seed):
    """One long sequence somewhere among n - 1 of 0 .. 5 rows."""
    lens = np.random.default_rng(seed).integers(0, 6, n)
    lens[n // 3] = long
    return [int(v) for v in lens]


@pytest.mark.parametrize("form,n,long", [("bf16", 63, 300), ("fp8", 64, 300), ("bf16", 65, 700), ("fp8_odd", 130, 700),
                                         ("none", 1000, 1500), ("none", 4096, 130), ("bf16", 300, 5), ("fp8", 300, 40)])
def test_prefill_of_many_sequences(form, n, long):
    """A long prompt among many short ones (tiles found by search, in one and two rounds of 64 sequences), and short
    ones only."""
    ol, gl = (lambda w: (O.Layer(CFG, w), GpuLayer(CFG, w)))(I.layer_weights(CFG, std=0.05))
    scales = {"fp8": (0.5, 0.125), "fp8_odd": (0.3, 0.07)}.get(form)
    lens = _many(n, long, n)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    x = I.hidden(int(cu[-1]), CFG["d_model"], seed=5, dtype="bf16")
    if form == "none":
        assert relmax(gl.prefill(x, cu), O.prefill(ol, x, cu)) <= TOL["bf16"]
    else:
        slots = list(range(n))[::-1]
        oc, gc = O.KVCache(ol, n, long, fp8_scales=scales), gl.cache(n, long, fp8_scales=scales)
        assert relmax(gl.prefill(x, cu, gc, slots), O.prefill(ol, x, cu, cache=oc, slots=slots)) <= TOL["bf16"]
        _check_cache(gl, gc, oc, [s for s in slots if pd.pd_kv_cache_len(gc, s)], scales)
    gl.close()


@pytest.mark.parametrize("form,long", [("bf16", 260), ("fp8", 260), ("fp8", 900)])
def test_chunk_of_many_sequences(form, long):
    """8-bit cache: row by row up to 10 rows per sequence on the average, by tiles that are searched beyond."""
    ol, gl = (lambda w: (O.Layer(CFG, w), GpuLayer(CFG, w)))(I.layer_weights(CFG, std=0.05))
    scales = (0.5, 0.125) if form == "fp8" else None
    n, cap = 90, 1050
    rng = np.random.default_rng(2)
    prefix, lens = rng.integers(0, 140, n), np.array(_many(n, long, 7))
    oc, gc = O.KVCache(ol, n, cap, fp8_scales=scales), gl.cache(n, cap, fp8_scales=scales)
    for s in range(n):
        k, v = I.kv_fill(2, 140, 128, seed=s, dtype="bf16")
        oc.set(s, k, v)
        pd.pd_kv_cache_set(gc, s, to_dev(k, "bf16"), to_dev(v, "bf16"))
        oc.lens[s] = prefix[s]
        pd.pd_kv_cache_set_len(gc, s, int(prefix[s]))
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    slots = [int(s) for s in rng.permutation(n)]
    x = I.hidden(int(cu[-1]), CFG["d_model"], seed=6, dtype="bf16")
    assert relmax(gl.prefill_chunk(x, cu, slots, gc), O.prefill_chunk(ol, x, cu, slots, oc)) <= TOL["bf16"]
    _check_cache(gl, gc, oc, [s for s in slots if pd.pd_kv_cache_len(gc, s)], scales)
    gl.close()


def test_time_follows_the_rows_not_the_longest_sequence():
    """8192 + 3999 x 4 rows against as many in 24 sequences: the rotation takes a few times as long (64-position tiles of
    4 rows), not the number of sequences times the tiles of the longest (70 times)."""
    cfg = dict(CFG, n_q_heads=32, n_kv_heads=8)
    gl = GpuLayer(cfg, I.layer_weights(cfg, std=0.05))

    def rope_ms(lens):
        cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
        x = torch.zeros((int(cu[-1]), cfg["d_model"]), dtype=torch.bfloat16, device="cuda")
        y, best = torch.empty_like(x), 1e9
        for _ in range(5):
            pd.pd_profile_enable(gl.h, True)
            pd.pd_prefill(gl.h, x, cu, y)
            best = min(best, dict(pd.pd_profile_read(gl.h))["rope_kv_write"])
        return best

    even = rope_ms([1008] * 24)
    assert rope_ms([8192] + [4] * 3999) <= 8 * even
    gl.close()


def test_more_kv_heads_than_half_a_grid_dimension():
    """33000 kv heads, 70 rows behind an empty slot: a chunk (tiled rotation, gather, matrix-core attention) against
    pd_prefill of the same rows (attention of the plain kernels)."""
    d, h = 8, 33000
    cfg = I.small_config(dtype="bf16", d_model=d, n_q_heads=h, n_kv_heads=h, head_dim=128, d_ff=8)
    gen = torch.Generator(device="cuda").manual_seed(5)
    draw = lambda *s, std: torch.empty(s, device="cuda", dtype=torch.bfloat16).normal_(0.0, std, generator=gen)
    w = {"g_attn": torch.ones(d, device="cuda", dtype=torch.bfloat16), "w_q": draw(h * 128, d, std=0.3), "w_k": draw(h * 128, d, std=0.3),
         "w_v": draw(h * 128, d, std=0.3), "w_o": draw(d, h * 128, std=0.001), "g_ffn": torch.ones(d, device="cuda", dtype=torch.bfloat16),
         "w_gate": draw(8, d, std=0.3), "w_up": draw(8, d, std=0.3), "w_down": draw(d, 8, std=0.3)}
    torch.cuda.synchronize()
    layer = pd.pd_layer_create(cfg, w)
    cache = pd.pd_kv_cache_create(layer, 1, 70)
    x = draw(70, d, std=1.0)
    want, got = torch.empty_like(x), torch.empty_like(x)
    pd.pd_prefill(layer, x, [0, 70], want)
    pd.pd_prefill_chunk(layer, x, [0, 70], [0], cache, got)
    torch.cuda.synchronize()
    assert relmax(to_np(got), to_np(want)) <= TOL["bf16"]
    pd.pd_kv_cache_destroy(cache)
    pd.pd_layer_destroy(layer)
