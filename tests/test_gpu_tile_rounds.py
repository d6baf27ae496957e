"""Products of up to 256 rows by their tile forms, the 256 x 128 form of longer K, and launches whose workgroups take
several tiles of C one after another (the requests of the next one start behind the last k-tiles of the one before)."""
import numpy as np
import pytest
import torch

import paper_2603_04716_amd as pd
import pd_inputs as I
from oracle import layer as O
from gpu_util import GpuLayer, TOL, relmax, tile_plan, to_dev, to_np

pytestmark = pytest.mark.gpu


# rows at the edges of the row tiles, columns ending inside a column tile, K of one k-tile and more; 16400 columns and more
# make more tiles than the 256 CUs
@pytest.mark.parametrize("T,V,d,form", [(33, 528, 64, "64"), (64, 4112, 256, "64"), (65, 528, 320, "64"), (129, 4112, 128, "64"),
                                        (129, 6160, 1024, "128x64"), (256, 6160, 1024, "128x64"), (255, 32784, 256, "256x128"),
                                        (256, 32784, 1024, "256x128"), (64, 32784, 1024, "64"), (64, 16400, 2048, "64x128"), (100, 16400, 1088, "deep"),
                                        (771, 6160, 2048, "256x128"), (1025, 6160, 2112, "256x128"), (300, 12304, 2048, "256x128"),
                                        (2100, 12304, 2048, "256"), (1500, 12304, 2048, "192"), (2000, 33040, 320, "256")])
def test_bf16(T, V, d, form):
    assert tile_plan(T, V, d) == form
    hw = I.head_weights(d, V, seed=d + V, dtype="bf16", std=0.05)
    dev = {k: to_dev(v, "bf16") for k, v in hw.items()}
    h = pd.pd_head_create(d, V, 1e-6, "bf16", dev["g_final"], dev["w_lm"], None, T)
    x = I.hidden(T, d, seed=T, dtype="bf16")
    logits = torch.empty((T, V), dtype=torch.bfloat16, device="cuda")
    pd.pd_lm_head(h, to_dev(x, "bf16"), logits)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(logits).all())
    rows = np.unique(np.r_[0, T - 1, T // 2, np.arange(15, T, 64)[:8], np.arange(16, T, 256)[:4]])
    ref = O.lm_head(x[rows], hw["g_final"], hw["w_lm"])
    got = to_np(logits)[rows]
    assert max(relmax(got[j], ref[j]) for j in range(len(rows))) <= TOL["bf16"]
    pd.pd_head_destroy(h)


@pytest.mark.parametrize("M,N,K,form", [(771, 6160, 4096, "256x128"), (1500, 3088, 4096, "256x128"), 
                                        (1500, 16400, 1024, "256"), (1500, 16400, 1152, "256"), (3000, 6160, 1280, "192")])
def test_codes(M, N, K, form):
    """Bound: one rounding to bf16, 2^-9 of an element, and the order of the fp32 sums; 2^-8 of the row's largest output.
    K = 1152 is an odd number of k-tiles, which ends in the other set of weight fragments."""
    assert tile_plan(M, N, K // 2, scratch=8 * 256 * N + M * N, codes=True) == form
    rng = np.random.default_rng(M + N)
    a, b = (rng.integers(0, 256, s, dtype=np.uint8) & 0xB7 for s in ((M, K), (N, K)))
    sa = (2.0 ** rng.integers(-6, 2, M)).astype(np.float32)
    sb = (2.0 ** rng.integers(-6, 2, N)).astype(np.float32)
    out = torch.empty(M, N, dtype=torch.bfloat16, device="cuda")
    pd.pd_gemm_e4m3(torch.from_numpy(a).cuda(), torch.from_numpy(sa).cuda(), torch.from_numpy(b).cuda(),
                    torch.from_numpy(sb).cuda(), out)
    got = out.float().cpu().numpy()
    assert np.isfinite(got).all()
    rows = np.unique(np.r_[0, M - 1, M // 2, np.arange(15, M, 256)])
    ref = O.gemm_e4m3(a[rows], sa[rows], b, sb)
    assert max(relmax(got[r], ref[j]) for j, r in enumerate(rows)) <= 2.0 ** -8


@pytest.mark.parametrize("d,d_ff,T,forms", [(1024, 2816, 40, ["64", "64/split", "64", "64/split"]),
                                            (1024, 2816, 256, ["64", "64/split", "128x64", "64/split"]),
                                            (2048, 5632, 130, ["64/split", "64/split", "deep", "128x64/split"]),
                                            (2048, 5632, 65, ["64/split", "64/split", "128x64", "64/split"])])
def test_layer_of_few_rows(d, d_ff, T, forms):
    """Weights of the benchmark's spread, 0.02: attention scores then have a spread of 128^-1/2 * 128^1/2 * (0.02^2 d) <= 0.8, and
    the bound's six roundings are not amplified.  (With 0.05 and d = 2048 the scores spread over 5, a relative error of 2^-8
    in one is 2 % of its weight, and the tiled kernels of any form are 2.03e-2 off at 130 rows.)"""
    cfg = I.small_config(dtype="bf16", d_model=d, n_q_heads=4, n_kv_heads=2, head_dim=128, d_ff=d_ff)
    scratch = 256 * (640 * 128 + 2 * max(1024, 2 * d_ff, d))
    assert [tile_plan(T, 1024, d, 0, 0, scratch), tile_plan(T, d, 512, 1, 0, scratch, 1), tile_plan(T, d_ff, d, 2, 0, scratch),
            tile_plan(T, d, d_ff, 1, 0, scratch)] == forms
    w = I.layer_weights(cfg, std=0.02)
    ol, gl = O.Layer(cfg, w), GpuLayer(cfg, w)
    x = I.hidden(T, d, seed=T, dtype="bf16")
    cu = np.array([0, T // 3, T], np.int32)
    got, ref = gl.prefill(x, cu), O.prefill(ol, x, cu)
    assert relmax(got, ref) <= TOL["bf16"]
    assert max(relmax(got[i], ref[i]) for i in range(T)) <= 2 * TOL["bf16"]
    gl.close()
