"""Products of more than 256 rows: every tile form, with the form that a size takes stated and asserted, ragged last
row and column tiles, one row over a tile.  Codes (plain store): all four forms, with and without a K split.  bf16,
plain store (head products, which have no scratch to split with): all four forms.  bf16 and codes, SwiGLU and residual
epilogues: the forms of test_layer_epilogues; splits of the wide forms in bf16 layers are with the full-shape tests,
grouped products with the mixture-of-experts tests."""
import numpy as np
import pytest
import torch

import paper_2603_04716_amd as pd
import pd_inputs as I
from oracle import layer as O
from gpu_util import GpuLayer, TOL, layer_plans, relmax, tile_plan, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K,form", [(257, 1040, 1536, "deep/split"), (300, 28672, 256, "deep"), (771, 6144, 256, "deep"),
                                        (513, 528, 2048, "deep/split"), (512, 28672, 256, "pair"), (1000, 4096, 1536, "deep"),
                                        (770, 4112, 3072, "deep"), (385, 272, 14336, "deep/split"), (1300, 3088, 512, "pair"),
                                        (1000, 2064, 6144, "pair/split"), (1300, 6160, 1024, "192"), (1300, 3088, 12288, "192/split"),
                                        (1025, 12288, 1024, "256"), (1000, 4112, 12288, "256/split")])
def test_codes_product(M, N, K, form):
    """Bound: one rounding to bf16, 2^-9 of an element, and the order of the fp32 sums; 2^-8 of the row's largest output."""
    assert tile_plan(M, N, K // 2, scratch=8 * 256 * N + M * N) == form
    rng = np.random.default_rng(M + N)
    a, b = (rng.integers(0, 256, s, dtype=np.uint8) & 0xB7 for s in ((M, K), (N, K)))
    sa = (2.0 ** rng.integers(-6, 2, M)).astype(np.float32)
    sb = (2.0 ** rng.integers(-6, 2, N)).astype(np.float32)
    out = torch.empty(M, N, dtype=torch.bfloat16, device="cuda")
    pd.pd_gemm_e4m3(torch.from_numpy(a).cuda(), torch.from_numpy(sa).cuda(), torch.from_numpy(b).cuda(),
                    torch.from_numpy(sb).cuda(), out)
    got = out.float().cpu().numpy()
    rows = np.unique(np.r_[0, M - 1, M // 2, 255, 256, rng.choice(M, 12)])
    ref = O.gemm_e4m3(a[rows], sa[rows], b, sb)
    assert max(relmax(got[r], ref[j]) for j, r in enumerate(rows)) <= 2.0 ** -8


@pytest.mark.parametrize("T,d,V,form", [(257, 1536, 1040, "deep"), (771, 256, 6144, "pair"), (513, 2048, 528, "deep"), (300, 256, 28672, "deep"),
                                        (700, 256, 12304, "deep"), (385, 256, 8208, "pair"), (513, 512, 14336, "192"),
                                        (385, 512, 28672, "256")])
def test_bf16_product(T, d, V, form):
    assert tile_plan(T, V, d) == form
    hw = I.head_weights(d, V, seed=d + V, dtype="bf16", std=0.05)
    dev = {k: to_dev(v, "bf16") for k, v in hw.items()}
    h = pd.pd_head_create(d, V, 1e-6, "bf16", dev["g_final"], dev["w_lm"], None, T)
    x = I.hidden(T, d, seed=T, dtype="bf16")
    logits = torch.empty((T, V), dtype=torch.bfloat16, device="cuda")
    pd.pd_lm_head(h, to_dev(x, "bf16"), logits)
    torch.cuda.synchronize()
    rows = np.unique(np.r_[0, T - 1, T // 2, 255, 256])
    ref = O.lm_head(x[rows], hw["g_final"], hw["w_lm"])
    got = to_np(logits)[rows]
    assert max(relmax(got[j], ref[j]) for j in range(len(rows))) <= TOL["bf16"]
    pd.pd_head_destroy(h)


@pytest.mark.parametrize("a8", [False, True])
@pytest.mark.parametrize("d,d_ff,rows,forms", [
    (256, 14336, 257, ["deep", "deep/split", "deep", "deep/split"]), (256, 14336, 300, ["deep", "deep/split", "deep", "deep/split"]),
    (256, 14336, 385, ["deep", "deep/split", "pair", "deep/split"]), (256, 14336, 513, ["deep", "deep/split", "pair", "deep/split"]),
    (512, 14336, 257, ["deep", "deep/split", "192", "deep/split"]), (512, 14336, 385, ["deep", "deep/split", "256", "deep/split"]),
    (1536, 256, 257, ["deep/split", "deep/split", "deep/split", "deep"]), (1536, 640, 300, ["deep/split", "deep/split", "deep/split", "deep"])])
def test_layer_epilogues(a8, d, d_ff, rows, forms):
    """Forms of QKV, O, gate / up (SwiGLU) and down (residual) of a bf16 layer.  A wide FFN (28672 gate / up columns) beside narrow
    products, and a long K; the bound with 8-bit activations is the one derived for the layer (6e-2)."""
    cfg = I.small_config(dtype="bf16", d_model=d, n_q_heads=4, n_kv_heads=2, head_dim=128, d_ff=d_ff)
    if not a8:
        assert layer_plans(cfg, rows) == forms
    w = I.layer_weights(cfg, std=0.05)
    ol, gl = O.Layer(cfg, O.quantise_layer_weights(w) if a8 else w), GpuLayer(cfg, w, a8=a8)
    x = I.hidden(rows, cfg["d_model"], seed=rows, dtype="bf16")
    cu = np.array([0, rows // 3, rows], np.int32)
    assert relmax(gl.prefill(x, cu), O.prefill(ol, x, cu, act8=a8)) <= (6e-2 if a8 else TOL["bf16"])
    gl.close()
