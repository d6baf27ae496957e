"""Helpers for the GPU parity tests: move seeded numpy inputs to the device in the layer's dtype,
call the C ABI through the binding, bring results back as fp32 numpy."""
import ctypes as C

import numpy as np
import torch

import paper_2603_04716_amd as pd
import pd_inputs as I

TOL = {"f32": 1e-5, "bf16": 2e-2}     # max-norm relative error bound per dtype


def to_dev(a, dtype):
    t = torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()
    return t.to(torch.bfloat16).contiguous() if dtype == "bf16" else t.contiguous()


def to_np(t):
    return t.detach().float().cpu().numpy()


def relmax(got, ref):
    """Largest difference over the largest value; infinite where a result is not finite (as NaN it would vanish in max())."""
    got, ref = np.asarray(got, np.float64), np.asarray(ref, np.float64)
    if not np.isfinite(got).all():
        return float("inf")
    return float(np.max(np.abs(got - ref)) / max(np.max(np.abs(ref)), 1e-30))


class GpuLayer:
    def __init__(self, cfg, weights, w8=False, a8=False):
        self.cfg = cfg
        self.dtype = cfg["dtype"]
        self.dev_w = {k: to_dev(v, self.dtype) for k, v in weights.items()}
        self.h = pd.pd_layer_create(cfg, self.dev_w, w8=w8 or a8, a8=a8)
        self.caches = []

    def cache(self, n_slots, max_len, fp8_scales=None):
        if fp8_scales is None:
            c = pd.pd_kv_cache_create(self.h, n_slots, max_len)
        else:
            c = pd.pd_kv_cache_create_fp8(self.h, n_slots, max_len, *fp8_scales)
        self.caches.append(c)
        return c

    def prefill(self, x, cu, cache=None, slots=None, router_logits=None):
        xd = to_dev(x, self.dtype)
        out = torch.empty_like(xd)
        rl = None if router_logits is None else torch.from_numpy(router_logits).cuda().contiguous()
        pd.pd_prefill(self.h, xd, cu, out, cache, slots, rl)
        torch.cuda.synchronize()
        return to_np(out)

    def prefill_chunk(self, x, cu, slots, cache, router_logits=None):
        xd = to_dev(x, self.dtype)
        out = torch.empty_like(xd)
        rl = None if router_logits is None else torch.from_numpy(router_logits).cuda().contiguous()
        pd.pd_prefill_chunk(self.h, xd, cu, slots, cache, out, rl)
        torch.cuda.synchronize()
        return to_np(out)

    def decode(self, x, slots, cache, router_logits=None):
        xd = to_dev(x, self.dtype)
        out = torch.empty_like(xd)
        rl = None if router_logits is None else torch.from_numpy(router_logits).cuda().contiguous()
        pd.pd_decode_step(self.h, xd, slots, cache, out, rl)
        torch.cuda.synchronize()
        return to_np(out)

    def experts(self, rows):
        e = torch.empty((rows, self.cfg["top_k"]), dtype=torch.int32, device="cuda")
        pd.pd_last_expert_choice(self.h, rows, e)
        torch.cuda.synchronize()
        return e.cpu().numpy()

    def close(self):
        for c in self.caches:
            pd.pd_kv_cache_destroy(c)
        pd.pd_layer_destroy(self.h)
        self.caches = []


def tile_plan(M, N, K, epilogue=0, n_groups=0, scratch=0, fused_norm=0, codes=False):
    """"form" or "form/split" of a product: what the library's planner says (host only).  Forms: 256, 192 (x 256 columns),
    pair (128 x 128, two workgroups per CU), deep (128 x 128, alone on its CU), and rows x columns.  Codes: half of K."""
    form, splits = C.c_int(), C.c_int()
    pd.lib.pd_internal_tile_plan(M, N, K, epilogue, n_groups, C.c_longlong(scratch), fused_norm, int(codes), C.byref(form), C.byref(splits))
    return ("256", "192", "pair", "deep", "256x128", "128x64", "64x128", "64")[form.value] + ("/split" if splits.value > 1 else "")


def layer_plans(cfg, T, a8=False):
    """The plans of the four products of a dense layer called with T rows, on the layer's own scratch (256 rows of
    640 x 128 columns and twice the widest weight matrix)."""
    d, f, nq, nkv = cfg["d_model"], cfg["d_ff"], cfg["n_q_heads"] * cfg["head_dim"], cfg["n_kv_heads"] * cfg["head_dim"]
    scratch, w = 256 * (640 * 128 + 2 * max(nq + 2 * nkv, 2 * f, d)), 2 if a8 else 1
    return [tile_plan(T, nq + 2 * nkv, d // w, 0, 0, scratch, codes=a8), tile_plan(T, d, nq // w, 1, 0, scratch, 0 if a8 else 1, a8),
            tile_plan(T, f, d // w, 2, 0, scratch, codes=a8), tile_plan(T, d, f // w, 1, 0, scratch, codes=a8)]
