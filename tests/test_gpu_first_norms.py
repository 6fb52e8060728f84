"""The norms that fetch their rows themselves (from the embedding at the start of a
pass, from the layer-l output at the start of the tail) and the decode rows whose K and
V go to their slots in the pass that finishes them: hidden sizes of 1024, 2048 and one
that is no multiple of 1024, more than 1024 tokens (row factors left to the GEMM) and
few, bf16 and e4m3 caches with given and computed scales; prompts in one call, their
last token in the next, against the oracle's one-shot prefill."""
import pytest
import torch

import workloads as WL
from tests import gpu_helpers as G
from workloads.configs import ModelShape, Workload

pytestmark = pytest.mark.gpu

SHAPES = {
    "d1024": ModelShape(3, 1024, 8, 2, 128, 1024, 512, 1e4, 1e-5),
    "d2048": ModelShape(2, 2048, 8, 4, 64, 1024, 512, 1e4, 1e-5),
    "d1280": ModelShape(2, 1280, 10, 5, 128, 512, 512, 1e4, 1e-5),
}


@pytest.mark.parametrize("name,lens,mode", [
    ("d1024", [3, 40, 1 + 1, 17], "bf16"), ("d2048", [90, 2, 30], "bf16"), ("d1280", [5, 33], "bf16"), ("d1024", [700, 390, 2], "bf16"),
    ("d1024", [64, 9, 20], "given"), ("d2048", [33, 2, 70], "given"), ("d1024", [40, 8], "token"), ("d2048", [600, 520], "given")], ids=str)
def test_prompts_then_one_decode_step(name, lens, mode):
    from oracle import swiftkv_oracle as O
    from paper_2410_03960_amd import binding as B
    print(name, lens, mode, flush=True)
    sh = SHAPES[name]
    wl = Workload(f"first_{name}", sh, l=1, g=1, seed=2510)
    store = WL.make_weights(wl, "cpu", keep=True)
    ctx = B.Context(sh, G.device_weights(store), wl.l, wl.g)
    full = WL.build_batch(wl, lens=lens, shuffled=True)
    n, C, fp8 = len(lens), ctx.n_cache_layers, mode != "bf16"
    kw = dict(fp8=fp8, scale_mode=0 if not fp8 else B.SWIFTKV_SCALE_USE_GIVEN if mode == "given" else B.SWIFTKV_SCALE_PER_TOKEN)
    cache = B.KVCache(C, full.n_blocks, sh.n_kv_heads, sh.head_dim, full.block_tables, [0] * n, **kw)
    ocache = O.PagedKVCache(C, full.n_blocks, sh.n_kv_heads, sh.head_dim, full.block_tables, fp8=fp8, per_token=mode == "token")
    if mode == "given":
        sc = 0.02 + 0.01 * torch.rand((C, 2, sh.n_kv_heads), generator=torch.Generator().manual_seed(3))
        cache.scales.copy_(sc)
        ocache.scales = sc.clone()
    cu = [sum(lens[:b]) for b in range(n + 1)]
    for new, cached in (([m - 1 for m in lens], [0] * n), ([1] * n, [m - 1 for m in lens])):
        part = WL.build_batch(wl, lens=new, ctx=cached, shuffled=True)
        part.block_tables, part.n_blocks = full.block_tables, full.n_blocks
        part.token_ids = torch.cat([full.token_ids[cu[b] + cached[b]:cu[b] + cached[b] + new[b]] for b in range(n)])
        cache.set_context_lens(cached)
        logits, cache, _ = G.run_gpu(ctx, part, fp8=fp8, cache=cache)
    ologits, ocache, _ = G.run_oracle(sh, store, full, wl.l, wl.g, fp8=fp8, compute_scales=False, cache=ocache)
    rel, cos = (G.FP8_REL, G.FP8_COS) if fp8 else (G.BF16_REL, G.BF16_COS)
    # (a value whose bf16 rounding differs may land on the neighbouring e4m3 code: at most 1/8 of the largest value apart)
    G.compare_caches(cache, ocache, full, rel=0.126 if fp8 else rel, cos=cos, label=name)
    G.compare_logits(logits, ologits, rel=rel, cos=cos, label=name)
