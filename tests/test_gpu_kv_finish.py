"""The pass that finishes Q, K and V of K-split projections stores K and V itself (paged slots, per-token scales, V^T columns): against
the CPU oracle at its edges, next to the calls that keep the separate commit pass."""
import pytest
import torch

import workloads as WL
from oracle import swiftkv_oracle as O
from workloads.configs import ModelShape, Workload
from tests import gpu_helpers as G

pytestmark = pytest.mark.gpu

# heads of 64 and 128; K rows of less than a wave's 1024 columns, and of more (several rounds of one wave for a token's scale)
SHAPES = {
    "narrow": ModelShape(3, 256, 4, 2, 64, 512, 256, 5e5, 1e-5),
    "hd128": ModelShape(3, 512, 8, 4, 128, 512, 256, 5e5, 1e-5),
    "wide": ModelShape(3, 256, 12, 12, 128, 256, 256, 5e5, 1e-5),
    "wider": ModelShape(3, 256, 36, 36, 128, 256, 256, 5e5, 1e-5),   # 4608 columns, past what one wave holds: a token's scale by passes of their own
}


@pytest.mark.parametrize("name,mode", [(n, m) for n in SHAPES for m in ("bf16", "given", "per_token")])
@pytest.mark.parametrize("lens", [[81], [64, 17, 1, 63], [129, 1, 70], [5, 9]])   # 64-token tiles: whole, one token, one short; at most 80 tokens
def test_fresh_prompts_and_single_tokens(name, mode, lens):
    from paper_2410_03960_amd import binding as B
    shape = SHAPES[name]
    wl = Workload("kv_finish_" + name, shape, l=2, g=1, seed=2911)
    store = WL.make_weights(wl, "cpu", keep=True)
    batch = WL.build_batch(wl, lens=lens, shuffled=True)
    ctx = B.Context(shape, G.device_weights(store), 2, 1)
    fp8 = mode != "bf16"
    if mode == "given":   # scales of the size the values have
        cache = B.KVCache(ctx.n_cache_layers, batch.n_blocks, shape.n_kv_heads, shape.head_dim, batch.block_tables, batch.context_lens.tolist(),
                          fp8=True, scale_mode=B.SWIFTKV_SCALE_USE_GIVEN)
        cache.scales.fill_(0.01)
        logits, cache, ws = G.run_gpu(ctx, batch, fp8=True, cache=cache)
        ocache = O.PagedKVCache(ctx.n_cache_layers, batch.n_blocks, shape.n_kv_heads, shape.head_dim, batch.block_tables, fp8=True)
        ocache.scales[:] = 0.01
        ologits, ocache, _ = G.run_oracle(shape, store, batch, 2, 1, fp8=True, compute_scales=False, cache=ocache)
    else:
        logits, cache, ws = G.run_gpu(ctx, batch, fp8=fp8, scale_mode=B.SWIFTKV_SCALE_PER_TOKEN if fp8 else 0)
        ologits, ocache, _ = G.run_oracle(shape, store, batch, 2, 1, fp8=fp8, per_token=fp8)
    G.check_plan(ctx, ws, batch)
    # (a code is up to 1/8 of its value from the next, and the largest one may be the one whose bf16 rounding crossed a boundary)
    G.compare_caches(cache, ocache, batch, label=f"{name} {mode}", **(dict(rel=0.126, cos=G.FP8_COS) if fp8 else {}))
    G.compare_logits(logits, ologits, label=f"{name} {mode}", **(dict(rel=G.FP8_REL, cos=G.FP8_COS) if fp8 else {}))
    if mode == "per_token":   # unused slots keep their zeros: no scale is written past the call's tokens
        used = torch.cat([ocache.slots(b, torch.arange(n)) for b, n in enumerate(lens)])
        mask = torch.ones(cache.scales.shape[-1], dtype=torch.bool)
        mask[used] = False
        assert not cache.scales[:, :, mask.cuda()].any()
