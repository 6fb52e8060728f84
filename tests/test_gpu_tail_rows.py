"""Where the tail's first operand comes from: one token per sequence, up to eight of them (the last down product leaves it), more (the norm
in front of the fused K/V projection does), and either with an early-exit head, which reads the same rows first: no row takes its logits, or
every row does."""
import pytest
import torch

import workloads as WL
from oracle import swiftkv_oracle as O
from workloads.configs import ModelShape, Workload
from tests import gpu_helpers as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("early_exit", [False, True])
@pytest.mark.parametrize("lens", [[1] * 8, [1] * 9, [1] * 90, [1, 2] * 3, [70, 1, 30, 2]], ids=lambda v: f"{len(v)}x{max(v)}")
def test_first_operand_of_the_tail(lens, early_exit):
    from paper_2410_03960_amd import binding as B
    shape = ModelShape(4, 1024, 8, 4, 128, 2048, 512, 5e5, 1e-5)
    wl = Workload("tail_rows", shape, l=2, g=1, seed=3111)
    store = WL.make_weights(wl, "cpu", keep=True)
    batch = WL.build_batch(wl, lens=lens, shuffled=True)
    ctx = B.Context(shape, G.device_weights(store), 2, 1)
    if early_exit:
        gen = torch.Generator().manual_seed(5)
        gain, head = torch.ones(1024).bfloat16(), (0.01 * torch.randn(512, 1024, generator=gen)).bfloat16()
        ctx.set_early_exit(gain.cuda(), head.cuda(), 1.5)      # no probability exceeds it
    logits, cache, _ = G.run_gpu(ctx, batch)
    ologits, ocache, _ = G.run_oracle(shape, store, batch, 2, 1)
    G.compare_caches(cache, ocache, batch, label=wl.name)
    G.compare_logits(logits, ologits, label=wl.name)


@pytest.mark.parametrize("lens", [[1] * 8, [1] * 9, [1] * 90, [70, 1, 30, 2]], ids=lambda v: f"{len(v)}x{max(v)}")
def test_operand_of_the_early_exit_head(lens):
    """Every row exits, so the logits are the extra head's, whose operand comes the same ways; a gain that is not one."""
    from paper_2410_03960_amd import binding as B
    shape = ModelShape(4, 1024, 8, 4, 128, 2048, 512, 5e5, 1e-5)
    wl = Workload("tail_rows", shape, l=2, g=1, seed=3111)
    store = WL.make_weights(wl, "cpu", keep=True)
    batch = WL.build_batch(wl, lens=lens, shuffled=True)
    gen = torch.Generator().manual_seed(6)
    gain, head = (1 + 0.3 * torch.randn(1024, generator=gen)).bfloat16(), (0.05 * torch.randn(512, 1024, generator=gen)).bfloat16()
    ctx = B.Context(shape, G.device_weights(store), 2, 1)
    ctx.set_early_exit(gain.cuda(), head.cuda(), -1.0)         # every row's largest probability exceeds it
    logits, _, ws = G.run_gpu(ctx, batch)
    assert ctx.export_exit_flags(ws, len(lens)).cpu().bool().all()
    cache = O.PagedKVCache(ctx.n_cache_layers, batch.n_blocks, 4, 128, batch.block_tables)
    ologits, _, flags = O.swiftkv_prefill(G.oracle_shape(shape), G.weight_fn(store), batch.token_ids, batch.seq_lens.tolist(),
                                          batch.context_lens.tolist(), 2, 1, cache, early_exit=(gain.double(), head.double(), -1.0))
    assert all(flags)
    G.compare_logits(logits, ologits, label=wl.name)
