"""The e4m3 codes a prefill stores under given scales, bit for bit those of the oracle's
quantiser (division in fp32) on the K/V a bf16 cache holds: saturating and underflowing
scales, both sides of the range in which the division runs as a product with the
reciprocal, a scale at its end; prompts with V^T tiles of all fills."""
import pytest
import torch

import workloads as WL
from oracle import swiftkv_oracle as O
from tests import gpu_helpers as G
from workloads.configs import ModelShape, Workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hd,scales", [
    (128, [0.0137, 0.4, 0.0093, 1.0]), (64, [0.0137, 0.4, 0.0093, 1.0]), (128, [1e-4, 1e-3, 300.0, 2e4]),
    (128, [2.0 ** -60, 2.0 ** 60, 1e-3, 0.5]), (128, [1e-25, 0.01, 1e25, 0.01]), (64, [0.01, 1e-30, 0.01, 3e-39])], ids=str)
def test_codes_are_those_of_the_division(hd, scales):
    from paper_2410_03960_amd import binding as B
    wl = Workload(f"codes{hd}", ModelShape(2, 512, 4, 2, hd, 1024, 512, 1e4, 1e-5), l=1, g=1, seed=2411)
    print(hd, scales, flush=True)
    ctx = B.Context(wl.shape, G.device_weights(WL.make_weights(wl, "cpu", keep=True)), wl.l, wl.g)
    batch = WL.build_batch(wl, lens=[130, 64, 33, 2], shuffled=True)
    _, plain, _ = G.run_gpu(ctx, batch)
    cache = B.KVCache(ctx.n_cache_layers, batch.n_blocks, 2, hd, batch.block_tables, batch.context_lens.tolist(), fp8=True,
                      scale_mode=B.SWIFTKV_SCALE_USE_GIVEN)
    cache.scales.copy_(torch.tensor(scales).view(1, 2, 2).expand_as(cache.scales))
    G.run_gpu(ctx, batch, fp8=True, cache=cache)
    used = torch.cat([torch.as_tensor(batch.block_tables[b, p // 16] * 16 + p % 16).view(1) for b, n in enumerate(batch.seq_lens.tolist()) for p in range(n)]).long()
    for kvsel in (0, 1):     # the first cache layer: its K/V come before anything that reads the quantised values
        x = plain.data[0, kvsel].cpu()[used].float()
        want = O.fp8_quantize(x, torch.tensor(scales[2 * kvsel:2 * kvsel + 2])[None, :, None])
        assert torch.equal(cache.data[0, kvsel].cpu()[used], want), kvsel
