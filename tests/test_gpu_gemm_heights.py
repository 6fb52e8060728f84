"""Parity of the GEMMs between the weight-streaming kernels (80 rows) and many
full rounds of 256-row tiles: every tile height, K splits with each epilogue's
finishing pass, ragged last tiles, packed and row-major weights."""
import sys

import pytest
import torch

import workloads as WL
from workloads.configs import ModelShape, Workload
from tests import gpu_helpers as G
from tests.helpers import rel_err

pytestmark = pytest.mark.gpu

# a long contraction over few output columns: Q/K/V, gate/up, the fused K/V projection and the residual GEMMs all split K
LONG = {
    "hd128": Workload("long_hd128", ModelShape(3, 4096, 4, 2, 128, 512, 512, 1e4, 1e-5), l=1, g=1, seed=2201),
    "hd64": Workload("long_hd64", ModelShape(3, 4096, 8, 4, 64, 512, 512, 1e4, 1e-5), l=2, g=1, seed=2202),
}
# many output columns over a short contraction: the tile height follows the number of rows
BROAD = Workload("broad", ModelShape(2, 256, 32, 8, 128, 3072, 256, 1e4, 1e-5), l=1, g=1, seed=2203)


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def _check(wl, lens, fp8, packed, ctx_lens=None):
    from paper_2410_03960_amd import binding as B
    store = WL.make_weights(wl, "cpu", keep=True)
    ctx = B.Context(wl.shape, G.device_weights(store), wl.l, wl.g, packed_weights=packed)
    batch = WL.build_batch(wl, lens=lens, shuffled=True)
    mode = B.SWIFTKV_SCALE_COMPUTE_ABSMAX if fp8 else 0
    logits, cache, _ = G.run_gpu(ctx, batch, fp8=fp8, scale_mode=mode)
    ologits, ocache, _ = G.run_oracle(wl.shape, store, batch, wl.l, wl.g, dtype=torch.float32, fp8=fp8, compute_scales=True)
    rel, cos = (G.FP8_REL, G.FP8_COS) if fp8 else (G.BF16_REL, G.BF16_COS)
    if fp8:
        assert rel_err(cache.scales.cpu(), ocache.scales) <= 2e-2
    _say(f"  worst cache {G.compare_caches(cache, ocache, batch, rel=rel, cos=cos, label=wl.name)}, "
         f"logits {G.compare_logits(logits, ologits, rel=rel, cos=cos, label=wl.name)}")
    logits2, cache2, _ = G.run_gpu(ctx, batch, fp8=fp8, scale_mode=mode)       # the splits are added in a fixed order
    assert torch.equal(cache.data, cache2.data) and torch.equal(logits, logits2)


@pytest.mark.parametrize("lens", [[81], [60, 37], [129], [160], [200, 133], [600, 424, 1]], ids=str)
@pytest.mark.parametrize("packed", [True, False])
@pytest.mark.parametrize("name", sorted(LONG))
def test_split_k_with_every_epilogue(name, packed, lens):
    _say(f"{name} packed={packed} lens={lens}")
    _check(LONG[name], lens, fp8=lens == [200, 133], packed=packed)


@pytest.mark.parametrize("rows", [1025, 1300, 2000, 2300, 2561])
def test_tile_heights_with_rotating_and_swiglu_epilogues(rows):
    _say(f"rows={rows}")
    lens = [190] * (rows // 190) + ([rows % 190] if rows % 190 else [])
    _check(BROAD, lens, fp8=rows == 2000, packed=True)


@pytest.mark.parametrize("rows", [1025, 2561, 4500])
def test_tile_heights_with_residual_epilogue(rows):
    _say(f"rows={rows}")
    lens = [256] * (rows // 256) + ([rows % 256] if rows % 256 else [])
    _check(LONG["hd128"], lens, fp8=False, packed=True)


def test_many_continuing_rows():
    """More than 80 sequences: the tail (row-major weights of the later layers, LM head) leaves the weight-streaming kernels."""
    _check(LONG["hd128"], [3] * 100 + [2] * 61, fp8=False, packed=True)


@pytest.mark.parametrize("M,N,K", [
    (1025, 512, 256), (1025, 4096, 256), (1025, 6144, 256), (1300, 6144, 256), (2561, 4096, 256), (2000, 6144, 256), (2300, 6144, 256), (1031, 768, 2048)])
def test_packed_gemm_at_every_tile_height(M, N, K):
    from paper_2410_03960_amd import binding as B
    _say(f"M={M} N={N} K={K}")
    A = WL.seeded_normal_bf16(1, f"A{M}{K}", (M, K), 0.0, 1.0)
    W = WL.seeded_normal_bf16(2, f"W{N}{K}", (N, K), 0.0, 0.05)
    got = B.op_gemm_packed(A.cuda(), W.cuda()).cpu()
    assert rel_err(got, A.double() @ W.double().T) <= 4e-3


@pytest.mark.parametrize("M,N,K", [
    (81, 192, 64), (96, 320, 192), (97, 256, 128), (129, 4096, 448), (161, 1088, 1024), (300, 2112, 64), (513, 640, 320), (1023, 64, 192), (160, 28672, 128)])
def test_row_major_gemm_between_81_and_1023_rows(M, N, K):
    from paper_2410_03960_amd import binding as B
    _say(f"M={M} N={N} K={K}")
    A = WL.seeded_normal_bf16(1, f"A{M}{K}", (M, K), 0.0, 1.0)
    W = WL.seeded_normal_bf16(2, f"W{N}{K}", (N, K), 0.0, 0.05)
    ref = A.double() @ W.double().T
    for out_f32, tol in ((True, 1e-5), (False, 4e-3)):     # fp32 sums of exact products / one bf16 rounding
        assert rel_err(B.op_gemm(A.cuda(), W.cuda(), out_f32=out_f32).cpu(), ref) <= tol
