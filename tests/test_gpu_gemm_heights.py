"""Parity of the GEMMs between the weight-streaming kernels (80 rows) and many
full rounds of 256-row tiles: every tile height, K splits with each epilogue's
finishing pass, ragged last tiles, packed and row-major weights.  Which kernel
and height a case reaches is stated beside it (PACKED_HEIGHTS, ROW_HEIGHTS,
BROAD_HEIGHTS) and checked against the library's plan without a GPU."""
import functools
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
# Fragment-order weights.  FEED: O (K 512) and down (K 256) write 6144 residual columns each, unsplit, so they leave the next
# projection's operand and the rows' sums of squares.  KV*: three groups of later layers, 6144 columns of K and V over a
# contraction of 256, unsplit, so K and V leave through the epilogue (bf16 to their slots; FP8 staged, with the heads' absmax).
FEED = Workload("feed", ModelShape(2, 6144, 4, 2, 128, 256, 256, 1e4, 1e-5), l=1, g=1, seed=2204)
KV = {
    "hd128": Workload("kv_hd128", ModelShape(4, 256, 8, 8, 128, 256, 256, 1e4, 1e-5), l=1, g=1, seed=2205),
    "hd64": Workload("kv_hd64", ModelShape(4, 256, 16, 16, 64, 256, 256, 1e4, 1e-5), l=1, g=1, seed=2206),
}
PACKED_HEIGHTS = {1100: 128, 1300: 160, 1700: 192, 2000: 224, 2300: 256}      # rows -> tile of both models' products
BROAD_HEIGHTS = {1025: 128, 1300: 160, 1700: 192, 2000: 224, 2300: 256, 2561: 128}   # ... of BROAD's Q/K/V and gate/up, unsplit
# Row-major weights.  TALL splits K, SHORT does not (gate/up of 5632 columns and 6144 columns of K and V over 256).
TALL = Workload("tall", ModelShape(2, 4096, 32, 8, 128, 3072, 512, 1e4, 1e-5), l=1, g=1, seed=2207)
SHORT = Workload("short", ModelShape(4, 256, 8, 8, 128, 5632, 256, 1e4, 1e-5), l=1, g=1, seed=2208)
# (model, tokens per sequence) -> {product: (rows of a tile, K splits)}; sequences of one token run the later layers on every row
ROW_HEIGHTS = {
    (TALL, (96,)): {"qkv": (96, 8), "swiglu": (96, 8), "o": (64, 8)},
    (TALL, (1,) * 97): {"qkv": (128, 8), "swiglu": (128, 8), "o": (64, 8)},
    (TALL, (1,) * 132): {"qkv": (160, 8), "swiglu": (160, 8), "o": (96, 8), "down": (96, 8), "kv": (96, 13)},
    (TALL, (140, 67)): {"qkv": (128, 5), "swiglu": (128, 5), "o": (128, 8), "down": (128, 6)},
    (TALL, (300,)): {"qkv": (160, 5), "swiglu": (160, 5), "o": (128, 5)},
    (SHORT, (328,)): {"swiglu": (96, 1), "kv": (64, 1)},
    (SHORT, (401, 89)): {"swiglu": (128, 1), "kv": (64, 1)},
    (SHORT, (699, 1)): {"swiglu": (160, 1), "kv": (96, 1)},
}


def planned(wl, rows, packed):
    """The library's choice for each product of the full layers, and for the later layers' K and V, over `rows` tokens."""
    from paper_2410_03960_amd import binding as B
    s, later = wl.shape, wl.shape.n_layers - wl.l
    qd, kvd = s.n_q_heads * s.head_dim, s.n_kv_heads * s.head_dim

    def of(epilogue, n, k, **kw):
        return B.op_gemm_plan(epilogue, rows, n, k, packed=packed, head_dim=s.head_dim if epilogue in ("qkv", "kv") else 0, **kw)
    d = s.hidden
    # both residual products unsplit: they leave the next projection's operand, nobody adds splits
    feed = packed and rows >= 1024 and all(of("resid", d, k, consumer_adds=True).n_splits == 1 for k in (qd, s.ffn))
    resid = {"norm_out": True} if feed else {"consumer_adds": True}
    return {"qkv": of("qkv", qd + 2 * kvd, d), "o": of("resid", d, qd, **resid), "swiglu": of("swiglu", s.ffn, d),
            "down": of("resid", d, s.ffn, **resid), "kv": of("kv", (later + wl.g - 1) // wl.g * 2 * kvd, d), "feed": feed}


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def _lens(rows, each=190):
    return [each] * (rows // each) + ([rows % each] if rows % each else [])


@functools.lru_cache(maxsize=1)
def _weights(wl):
    return WL.make_weights(wl, "cpu", keep=True)


def _check(wl, lens, fp8, packed, ctx_lens=None):
    from paper_2410_03960_amd import binding as B
    store = _weights(wl)
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


@pytest.mark.parametrize("rows", sorted(BROAD_HEIGHTS))
def test_tile_heights_with_rotating_and_swiglu_epilogues(rows):
    _say(f"rows={rows}")
    _check(BROAD, _lens(rows), fp8=rows == 2000, packed=True)


@pytest.mark.parametrize("rows", [1025, 2561, 4500])
def test_tile_heights_with_residual_epilogue(rows):
    _say(f"rows={rows}")
    _check(LONG["hd128"], _lens(rows, 256), fp8=False, packed=True)


@pytest.mark.parametrize("rows", sorted(PACKED_HEIGHTS))
def test_residual_epilogue_that_feeds_the_next_projection(rows):
    _say(f"rows={rows}")
    _check(FEED, _lens(rows), fp8=False, packed=True)


@pytest.mark.parametrize("rows", sorted(PACKED_HEIGHTS))
@pytest.mark.parametrize("name", sorted(KV))
def test_unsplit_kv_epilogue(name, rows):
    _say(f"{name} rows={rows}")
    for fp8 in (False, True):
        _check(KV[name], _lens(rows), fp8=fp8, packed=True)


@pytest.mark.parametrize("wl,lens", sorted(ROW_HEIGHTS, key=str), ids=lambda v: v.name if isinstance(v, Workload) else f"{len(v)}x{sum(v)}")
def test_row_major_tile_heights(wl, lens):
    _say(f"{wl.name} lens={lens}")
    _check(wl, list(lens), fp8=len(lens) == 2, packed=False)


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
    (81, 192, 64), (96, 320, 192), (97, 256, 128), (129, 4096, 448), (161, 1088, 1024), (300, 2112, 64), (513, 640, 320), (1023, 64, 192), (160, 28672, 128), (641, 11008, 512)])
def test_row_major_gemm_between_81_and_1023_rows(M, N, K):
    """swiftkv_op_gemm, which has no room for K splits: the 128 x 128 tile but for the last shape."""
    from paper_2410_03960_amd import binding as B
    _say(f"M={M} N={N} K={K}")
    A = WL.seeded_normal_bf16(1, f"A{M}{K}", (M, K), 0.0, 1.0)
    W = WL.seeded_normal_bf16(2, f"W{N}{K}", (N, K), 0.0, 0.05)
    ref = A.double() @ W.double().T
    for out_f32, tol in ((True, 1e-5), (False, 4e-3)):     # fp32 sums of exact products / one bf16 rounding
        assert rel_err(B.op_gemm(A.cuda(), W.cuda(), out_f32=out_f32).cpu(), ref) <= tol


@pytest.mark.parametrize("hd,tokens", [(64, 81), (64, 515), (128, 100), (128, 513), (64, 37)])
def test_computed_scales_of_split_kv_products(hd, tokens):
    """The finishing pass of a split K/V product takes the heads' absmax over groups of rows: the scales are those of the
    values that the same call stores into a bf16 cache, bit by bit, and the codes are those values rounded once."""
    from oracle import swiftkv_oracle as O
    from paper_2410_03960_amd import binding as B
    sh = ModelShape(9, 2048, 1024 // hd, 256 // hd, hd, 256, 256, 1e4, 1e-5)
    kvd = sh.n_kv_heads * hd
    plan = B.op_gemm_plan("kv", tokens, 8 * 2 * kvd, sh.hidden, packed=True, head_dim=hd)
    assert plan.n_splits > 1
    _say(f"hd={hd} tokens={tokens} {plan}")
    ctx = B.Context(sh, G.device_weights(_weights(Workload(f"scales{hd}", sh, l=1, g=1, seed=2209))), 1, 1)
    hidden = WL.seeded_normal_bf16(3, f"hidden{tokens}", (tokens, sh.hidden), 0.0, 1.0).cuda()
    n_blocks = (tokens + 15) // 16
    table = torch.randperm(n_blocks, generator=torch.Generator().manual_seed(tokens)).int().view(1, -1)
    caches = []
    for fp8 in (False, True):
        cache = B.KVCache(ctx.n_cache_layers, n_blocks, sh.n_kv_heads, hd, table, [0], fp8=fp8,
                          scale_mode=B.SWIFTKV_SCALE_COMPUTE_ABSMAX if fp8 else 0)
        kind = B.SWIFTKV_KV_FP8_E4M3 if fp8 else B.SWIFTKV_KV_BF16
        ctx.kv_from_hidden(hidden, [tokens], cache, torch.empty(ctx.workspace_bytes(tokens, 1, kind, 0), dtype=torch.uint8, device="cuda"))
        caches.append(cache)
    pos = torch.arange(tokens)
    slots = table[0].long()[pos // 16] * 16 + pos % 16
    stored = caches[0].data[1:, :, slots.cuda()].float().cpu()             # [later layers, K|V, tokens, heads, hd]
    scales = torch.maximum(stored.abs().amax(dim=(2, 4)), torch.tensor(1e-12)) / 448.0
    assert torch.equal(caches[1].scales[1:].cpu(), scales)
    got = O.fp8_e4m3fn_decode_table().float()[caches[1].data[1:, :, slots.cuda()].cpu().long()] * scales[:, :, None, :, None]
    # three mantissa bits: half a unit is 2^-4 of the value, or 2^-10 of the scale below its normal range
    assert ((got - stored).abs() <= 2.0 ** -4 * stored.abs() + 2.0 ** -10 * scales[:, :, None, :, None]).all()
