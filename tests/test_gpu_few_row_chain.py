"""Up to eight rows: the residual GEMM leaves the next projection's operand and sums of squares, which that projection turns into 1/rms;
against the CPU oracle at the edges of the rule."""
import pytest

import workloads as WL
from workloads.configs import ModelShape, Workload
from tests import gpu_helpers as G
from tests.helpers import rel_err

pytestmark = pytest.mark.gpu

SHAPES = {
    # K ranges of the eight waves: whole steps each; two waves without any (6 steps); one step each and 320 column blocks, which keep the norm pass
    "even": ModelShape(4, 1024, 8, 4, 128, 2048, 512, 5e5, 1e-5),
    "short": ModelShape(4, 512, 6, 6, 64, 1536, 512, 5e5, 1e-5),
    "uneven": ModelShape(2, 5120, 4, 2, 128, 512, 512, 5e5, 1e-5),
}


@pytest.mark.parametrize("name,l,g", [("even", 2, 1), ("even", 4, 1), ("even", 1, 3), ("short", 2, 2), ("uneven", 1, 1)])
@pytest.mark.parametrize("lens", [[1], [8], [9], [3, 2, 1, 1], [30] * 7 + [1], [12] * 9])   # all rows; the last tokens of 8 and of 9 sequences
def test_rows_through_both_forms(name, l, g, lens):
    from paper_2410_03960_amd import binding as B
    if name == "uneven" and (len(lens) > 4 or sum(lens) > 9):
        pytest.skip("the same kernels as the other shapes'")
    shape = SHAPES[name]
    wl = Workload("chain_" + name, shape, l=l, g=g, seed=3011)
    store = WL.make_weights(wl, "cpu", keep=True)
    batch = WL.build_batch(wl, lens=lens, shuffled=True)
    ctx = B.Context(shape, G.device_weights(store), l, g)
    logits, cache, ws = G.run_gpu(ctx, batch)
    G.check_plan(ctx, ws, batch)
    ologits, ocache, _ = G.run_oracle(shape, store, batch, l, g)
    G.compare_caches(cache, ocache, batch, label=name)
    G.compare_logits(logits, ologits, label=name)


@pytest.mark.parametrize("per_token", [False, True])
@pytest.mark.parametrize("lens", [[1] * 8, [3, 2, 1, 1], [30] * 7 + [1]])
def test_codes_and_scales_of_rows_without_a_norm_pass(lens, per_token):
    """Over an e4m3 cache: the absmax of each head, or of each token, comes from sums that carry the rows' 1/rms."""
    from paper_2410_03960_amd import binding as B
    shape = SHAPES["even"]
    for rows in {min(8, sum(lens)), len(lens)}:
        assert all(B.op_gemm_plan_folded("resid", rows, shape.hidden, k).kernel == "stream_folded" for k in (shape.q_dim, shape.ffn))
    wl = Workload("chain_fp8", shape, l=2, g=1, seed=3012)
    store = WL.make_weights(wl, "cpu", keep=True)
    batch = WL.build_batch(wl, lens=lens, shuffled=True)
    ctx = B.Context(shape, G.device_weights(store), 2, 1)
    logits, cache, ws = G.run_gpu(ctx, batch, fp8=True, scale_mode=B.SWIFTKV_SCALE_PER_TOKEN if per_token else B.SWIFTKV_SCALE_COMPUTE_ABSMAX)
    G.check_plan(ctx, ws, batch)
    ologits, ocache, _ = G.run_oracle(shape, store, batch, 2, 1, fp8=True, per_token=per_token)
    assert rel_err(cache.scales.cpu(), ocache.scales) <= 2e-2
    G.compare_caches(cache, ocache, batch, rel=G.FP8_REL, cos=G.FP8_COS, label=wl.name)
    G.compare_logits(logits, ologits, rel=G.FP8_REL, cos=G.FP8_COS, label=wl.name)
