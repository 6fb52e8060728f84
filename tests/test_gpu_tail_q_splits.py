"""Last tokens whose q projection leaves its K ranges apart: the attention kernels of the matrix unit add
them up (bf16 and e4m3 caches; one row, one and several 16-row blocks, more rows than the
weight-streaming kernels take), against the oracle.  The vector unit's: test_gpu_decode_units."""
import pytest

import workloads as WL
from tests import gpu_helpers as G
from workloads.configs import ModelShape, Workload

pytestmark = pytest.mark.gpu

SHAPES = {
    "r4_hd128": ModelShape(2, 2048, 16, 4, 128, 512, 512, 1e4, 1e-5),
    "r8_hd128": ModelShape(2, 2048, 16, 2, 128, 512, 512, 1e4, 1e-5),
    "r2_hd64": ModelShape(2, 1024, 16, 8, 64, 512, 512, 1e4, 1e-5),
}


@pytest.mark.parametrize("name,n_seqs,fp8", [
    ("r4_hd128", 1, False), ("r4_hd128", 70, False), ("r4_hd128", 90, False), ("r8_hd128", 3, False), ("r8_hd128", 20, False),
    ("r2_hd64", 17, False), ("r4_hd128", 33, True), ("r8_hd128", 90, True), ("r2_hd64", 2, True)])
def test_tail_matches_oracle(name, n_seqs, fp8):
    from paper_2410_03960_amd import binding as B
    print(name, n_seqs, fp8, flush=True)
    sh = SHAPES[name]
    plan = B.op_gemm_plan("bf16", n_seqs, sh.q_dim, sh.hidden, consumer_adds=True, last_tokens=n_seqs > 80)
    assert plan.kernel == ("stream_seq" if n_seqs <= 80 else "stream_tile") and plan.n_splits > 1
    wl = Workload(f"tailq_{name}", sh, l=1, g=1, seed=2610)
    store = WL.make_weights(wl, "cpu", keep=True)
    batch = WL.build_batch(wl, lens=[1 + (7 * i + 3) % 5 for i in range(n_seqs)] if n_seqs > 3 else [150, 40, 2][:n_seqs], shuffled=True)
    ctx = B.Context(sh, G.device_weights(store), wl.l, wl.g)
    if fp8:
        logits, cache, _ = G.run_gpu(ctx, batch, fp8=True, scale_mode=B.SWIFTKV_SCALE_COMPUTE_ABSMAX)
        ologits, ocache, _ = G.run_oracle(sh, store, batch, wl.l, wl.g, fp8=True, compute_scales=True)
        rel, cos = G.FP8_REL, G.FP8_COS
    else:
        logits, cache, _ = G.run_gpu(ctx, batch)
        ologits, ocache, _ = G.run_oracle(sh, store, batch, wl.l, wl.g)
        rel, cos = G.BF16_REL, G.BF16_COS
    G.compare_logits(logits, ologits, rel=rel, cos=cos, label=name)
