"""Single-query attention over bf16 caches with one and two query heads per KV head on the vector unit: one and several key
splits, splits of 32 and of 128 keys, rows with fewer splits than others, both head sizes; queries as they are, rotated on
the way, and added up from the K ranges of their projection.  That these shapes take the vector unit is checked."""
import pytest

import workloads as WL
from paper_2410_03960_amd import binding as B
from tests import gpu_helpers as G
from tests.test_gpu_ops import test_single_query_attention_over_paged_cache as check
from workloads.configs import ModelShape, Workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hd,Hq,Hkv,lens,splits,min_keys", [
    (128, 8, 8, [1], 1, 32), (128, 8, 8, [333], 11, 32), (128, 8, 8, [778], 25, 32), (128, 16, 8, [500], 16, 32), (128, 4, 2, [600, 40, 130, 7], 19, 32),
    (128, 8, 8, [40] * 200, 1, 128), (128, 16, 8, [97] * 128, 1, 128), (128, 8, 8, [900, 1] * 8, 8, 128), (128, 16, 8, [900, 129] * 8, 8, 128),
    (128, 32, 32, [600, 40, 130, 7], 8, 128), (128, 32, 32, [3000, 200], 16, 128), (128, 32, 32, [2048], 32, 128), (128, 8, 8, [3000, 200], 32, 128),
    (64, 8, 8, [778], 25, 32), (64, 8, 8, [64] * 300, 1, 128), (64, 8, 8, [97, 1] * 64, 1, 128), (64, 8, 8, [900, 129] * 8, 8, 128), (64, 8, 8, [3000, 200], 32, 128),
], ids=lambda v: f"{len(v)}x{max(v)}" if isinstance(v, list) else None)
def test_vector_unit(hd, Hq, Hkv, lens, splits, min_keys):
    assert B.op_attention_decode_plan(lens, Hq, Hkv, hd) == ("vector", splits, min_keys)
    check(hd, Hq, Hkv, "bf16", lens)


@pytest.mark.parametrize("heads,kv_heads,hidden,q_ranges", [(8, 8, 512, 1), (8, 8, 2048, 2), (16, 8, 512, 1), (16, 8, 2048, 2)])
def test_last_token_on_the_vector_unit(heads, kv_heads, hidden, q_ranges):
    assert B.op_attention_decode_plan([500], heads, kv_heads, 128).unit == "vector"
    assert min(2, B.op_gemm_plan("f32", 1, heads * 128, hidden, consumer_adds=True).n_splits) == q_ranges
    wl = Workload(f"unit{heads}_{hidden}", ModelShape(2, hidden, heads, kv_heads, 128, 512, 512, 1e4, 1e-5), l=1, g=1, seed=2901)
    store = WL.make_weights(wl, "cpu", keep=True)
    batch = WL.build_batch(wl, lens=[500], shuffled=True)
    logits, cache, _ = G.run_gpu(B.Context(wl.shape, G.device_weights(store), 1, 1), batch)
    ologits, ocache, _ = G.run_oracle(wl.shape, store, batch, 1, 1)
    G.compare_caches(cache, ocache, batch, label=wl.name)
    G.compare_logits(logits, ologits, label=wl.name)
