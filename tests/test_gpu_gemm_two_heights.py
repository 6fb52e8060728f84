"""Gate and up in a launch of two tile heights: 256-row tiles over the first columns, 192- or 128-row tiles over the last ones.  Row
counts whose single heights leave a last round nearly empty over 112 columns of tiles (28672 / 256), so that the rule takes two:
192 rows for 897 and 3300 rows, 128 rows for 2045 and 2048 (1000 keep one height); ragged last tiles of both heights, and CUs that have no tile of the last
round of the taller ones (3300 rows: 13 tiles do not divide 1280)."""
import pytest
import torch

import workloads as WL
from tests import gpu_helpers as G
from workloads.configs import ModelShape, Workload

pytestmark = pytest.mark.gpu
FEED = Workload("two_heights", ModelShape(2, 256, 2, 2, 128, 14336, 256, 1e4, 1e-5), l=1, g=1, seed=2311)
LONG = Workload("two_heights_long", ModelShape(2, 1024, 8, 2, 128, 14336, 256, 1e4, 1e-5), l=1, g=1, seed=2312)   # (16 steps: stages refilled with live data)
LOW_TILES = {897: (192, 12288), 1000: (0, 0), 2045: (128, 4096), 2048: (128, 4096), 3300: (192, 3584)}            # rows -> rows and columns of the lower tiles


@pytest.mark.parametrize("wl,rows", [(FEED, r) for r in LOW_TILES] + [(LONG, 897), (LONG, 2045)], ids=lambda v: str(getattr(v, "name", v)))
def test_two_heights(wl, rows):
    from paper_2410_03960_amd import binding as B
    assert B.op_gemm_low_tiles(rows, wl.shape.ffn, wl.shape.hidden) == LOW_TILES[rows]
    store = WL.make_weights(wl, "cpu", keep=True)
    ctx = B.Context(wl.shape, G.device_weights(store), wl.l, wl.g, packed_weights=True)
    batch = WL.build_batch(wl, lens=[190] * (rows // 190) + [rows % 190], shuffled=True)
    logits, cache, _ = G.run_gpu(ctx, batch)
    ologits, ocache, _ = G.run_oracle(wl.shape, store, batch, wl.l, wl.g, dtype=torch.float32)
    G.compare_caches(cache, ocache, batch, label=wl.name)
    G.compare_logits(logits, ologits, label=wl.name)
    assert all(torch.equal(a, b) for a, b in zip((logits, cache.data), (lambda r: (r[0], r[1].data))(G.run_gpu(ctx, batch))))
