"""Products of 81 to 512 rows with 128-column tiles, both operands streamed through LDS: every
tile height, whole and ragged, with and without K ranges, fragment-order weights (full layers,
the fused K/V projection) and row-major ones (the last tokens of more than 80 sequences, whose
vocabulary ends inside a tile), rotary heads of 128 and 64; against the oracle."""
import pytest

from tests import test_gpu_gemm_heights as H
from workloads.configs import ModelShape, Workload

pytestmark = pytest.mark.gpu

WIDE = Workload("stream_wide", ModelShape(2, 2048, 16, 4, 128, 8192, 544, 1e4, 1e-5), l=1, g=1, seed=2701)
SMALL = Workload("stream_small", ModelShape(3, 1024, 16, 4, 64, 1536, 544, 1e4, 1e-5), l=1, g=2, seed=2702)


@pytest.mark.parametrize("wl,lens,tiles", [
    (WIDE, [1] * 81, {64, 96}), (WIDE, [2] * 64, {64}), (WIDE, [1] * 160 + [33], {64, 128}), (WIDE, [150, 150], {64, 96, 160}),
    (WIDE, [1] * 329 + [1], {64, 96, 192}), (WIDE, [256, 255, 1], {64, 128}), (SMALL, [1] * 100, {64}), (SMALL, [1] * 257, {64})],
    ids=lambda v: v.name if isinstance(v, Workload) else f"{len(v)}x{sum(v)}" if isinstance(v, list) else "")
def test_stream_tiles_match_oracle(wl, lens, tiles):
    plans = [p for k, p in H.planned(wl, sum(lens), True).items() if k != "feed"]
    assert {p.tile for p in plans if p.kernel == "stream_tile"} == tiles
    H._say(f"{wl.name} {len(lens)} sequences, {sum(lens)} rows")
    H._check(wl, lens, fp8=len(lens) == 64, packed=True)
