"""Products of 81 to 1023 rows with 128-column tiles, both operands streamed through LDS: every
tile height, whole and ragged, with and without K ranges, fragment-order weights (full layers,
the fused K/V projection) and row-major ones (the last tokens of more than 80 sequences, with
columns that end inside a tile), rotary heads of 128 and 64; against the oracle.  Which product
takes which tile is checked."""
import functools

import pytest

from tests import test_gpu_gemm_heights as H
from workloads.configs import ModelShape, Workload

pytestmark = pytest.mark.gpu

WIDE = Workload("stream_wide", ModelShape(2, 2048, 16, 4, 128, 8192, 544, 1e4, 1e-5), l=1, g=1, seed=2701)
SMALL = Workload("stream_small", ModelShape(3, 1024, 16, 4, 64, 1536, 544, 1e4, 1e-5), l=1, g=2, seed=2702)


def tail_tiles(wl, n):
    """{product: (rows of a tile, K ranges)} of the streamed tiles among the later layers' products over n last tokens."""
    from paper_2410_03960_amd import binding as B
    s = wl.shape
    of = functools.partial(B.op_gemm_plan, last_tokens=True)
    plans = {"q": of("bf16", n, s.q_dim, s.hidden, consumer_adds=True), "o": of("resid", n, s.hidden, s.q_dim, consumer_adds=True),
             "swiglu": of("swiglu", n, s.ffn, s.hidden), "down": of("resid", n, s.hidden, s.ffn, consumer_adds=True), "head": of("f32", n, s.vocab, s.hidden)}
    return {k: (p.tile, p.n_splits) for k, p in plans.items() if p.kernel == "stream_tile"}


@pytest.mark.parametrize("wl,lens,tiles", [
    (WIDE, [1] * 81, {64, 96}), (WIDE, [2] * 64, {64}), (WIDE, [1] * 160 + [33], {64, 128}), (WIDE, [150, 150], {64, 96, 160}),
    (WIDE, [1] * 329 + [1], {64, 96, 192}), (WIDE, [256, 255, 1], {64, 128}), (SMALL, [1] * 100, {64}), (SMALL, [1] * 257, {64}),
    (WIDE, [300, 299, 1], {96, 128, 160}), (WIDE, [1023], {64, 128}), (SMALL, [900], {64, 96})],
    ids=lambda v: v.name if isinstance(v, Workload) else f"{len(v)}x{sum(v)}" if isinstance(v, list) else "")
def test_stream_tiles_match_oracle(wl, lens, tiles):
    plans = [p for k, p in H.planned(wl, sum(lens), True).items() if k != "feed"]
    assert {p.tile for p in plans if p.kernel == "stream_tile"} == tiles
    H._say(f"{wl.name} {len(lens)} sequences, {sum(lens)} rows")
    H._check(wl, lens, fp8=len(lens) == 64, packed=True)


# Last tokens: 2048 and 1024 columns of q, and gate/up, the residual products and the vocabulary in turn with a last tile of 64
# columns.  {sequences: {product: (rows of a tile, K ranges)}}; other products have a contraction that is no multiple of 128.
TAILS = {
    Workload("tail_head", ModelShape(2, 2048, 16, 4, 128, 1056, 576, 1e4, 1e-5), l=1, g=1, seed=2703): {
        81: {"q": (96, 8), "o": (96, 8), "swiglu": (96, 8), "head": (64, 16)}, 193: {"q": (64, 4), "o": (64, 4), "swiglu": (96, 4), "head": (64, 8)},
        600: {"q": (96, 2), "o": (96, 2), "swiglu": (64, 1), "head": (64, 4)}},
    Workload("tail_resid", ModelShape(2, 1088, 8, 2, 128, 1024, 544, 1e4, 1e-5), l=1, g=1, seed=2704): {
        100: {"o": (64, 8), "down": (64, 8)}, 600: {"o": (64, 2), "down": (64, 2)}},
    Workload("tail_wide", ModelShape(2, 512, 8, 2, 128, 6176, 8256, 1e4, 1e-5), l=1, g=1, seed=2705): {
        300: {"q": (64, 2), "o": (64, 4), "swiglu": (160, 1), "head": (128, 1)}, 330: {"q": (64, 2), "o": (64, 4), "swiglu": (192, 1), "head": (128, 1)},
        900: {"q": (64, 1), "o": (64, 4), "swiglu": (192, 1), "head": (160, 1)}},
}


@pytest.mark.parametrize("wl,n", [(wl, n) for wl, cases in TAILS.items() for n in cases], ids=lambda v: getattr(v, "name", str(v)))
def test_last_tokens_match_oracle(wl, n):
    assert tail_tiles(wl, n) == TAILS[wl][n]
    H._say(f"{wl.name} {n} sequences")
    H._check(wl, [1] * n, fp8=False, packed=True)
