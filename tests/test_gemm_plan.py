"""The choice of GEMM kernel by shape (host code, no GPU)."""
import os

import pytest

from paper_2410_03960_amd import binding as B
from tests import test_gpu_gemm_heights as H
from tests import test_gpu_gemm_two_heights as TWO
from tests import test_gpu_mid as MID


@pytest.fixture(scope="module", autouse=True)
def built():
    if not os.path.exists(B.LIB_PATH):
        from paper_2410_03960_amd import build
        build.build(verbose=False)


# down GEMMs around the number of rows at which their activations reach 4 GiB: 74899 rows of 28672, 149797 of 14336
@pytest.mark.parametrize("M,N,K", [(74898, 8192, 28672), (74899, 8192, 28672), (131072, 8192, 28672), (149797, 4096, 14336)])
@pytest.mark.parametrize("epilogue", ["bf16", "resid", "swiglu"])
def test_packed_loop_beyond_4_gib_of_activations(epilogue, M, N, K):
    for norm_out in (False, True):
        for consumer_adds in (False, True):
            plan = B.op_gemm_plan(epilogue, M, N, K, packed=True, norm_out=norm_out, consumer_adds=consumer_adds)
            assert (plan.kernel, plan.tile, plan.n_splits) == ("packed_dma", 256, 1)


# Weight streaming beyond 4 GiB of activations: skinny_ring_kernel holds a row's offset in 32 bits.  128 MiB of K lie in a row here.
@pytest.mark.parametrize("M,K,kernel", [(80, 1 << 26, "stream_first"), (33, 1 << 26, "stream_first"), (31, 1 << 26, "stream_seq"), (80, 1 << 24, "stream_seq")])
def test_weight_streaming_beyond_4_gib_of_activations(M, K, kernel):
    assert B.op_gemm_plan("f32", M, 16, K, consumer_adds=True).kernel == kernel
    assert B.op_gemm_plan("swiglu", M, 16384, K).kernel == kernel
    if M > 32:
        assert B.op_gemm_plan("bf16", M, 16, K).kernel == kernel


# Row-major weights and no room for K splits (swiftkv_op_gemm): the 128 x 128 tile, but for shapes whose last round of its
# tiles is nearly empty (6 x 86 = 512 + 4, 8 x 80 = 512 + 128, 2 x 1002 = 3 x 512 + 468 tiles).
@pytest.mark.parametrize("M,N,K,kernel", [
    (81, 4096, 4096, "tile_128"), (128, 8192, 8192, "tile_128"), (160, 8192, 8192, "tile_128"), (333, 11008, 4096, "tile_128"),
    (420, 10240, 8192, "tile_128"), (512, 4096, 14336, "tile_128"), (700, 6144, 4096, "tile_128"), (1023, 4096, 11008, "tile_128"),
    (1023, 512, 4096, "tile_128"), (700, 11008, 4096, "rows_reg"), (900, 10240, 8192, "rows_reg"), (160, 128256, 4096, "rows_reg")])
def test_row_major_products_without_scratch(M, N, K, kernel):
    for epilogue in ("bf16", "f32"):
        plan = B.op_gemm_plan(epilogue, M, N, K, scratch=0)
        assert (plan.kernel, plan.n_splits) == (kernel, 1)


# ... and with it: K splits, which fill the CUs
@pytest.mark.parametrize("M,N,K", [(81, 4096, 4096), (160, 4096, 14336), (333, 8192, 2048)])
def test_row_major_products_with_scratch_split_k(M, N, K):
    plan = B.op_gemm_plan("resid", M, N, K, consumer_adds=True)
    assert plan.kernel == "rows_reg" and plan.n_splits > 1


# Q, K and V leave the streamed 128-column tiles as partial sums: only where the other forms split K as well.
@pytest.mark.parametrize("M,N,K,hd,kernel", [
    (700, 4096, 2048, 64, "packed_reg"), (640, 4096, 2048, 64, "packed_reg"), (330, 8192, 2048, 64, "packed_reg"), (130, 8192, 1024, 64, "packed_reg"),
    (330, 4096, 2048, 64, "stream_tile"), (450, 8192, 4096, 128, "stream_tile"), (1020, 2048, 4096, 64, "stream_tile")])
def test_rotary_products_that_need_no_second_pass(M, N, K, hd, kernel):
    for epilogue in ("kv", "qkv"):
        plan = B.op_gemm_plan(epilogue, M, N, K, packed=True, head_dim=hd)
        assert plan.kernel == kernel and (kernel == "stream_tile" or plan.n_splits == 1)


# The last tokens of more than 80 sequences: 128-column tiles, with K ranges for whoever adds them and for those that nobody does.
@pytest.mark.parametrize("M,N,K", [(81, 4096, 4096), (160, 4096, 14336), (333, 8192, 2048), (600, 2048, 2048), (1023, 2048, 8192)])
def test_last_tokens_stream_their_weights(M, N, K):
    for epilogue in ("bf16", "f32", "resid"):
        for adds in (False, True):
            plan = B.op_gemm_plan(epilogue, M, N, K, consumer_adds=adds, last_tokens=True)
            assert plan.kernel == "stream_tile"
    assert B.op_gemm_plan("swiglu", M, N, K, last_tokens=True).kernel == "stream_tile"
    assert B.op_gemm_plan("resid", M, N, K, consumer_adds=True).kernel != "stream_tile"     # row-major weights of a context's full layers
    assert B.op_gemm_plan("resid", M, N, K + 64, last_tokens=True).kernel != "stream_tile"


@pytest.mark.parametrize("M,slice_", [(33, 512), (64, 512), (65, 256), (80, 256)])
@pytest.mark.parametrize("N,K", [(2048, 2048), (4096, 4096), (13824, 5120), (20480, 10240)])
def test_slices_of_33_to_80_rows(M, slice_, N, K):
    for epilogue, adds, weights in (("bf16", False, 1), ("f32", True, 1), ("swiglu", False, 2)):
        plan = B.op_gemm_plan(epilogue, M, N, K, consumer_adds=adds)
        large = 2 * weights * N * K >= 430e6          # at 65 to 80 rows too, the longer slices are ahead
        assert (plan.kernel, plan.slice) == ("stream_seq", 512 if large else slice_)


# Up to 32 rows with a result that is final: shapes that the first kernel (16 rows x 13824 x 5120: 51 us) or one long walk of
# slices (1 row x 28672 x 8192: 103 us) serves 10 to 50 % slower than the kernel named.
@pytest.mark.parametrize("M,N,K,kernel", [
    (16, 13824, 5120, "stream_seq"), (16, 5120, 13824, "stream_seq"), (24, 11008, 4096, "stream_slice"), (32, 11008, 4096, "stream_slice"),
    (16, 14336, 4096, "stream_slice"), (1, 28672, 8192, "stream_first"), (8, 28672, 8192, "stream_slice"), (1, 32000, 2048, "stream_slice"),
    (16, 8192, 28672, "stream_slice"), (24, 5120, 5120, "stream_slice"),
    (1, 4096, 4096, "stream_first"), (1, 8192, 2048, "stream_first"), (24, 128256, 4096, "stream_seq")])
def test_final_results_of_up_to_32_rows(M, N, K, kernel):
    plan = B.op_gemm_plan("bf16", M, N, K, scratch=16 * M * N * 4)
    assert plan.kernel == kernel and (kernel != "stream_seq" or N > 100000 or plan.n_splits > 1)


# The GPU parity tests of the tiled kernels reach the kernels and heights that they are there for.
def test_parity_cases_reach_every_packed_height():
    for rows, tile in H.PACKED_HEIGHTS.items():
        feed = H.planned(H.FEED, rows, True)
        assert feed["feed"]
        for plan in (feed["o"], feed["down"], *(H.planned(wl, rows, True)["kv"] for wl in H.KV.values())):
            assert (plan.kernel, plan.tile, plan.n_splits) == ("packed_dma", tile, 1)
    for rows, tile in H.BROAD_HEIGHTS.items():
        for product in ("qkv", "swiglu"):
            plan = H.planned(H.BROAD, rows, True)[product]
            assert (plan.kernel, plan.tile, plan.n_splits) == ("packed_dma", tile, 1)
    assert sorted(set(H.PACKED_HEIGHTS.values())) == sorted(set(H.BROAD_HEIGHTS.values())) == [128, 160, 192, 224, 256]


def test_parity_cases_reach_every_row_major_height():
    reached = set()
    for (wl, lens), want in H.ROW_HEIGHTS.items():
        plans = H.planned(wl, sum(lens), False)
        for product, (tile, splits) in want.items():
            plan = plans[product]
            assert (plan.kernel, plan.tile, plan.n_splits) == ("rows_reg", tile, splits), (wl.name, sum(lens), product)
            reached.add((tile, splits > 1))
    assert reached == {(tile, split) for tile in (64, 96, 128, 160) for split in (False, True)}
    assert B.op_gemm_plan("f32", 641, 11008, 512, scratch=0)[:3] == ("rows_reg", 160, 1)


def test_parity_cases_of_the_mid_size_decoders():
    for wl in MID.MID.values():
        for product, plan in H.planned(wl, sum(MID.LENS), True).items():
            assert product == "feed" or (plan.kernel, plan.tile) == ("packed_reg", 64)
        for product, plan in H.planned(wl, sum(MID.LENS), False).items():
            assert product == "feed" or plan.kernel == "five_stage"


# Gate and up in two tile heights, as the GPU parity cases say; one height where K is split, and for other products.
def test_parity_cases_reach_two_tile_heights():
    for wl in (TWO.FEED, TWO.LONG):
        for rows, low in TWO.LOW_TILES.items():
            assert B.op_gemm_low_tiles(rows, wl.shape.ffn, wl.shape.hidden) == low
    assert {low[0] for low in TWO.LOW_TILES.values()} == {0, 128, 192}
    assert B.op_gemm_plan("swiglu", 100, 512, 4096, packed=True).n_splits > 1 and B.op_gemm_low_tiles(100, 512, 4096) == (0, 0)


# Up to eight rows with no norm pass between the products: the residual one is final, the others take 1/rms in the ring kernel.
def test_products_of_up_to_eight_rows_without_norm_passes():
    for rows in (1, 8):
        assert B.op_gemm_plan_folded("resid", rows, 4096, 14336) == ("stream_folded", 1, 1, 0)
        for epilogue, N in (("swiglu", 4096), ("qkv", 6144), ("bf16", 4096)):
            assert B.op_gemm_plan_folded(epilogue, rows, N, 4096, consumer_adds=epilogue == "bf16").kernel == "stream_seq"
    assert B.op_gemm_plan("swiglu", 8, 4096, 4096).kernel == "stream_first"
    for rows, N, K in ((9, 4096, 14336), (1, 5120, 13824)):                 # nine rows; 320 blocks of 16 columns over 256 CUs
        assert B.op_gemm_plan_folded("resid", rows, N, K, consumer_adds=True) == B.op_gemm_plan("resid", rows, N, K, consumer_adds=True)


# ... and only where a wave's walk through K / 8 does not outlast the K ranges of the other kernel on the CUs that few columns leave over.
@pytest.mark.parametrize("N,K,rows", [      # most rows that take the form
    (1024, 4096, 8), (1024, 8192, 8), (1024, 14336, 3), (1024, 16384, 2), (1024, 20480, 0), (2048, 8192, 8), (2048, 16384, 7), (2048, 32768, 2), (2048, 40960, 0),
    (3072, 32768, 8), (3072, 49152, 7), (4096, 49152, 8), (8192, 28672, 8), (512, 16384, 8), (512, 32768, 0), (1536, 32768, 8), (1536, 49152, 4)])
def test_few_columns_over_a_long_contraction_keep_k_ranges(N, K, rows):
    taken = [m for m in range(1, 10) if B.op_gemm_plan_folded("resid", m, N, K, consumer_adds=True).kernel == "stream_folded"]
    assert taken == list(range(1, rows + 1))
