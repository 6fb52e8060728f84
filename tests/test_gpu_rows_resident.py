"""Weight-streaming GEMMs with the activations in LDS.  Up to 32 rows: one and two row
blocks at their edges, ragged last workgroups, one to nine K ranges or slices, the
shapes beside the rules' lines that keep another form, and (through a decoder whose
MLP is wide enough) the SwiGLU pair, whose weights and activations both pass through
LDS; 65 to 80 rows: the longer slices of large weights."""
import pytest
import torch

import workloads as WL
from tests import gpu_helpers as G
from tests.helpers import rel_err
from workloads.configs import ModelShape, Workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [
    (2, 13120, 512), (5, 16384, 1024), (16, 14352, 4096), (8, 28672, 512), (3, 32768, 1024), (16, 32064, 512), (9, 14336, 8704),
    (1, 14336, 512), (16, 8192, 4096), (2, 12288, 512), (16, 13104, 512), (10, 14336, 8704), (17, 14336, 512),
    (17, 4096, 4096), (32, 4112, 14336), (31, 6144, 2048), (18, 32784, 1536), (32, 12288, 512), (24, 3056, 512)])
def test_rows_gemm_at_the_edges(M, N, K):
    from paper_2410_03960_amd import binding as B
    print(f"M={M} N={N} K={K}", flush=True)
    A = WL.seeded_normal_bf16(1, f"A{M}{K}", (M, K), 0.0, 1.0)
    W = WL.seeded_normal_bf16(2, f"W{N}{K}", (N, K), 0.0, 0.05, device="cuda")
    ref = A.double() @ W.cpu().double().T
    for out_f32, tol in ((True, 1e-5), (False, 4e-3)):     # fp32 sums of exact products / one bf16 rounding
        assert rel_err(B.op_gemm_rows(A.cuda(), W, out_f32=out_f32).cpu(), ref) <= tol


# one slice of K per workgroup: a single one, several of one length, a shorter last one; one and two column blocks in a row
# per wave; ragged and whole last workgroups; one and two row blocks at their edges
@pytest.mark.parametrize("M,N,K,blocks,splits", [
    (5, 16400, 512, 8, 1), (16, 16400, 1536, 8, 1), (1, 8208, 5120, 8, 3), (16, 10256, 8704, 16, 5), (8, 33024, 3072, 16, 3),
    (17, 16400, 1024, 8, 1), (17, 8208, 2560, 8, 3), (32, 20496, 2560, 16, 3), (24, 33024, 3072, 16, 3), (31, 4112, 7168, 8, 7)])
def test_one_slice_per_workgroup(M, N, K, blocks, splits):
    from paper_2410_03960_amd import binding as B
    A = WL.seeded_normal_bf16(1, f"A{M}{K}", (M, K), 0.0, 1.0, device="cuda")
    W = WL.seeded_normal_bf16(2, f"W{N}{K}", (N, K), 0.0, 0.05, device="cuda")
    ref = torch.cat([A.double() @ w.double().T.contiguous() for w in W.split(4096)], 1)
    for out_f32, tol in ((True, 1e-5), (False, 4e-3)):     # fp32 sums of exact products / one bf16 rounding
        assert B.op_gemm_plan("f32" if out_f32 else "bf16", M, N, K, scratch=16 * M * N * 4)[:3] == ("stream_slice", blocks, splits)
        assert rel_err(B.op_gemm_rows(A, W, out_f32=out_f32), ref) <= tol


@pytest.mark.parametrize("M", [65, 80])
def test_long_slices_of_large_weights(M):
    """65 to 80 rows over weights of 430 MB and more: K ranges of whole 512-column slices."""
    from paper_2410_03960_amd import binding as B
    N, K = 8192, 26624
    for f32 in (True, False):
        assert B.op_gemm_plan("f32" if f32 else "bf16", M, N, K)[::3] == ("stream_seq", 512)
    A = WL.seeded_normal_bf16(1, f"A{M}{K}", (M, K), 0.0, 1.0, device="cuda")
    W = WL.seeded_normal_bf16(2, f"W{N}{K}", (N, K), 0.0, 0.05, device="cuda")
    ref = torch.cat([A.double() @ w.double().T.contiguous() for w in W.split(1024)], 1)
    for out_f32, tol in ((True, 1e-5), (False, 4e-3)):     # fp32 sums of exact products / one bf16 rounding
        assert rel_err(B.op_gemm_rows(A, W, out_f32=out_f32), ref) <= tol


@pytest.fixture(scope="module")
def wide_mlp():
    wl = Workload("wide_mlp", ModelShape(2, 512, 4, 2, 128, 13136, 512, 1e4, 1e-5), l=1, g=1, seed=2310)   # 821 column blocks
    store = WL.make_weights(wl, "cpu", keep=True)
    return wl, store, G.device_weights(store)


@pytest.mark.parametrize("lens", [[1], [5, 1, 1], [3, 2, 1, 1, 1], [6, 1, 1, 1], [9, 1, 7], [20, 11, 1]], ids=str)
def test_wide_mlp_matches_oracle(wide_mlp, lens):
    from paper_2410_03960_amd import binding as B
    wl, store, dev_w = wide_mlp
    print(lens, flush=True)
    batch = WL.build_batch(wl, lens=lens, shuffled=True)
    logits, cache, _ = G.run_gpu(B.Context(wl.shape, dev_w, wl.l, wl.g), batch)
    ologits, ocache, _ = G.run_oracle(wl.shape, store, batch, wl.l, wl.g)
    G.compare_caches(cache, ocache, batch, label=wl.name)
    G.compare_logits(logits, ologits, rel=G.BF16_REL, cos=G.BF16_COS, label=wl.name)
