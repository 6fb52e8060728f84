"""Weight-streaming GEMM with weights and activations through LDS, 33 to 80 rows: every
number of 16-row blocks at its edges, ragged last workgroups, one to sixteen K ranges (the
last one shorter) and the fewest columns of K; the same kernel below 33 rows and under
the other epilogues: the decode batches of test_gpu_mid and test_gpu_rows_resident."""
import pytest
import torch

import workloads as WL
from tests.helpers import rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [
    (33, 16, 512), (48, 208, 1024), (49, 2064, 512), (64, 4112, 4608), (64, 1024, 8192), (65, 528, 2560), (80, 8208, 1536), (72, 1040, 13824), (41, 20496, 512)])
def test_rows_gemm_at_the_edges(M, N, K):
    from paper_2410_03960_amd import binding as B
    print(f"M={M} N={N} K={K}", flush=True)
    A = WL.seeded_normal_bf16(1, f"A{M}{K}", (M, K), 0.0, 1.0, device="cuda")
    W = WL.seeded_normal_bf16(2, f"W{N}{K}", (N, K), 0.0, 0.05, device="cuda")
    ref = torch.cat([A.double() @ w.double().T.contiguous() for w in W.split(4096)], 1)
    for out_f32, tol in ((True, 1e-5), (False, 4e-3)):     # fp32 sums of exact products / one bf16 rounding
        assert B.op_gemm_plan("f32" if out_f32 else "bf16", M, N, K, scratch=16 * M * N * 4).kernel == "stream_seq"
        assert rel_err(B.op_gemm_rows(A, W, out_f32=out_f32), ref) <= tol
