"""Weight-streaming GEMM of up to 16 rows with all rows resident in LDS: both
workgroup widths, ragged last workgroup, the row counts at the edges, the largest
operand LDS holds, and the shapes next to the rule's line that keep another form."""
import pytest
import torch

import workloads as WL
from tests.helpers import rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [
    (2, 13120, 512), (5, 16384, 1024), (16, 14352, 4096), (8, 28672, 512), (3, 32768, 1024), (16, 32064, 512), (9, 14336, 8704),
    (1, 14336, 512), (16, 8192, 4096), (2, 12288, 512), (16, 13104, 512), (10, 14336, 8704), (17, 14336, 512)])
def test_rows_gemm_at_the_edges(M, N, K):
    from paper_2410_03960_amd import binding as B
    print(f"M={M} N={N} K={K}", flush=True)
    A = WL.seeded_normal_bf16(1, f"A{M}{K}", (M, K), 0.0, 1.0)
    W = WL.seeded_normal_bf16(2, f"W{N}{K}", (N, K), 0.0, 0.05, device="cuda")
    ref = A.double() @ W.cpu().double().T
    for out_f32, tol in ((True, 1e-5), (False, 4e-3)):     # fp32 sums of exact products / one bf16 rounding
        assert rel_err(B.op_gemm_rows(A.cuda(), W, out_f32=out_f32).cpu(), ref) <= tol
