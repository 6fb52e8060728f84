"""The choice of GEMM kernel by shape (host code, no GPU)."""
import os

import pytest

from paper_2410_03960_amd import binding as B


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
