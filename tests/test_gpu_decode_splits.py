"""Single-query attention at the edges of the key splits: whole blocks of 32 keys
on few short rows, one and several rounds of workgroups on the matrix-unit
kernels, rows of very different length (they run longest first)."""
import pytest

from tests.test_gpu_ops import test_single_query_attention_over_paged_cache as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hd,Hq,Hkv,mode,lens", [
    (128, 32, 8, "bf16", [1, 31, 32, 33]), (128, 32, 8, "bf16", [778]), (64, 32, 8, "bf16", [99, 211, 64, 65]), (128, 8, 8, "bf16", [1023, 1]),
    (128, 64, 8, "bf16", [4100, 127, 128, 129, 1]), (64, 16, 2, "bf16", [200, 3000]),
    (128, 32, 8, "fp8_head", [128, 129, 1, 2000]), (128, 64, 8, "fp8_token", [1500, 16, 700]), (64, 4, 4, "fp8_head", [255, 257]),
    (128, 32, 8, "fp8_token", [60 + 17 * i for i in range(40)]), (128, 32, 8, "bf16", [5 + 23 * i for i in range(50)]),
], ids=str)
def test_key_splits(hd, Hq, Hkv, mode, lens):
    check(hd, Hq, Hkv, mode, lens)
