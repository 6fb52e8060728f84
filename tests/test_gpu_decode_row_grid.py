"""Single-query attention over e4m3 heads of 64: from 33 rows on the grid's rows are rounded up to whole eights, and the workgroups
of the extra rows do nothing; with more than 1024 workgroups it goes by pairs of heads.  Row counts on both sides of the rules and of
a multiple of eight."""
import pytest
import torch

from paper_2410_03960_amd import binding as B
from tests.test_gpu_ops import test_single_query_attention_over_paged_cache as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [31, 32, 33, 39, 40, 41])
@pytest.mark.parametrize("mode", ["fp8_head", "fp8_token"])
def test_rows_around_the_rule(rows, mode):
    check(64, 8, 4, mode, [1 + 37 * i % 300 for i in range(rows)])


# More than 1024 workgroups: eight rows of a head and the same rows of its neighbour take turns.  The order leaves every row's result as it
# is, to the bit, in calls of few rows (up to 128 keys there is one key split everywhere).
@pytest.mark.parametrize("rows,heads", [(128, 8), (129, 8), (211, 5), (520, 2)])      # 1024 workgroups, by rows; more; an odd number of heads; one pair
@pytest.mark.parametrize("per_token", [False, True])
def test_pairs_of_heads(rows, heads, per_token):
    gen = torch.Generator().manual_seed(rows)
    lens = [1 + 37 * i % 128 for i in range(rows)]
    table = torch.randperm(rows * 8, generator=gen).int().view(rows, 8)
    q = torch.randn(rows, heads * 128, generator=gen).bfloat16().cuda()
    k, v = (torch.randn(rows * 128, heads, 64, generator=gen).to(torch.float8_e4m3fn).view(torch.uint8).cuda() for _ in range(2))
    scales = [(0.5 + torch.rand(rows * 128 if per_token else heads, generator=gen)).cuda() for _ in range(2)]

    def call(a, b):
        assert B.op_attention_decode_plan(lens[a:b], 2 * heads, heads, 64, fp8=True, per_token=per_token).n_splits == 1
        return B.op_attention_decode(q[a:b].contiguous(), lens[a:b], k, v, table[a:b].contiguous(), 2 * heads, heads, 64, *scales, per_token=per_token)
    assert torch.equal(call(0, rows), torch.cat([call(a, min(a + 24, rows)) for a in range(0, rows, 24)]))


@pytest.mark.parametrize("mode", ["fp8_head", "fp8_token"])
def test_pairs_of_heads_in_key_splits(mode):
    lens = [4000] + [1 + 37 * i % 300 for i in range(70)]
    assert len(lens) * 8 * B.op_attention_decode_plan(lens, 16, 8, 64, fp8=True, per_token=mode == "fp8_token").n_splits > 2 * 1024
    check(64, 16, 8, mode, lens)
