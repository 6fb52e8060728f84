"""Single-query attention over e4m3 heads of 64: from 33 rows on the grid's rows are rounded up to whole eights, and the workgroups
of the extra rows do nothing.  Row counts on both sides of the rule and of a multiple of eight."""
import pytest

from tests.test_gpu_ops import test_single_query_attention_over_paged_cache as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [31, 32, 33, 39, 40, 41])
@pytest.mark.parametrize("mode", ["fp8_head", "fp8_token"])
def test_rows_around_the_rule(rows, mode):
    check(64, 8, 4, mode, [1 + 37 * i % 300 for i in range(rows)])
