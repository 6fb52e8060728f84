"""Prefill attention where the items are few: at most one per CU (two groups of
waves share the key tiles of an item), at most one per workgroup (none is pulled
from a queue), one more than that, one queue instead of eight; key tiles in odd and
even numbers, sequences of one tile, whose second group has nothing."""
import pytest

from tests.test_gpu_ops import test_prefill_attention_matches_bruteforce_softmax as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hd,Hq,Hkv,lens", [
    (128, 32, 8, [1]), (128, 32, 8, [64, 65, 63, 1]), (64, 32, 8, [128, 129, 191, 2]), (128, 8, 2, [1000]),
    (128, 32, 8, [897, 128]), (128, 32, 8, [897, 129]), (64, 32, 4, [1025, 7]),             # 256 and 288 items
    (128, 64, 8, [513, 449]), (64, 64, 8, [900, 130]), (128, 40, 8, [1500, 70]),            # 512, 576 and 520 items: 8 queues
    (64, 12, 4, [300, 17]), (128, 12, 4, [2400, 70, 70, 300]), (64, 4, 4, [129, 1, 1, 400]),   # one queue
], ids=str)
def test_few_items(hd, Hq, Hkv, lens):
    check(hd, Hq, Hkv, lens)
