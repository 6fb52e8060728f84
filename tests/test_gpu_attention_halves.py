"""Prefill attention where a 128-query block is two items of 64 (up to half a block per CU): edges of the
halves, last blocks that end in the first or the second half, several sequences, both head sizes, head
counts with one queue and with eight; against the brute-force softmax."""
import pytest
import torch

import workloads as WL
from oracle import swiftkv_oracle as O
from tests.helpers import cosine, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hd,Hq,Hkv,lens", [
    (128, 8, 2, [64]), (128, 8, 2, [65, 1, 7]), (128, 32, 8, [333]), (128, 12, 4, [129, 192]), (128, 3, 1, [193, 63]),
    (64, 8, 4, [32, 33, 128]), (64, 6, 2, [1, 300]), (64, 16, 2, [1023]), (128, 4, 2, [4096]),   # 4096: 32 blocks x 4 heads, the last count that is halved
    (128, 43, 1, [385]),                                                                     # 172 items: the first form past it
])
def test_half_blocks_match_bruteforce_softmax(hd, Hq, Hkv, lens):
    from paper_2410_03960_amd import binding as B
    T = sum(lens)
    q = WL.seeded_normal_bf16(21, f"q{T}", (T, Hq * hd), 0.0, 1.0)
    k = WL.seeded_normal_bf16(22, f"k{T}", (T, Hkv * hd), 0.0, 1.0)
    v = WL.seeded_normal_bf16(23, f"v{T}", (T, Hkv * hd), 0.0, 1.0)
    got = B.op_attention_prefill(q.cuda(), k.cuda(), v.cuda(), lens, Hq, Hkv, hd).cpu()
    off = 0
    for n in lens:
        rows = torch.arange(max(0, n - 400), n)
        ref = O.gqa_attention(q[off:off + n][rows].float().view(-1, Hq, hd), rows,
                              k[off:off + n].float().view(n, Hkv, hd), v[off:off + n].float().view(n, Hkv, hd))
        g = got[off:off + n][rows].view(-1, Hq, hd)
        assert rel_err(g, ref) <= 1e-2 and cosine(g, ref) >= 0.9995, (n, rel_err(g, ref), cosine(g, ref))
        off += n
