"""Single-query attention on the matrix unit where one workgroup walks more than the 4096 keys whose
block ids it looks up at once: rows of so many keys that every split does, one and two look-ups
later, splits that end just behind one, beside rows that end beside that line; against 64 bits."""
import pytest
import torch

from paper_2410_03960_amd import binding as B
from tests.helpers import rel_err

pytestmark = pytest.mark.gpu

MOST = 32      # splits of a row


@pytest.mark.parametrize("n_keys,looks", [
    ([MOST * 4224, 4095, 4096, 4097], 2),                   # 33 steps of 128 keys to a split: the last one behind the second look-up
    ([MOST * 8320 + 1, 8191, 8192, 8193, 33], 3),            # 65 steps and a key
], ids=["two", "three"])
@pytest.mark.parametrize("fp8", [False, True])
def test_rows_beyond_one_block_id_load(fp8, n_keys, looks):
    Hq, Hkv, hd = 8, 1, 64
    plan = B.op_attention_decode_plan(n_keys, Hq, Hkv, hd, fp8=fp8)
    assert plan.unit == "matrix" and -(-plan.split_keys(n_keys[0]) // 4096) >= looks     # (split over at most MOST: more keys otherwise)
    need = [(n + 15) // 16 for n in n_keys]
    gen = torch.Generator().manual_seed(27)
    order, at = torch.randperm(sum(need) + 3, generator=gen).int(), 0
    table = torch.full((len(n_keys), max(need)), -1, dtype=torch.int32)
    for b, n in enumerate(need):
        table[b, :n] = order[at:at + n]
        at += n
    slots = order.numel() * 16
    k, v = (torch.randn(slots, Hkv, hd, generator=gen).cuda() for _ in range(2))
    q = torch.randn(len(n_keys), Hq * hd, generator=gen).bfloat16().cuda()
    kw = {}
    if fp8:
        kw = {"scale_k": torch.full((Hkv,), 0.02).cuda(), "scale_v": torch.full((Hkv,), 0.03).cuda()}
        k, v = ((x / s).clamp(-448, 448).to(torch.float8_e4m3fn) for x, s in ((k, 0.02), (v, 0.03)))
        kd, vd = k.double() * 0.02, v.double() * 0.03
        k, v = k.view(torch.uint8), v.view(torch.uint8)
    else:
        k, v = k.bfloat16(), v.bfloat16()
        kd, vd = k.double(), v.double()
    out = B.op_attention_decode(q, n_keys, k, v, table, Hq, Hkv, hd, **kw)
    for b, n in enumerate(n_keys):
        s = (table[b].long()[:, None] * 16 + torch.arange(16)).view(-1)[:n].cuda()
        qb = q[b].double().view(Hkv, Hq // Hkv, hd)
        p = torch.softmax(torch.matmul(qb, kd[s].permute(1, 2, 0).contiguous()) / hd ** 0.5, -1)
        # (the steps behind one look-up read from other blocks: 0.2 of the result and more)
        assert rel_err(out[b].double().cpu(), torch.matmul(p, vd[s].permute(1, 0, 2).contiguous()).view(-1).cpu()) <= 1e-2, b
