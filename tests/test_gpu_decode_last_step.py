"""Single-query attention at the ends of the 32-key steps a wave takes and of the 128-key steps of a workgroup: only a wave's last
step has keys to leave out, and only the steps before it read at offsets that do not depend on the row's length.  The slots of a
row's last block behind its last token hold NaN (values and scales), and in bf16 half of the keys have a score of minus infinity."""
import pytest
import torch

import workloads as WL
from oracle import swiftkv_oracle as O
from paper_2410_03960_amd import binding as B
from tests.gpu_helpers import cosine, rel_err

pytestmark = pytest.mark.gpu
LENS = [1, 15, 16, 17, 31, 32, 33, 47, 48, 63, 64, 65, 96, 97, 127, 128, 129, 143, 159, 160, 161, 255, 256, 257, 383, 513, 640, 800]


@pytest.mark.parametrize("mode", ["bf16", "fp8_head", "fp8_token"])
@pytest.mark.parametrize("hd,Hq,Hkv,rows", [(128, 32, 8, 28), (64, 8, 1, 28), (64, 16, 4, 3)])
def test_ends_of_steps(hd, Hq, Hkv, rows, mode):
    lens = LENS if rows == len(LENS) else [33, 161, 800]     # (few rows: each in several splits)
    need = [(n + 15) // 16 for n in lens]
    bt = torch.zeros((len(lens), max(need)), dtype=torch.int32)
    unseen = torch.ones(sum(need) * 16, dtype=torch.bool)
    perm, pos = torch.from_numpy(WL.seeded_permutation(7, "blocks", sum(need))), 0
    slots = []
    for b, n in enumerate(lens):
        bt[b, :need[b]] = perm[pos:pos + need[b]].to(torch.int32)
        pos += need[b]
        slots.append(bt[b].long()[torch.arange(n) // 16] * 16 + torch.arange(n) % 16)
        unseen[slots[b]] = False
    gen = torch.Generator().manual_seed(hd + Hq)
    shape = (len(unseen), Hkv, hd)
    q = torch.randn(len(lens), Hq * hd, generator=gen).bfloat16()
    sk = sv = None
    if mode == "bf16":
        ck, cv = torch.randn(shape, generator=gen).bfloat16(), torch.randn(shape, generator=gen).bfloat16()
        q[:, ::hd] = 1.0
        for s in slots:      # the first half of a row's keys
            ck[s[:len(s) // 2], :, 0] = float("-inf")
        ck[unseen], cv[unseen] = float("nan"), float("nan")
        kf, vf = ck.double(), cv.double()
    else:
        ck, cv = (torch.randint(0, 256, shape, generator=gen, dtype=torch.uint8) & 0xF7 for _ in range(2))   # (no NaN code)
        ck[unseen], cv[unseen] = 0x7F, 0x7F
        n_scales = Hkv if mode == "fp8_head" else len(unseen)
        sk, sv = (0.001 * 2.0 ** (3 * torch.rand(n_scales, generator=gen)) for _ in range(2))
        if mode == "fp8_token":
            sk[unseen], sv[unseen] = float("nan"), float("nan")
        by = (lambda s: s.double()[None, :, None]) if mode == "fp8_head" else (lambda s: s.double()[:, None, None])
        tab = O.fp8_e4m3fn_decode_table()
        kf, vf = tab[ck.long()] * by(sk), tab[cv.long()] * by(sv)
    dev = lambda t: None if t is None else t.cuda()
    got = B.op_attention_decode(q.cuda(), lens, ck.cuda(), cv.cuda(), bt, Hq, Hkv, hd, dev(sk), dev(sv), per_token=(mode == "fp8_token")).cpu()
    for b, n in enumerate(lens):
        ref = O.gqa_attention(q[b:b + 1].double().view(1, Hq, hd), torch.tensor([n - 1]), kf[slots[b]], vf[slots[b]])
        g = got[b].view(1, Hq, hd)
        # bf16 results (2^-9), the weights in two e4m3 terms (2^-8), and q in two of them: a score's own error is below
        # 2^-8 / sqrt(3) * rms(q) rms(K), with codes of 120 (rms) and scales of 0.0025 below 2^-8 / 5, so that it adds as much to a
        # weight (scales of four times that made it the largest term: 0.012).  Twice the first two
        assert rel_err(g, ref) <= 2 * (2.0 ** -9 + 2.0 ** -8) and cosine(g, ref) >= 0.9995, (b, n, rel_err(g, ref))
