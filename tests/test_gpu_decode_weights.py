"""Softmax weights of single-query attention over a bf16 cache, one to eight query heads per KV head: their bits (a result
that is what nearly cancelling values leave) and infinite values, against 64 bits."""
import pytest
import torch

from tests.helpers import rel_err

pytestmark = pytest.mark.gpu

HEADS = [(8, 8, 128), (8, 4, 128), (16, 4, 128), (16, 2, 128), (8, 8, 64), (32, 4, 64)]


def _run(q, n, k, v, Hq, Hkv, hd):
    """Rows of n keys each, their blocks one after the other; k, v: CPU bf16 [rows, n, Hkv, hd]"""
    from paper_2410_03960_amd import binding as B
    rows, nb = q.shape[0], (n + 15) // 16
    ck, cv = (torch.zeros(rows, nb * 16, Hkv, hd).bfloat16() for _ in range(2))
    ck[:, :n], cv[:, :n] = k, v
    table = torch.arange(rows * nb).int().view(rows, nb)
    out = B.op_attention_decode(q.cuda(), [n] * rows, ck.view(-1, Hkv, hd).cuda(), cv.view(-1, Hkv, hd).cuda(), table, Hq, Hkv, hd)
    return out.cpu().view(rows, Hkv, Hq // Hkv, hd)


@pytest.mark.parametrize("Hq,Hkv,hd", HEADS)
@pytest.mark.parametrize("n", [3, 300, 2100])
def test_cancelling_values_leave_what_fp32_weights_leave(Hq, Hkv, hd, n):
    R, rows = Hq // Hkv, 8
    gen = torch.Generator().manual_seed(n + Hq + hd)
    q = torch.randn(rows, Hq * hd, generator=gen).bfloat16()
    k = torch.randn(rows, n, Hkv, hd, generator=gen).bfloat16()
    v = torch.zeros(rows, n, Hkv, hd).bfloat16()
    at = (0, n // 2, n - 1)
    ref = torch.zeros(rows, Hkv, hd, dtype=torch.float64)
    for b in range(rows):
        for h in range(Hkv):
            w = torch.softmax(k[b, :, h].double() @ q[b].view(Hkv, R, hd)[h, b % R].double() / hd ** 0.5, 0)
            x = torch.randn(hd, generator=gen).bfloat16()
            left = torch.zeros(hd, dtype=torch.float64)
            for i, key in enumerate(at):    # the second key cancels the first to eight bits, the third three quarters of the rest
                v[b, key, h] = x
                left = left + w[key] * x.double()
                if i < 2:
                    x = (-left * (1 if i == 0 else 0.75) / w[at[i + 1]]).bfloat16()
            ref[b, h] = left
    out = _run(q, n, k, v, Hq, Hkv, hd)
    got = torch.stack([out[b, :, b % R] for b in range(rows)])
    # What is left is about 2^-12.5 of the values (quarter of a bf16 rounding, 2^-10.5 rms): 1.5 units of 2^-23 in a weight (score,
    # exponential, sum) are 2^-10 of it each, beside the result's own rounding of 2^-9.8 rms.  Weights of 16 bits (2^-18.8 rms
    # and up to 2^-17) would show 1e-2 and more.
    assert rel_err(got, ref) <= 5e-3


@pytest.mark.parametrize("Hq,Hkv,hd", HEADS)
@pytest.mark.parametrize("n", [1, 17, 40, 128, 300, 778, 2100])
def test_infinite_values_stay_infinite(Hq, Hkv, hd, n):
    gen = torch.Generator().manual_seed(n)
    q = torch.randn(3, Hq * hd, generator=gen).bfloat16()
    k, v = (torch.randn(3, n, Hkv, hd, generator=gen).bfloat16() for _ in range(2))
    want = torch.zeros(3, Hkv, 1, hd)
    for b, key in enumerate((0, n // 2, n - 1)):
        v[b, key, 0, 5], v[b, key, 1, hd - 1] = float("inf"), -float("inf")
        want[b, 0, 0, 5], want[b, 1, 0, hd - 1] = float("inf"), -float("inf")
    out = _run(q, n, k, v, Hq, Hkv, hd).float()
    assert torch.equal(torch.where(out.isfinite(), 0.0, out), want.expand_as(out))
    w = torch.softmax(torch.matmul(q.double().view(3, Hkv, -1, hd), k.double().permute(0, 2, 3, 1).contiguous()) / hd ** 0.5, -1)
    ref = torch.matmul(w, torch.where(v.isfinite(), v, 0).double().permute(0, 2, 1, 3).contiguous())
    ref[want.expand_as(ref) != 0] = 0
    assert rel_err(torch.where(out.isfinite(), out, 0.0), ref) <= 4e-3     # one bf16 rounding
