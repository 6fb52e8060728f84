"""The rotation rounds in one stated way (b s and a s rounded, the other products fused to them) whichever kernel a batch's K goes through:
the cached K of rows whose projections are exact, bit for bit.  Rows are 16 times a unit vector of 256 entries, so that each product
is 16 times a weight, 1/rms is one and only the rotation rounds."""
import pytest
import torch

import workloads as WL
from workloads.configs import ModelShape, Workload
from tests import gpu_helpers as G

pytestmark = pytest.mark.gpu

SHAPES = {hd: ModelShape(4, 256, 1024 // hd, 1024 // hd, hd, 256, 256, 1e4, 1e-30) for hd in (64, 128)}
# weight streaming, tiles of 64 to 160 rows with activations through registers, the large loop at each height; row-major weights
ROWS = {True: (60, 500, 700, 1000, 1300, 1700, 2000, 2300), False: (300, 1000, 1300)}


@pytest.mark.parametrize("packed,rows", [(p, r) for p in ROWS for r in ROWS[p]])
@pytest.mark.parametrize("hd", sorted(SHAPES))
def test_cached_k_to_the_bit(hd, packed, rows):
    from paper_2410_03960_amd import binding as B
    sh = SHAPES[hd]
    weights = G.device_weights(WL.make_weights(Workload(f"rotation{hd}", sh, l=1, g=1, seed=3211), "cpu", keep=True))
    for j in range(1, 4):
        weights[f"norm1.{j}"].fill_(1.0)
    ctx = B.Context(sh, weights, 1, 1, packed_weights=packed)
    print(hd, packed, rows, B.op_gemm_plan("kv", rows, 6144, 256, packed=packed, head_dim=hd), flush=True)
    hidden = torch.zeros(rows, 256, dtype=torch.bfloat16, device="cuda")
    pos = torch.arange(rows)
    hidden[pos, pos % 256] = 16.0
    n_blocks = (rows + 15) // 16
    cache = B.KVCache(ctx.n_cache_layers, n_blocks, sh.n_kv_heads, hd, torch.arange(n_blocks).int().view(1, -1), [0])
    ctx.kv_from_hidden(hidden, [rows], cache, torch.empty(ctx.workspace_bytes(rows, 1), dtype=torch.uint8, device="cuda"))
    angle = pos.double()[:, None] * 1e4 ** (-2.0 * torch.arange(hd // 2).double() / hd)
    c, s = angle.cos().float().double()[:, None], angle.sin().float().double()[:, None]      # [rows, 1, hd / 2]
    for j in range(1, 4):
        k = 16.0 * weights[f"wk.{j}"].cpu().double().T[pos % 256].view(rows, -1, hd)
        a, b = k[..., :hd // 2], k[..., hd // 2:]
        # (products of two fp32 values are exact in 64 bits; the sum is rounded once to fp32)
        want = torch.cat([(a * c - (b * s).float().double()).float(), (b * c + (a * s).float().double()).float()], -1).bfloat16()
        assert torch.equal(cache.data[j, 0, :rows].cpu(), want), (j, int((cache.data[j, 0, :rows].cpu() != want).sum()))
        assert torch.equal(cache.data[j, 1, :rows].cpu(), (16.0 * weights[f"wv.{j}"].cpu().float()).T[pos % 256].view(rows, -1, hd).bfloat16())
