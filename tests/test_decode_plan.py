"""The choice of kernel and key splits of single-query attention by shape (host code, no GPU)."""
import os

import pytest

from paper_2410_03960_amd import binding as B


@pytest.fixture(scope="module", autouse=True)
def built():
    if not os.path.exists(B.LIB_PATH):
        from paper_2410_03960_amd import build
        build.build(verbose=False)


# Few long rows over an e4m3 cache: workgroups that fill the CUs evenly.  Between two and three to a CU, or three (their
# limit) to each, the same keys take 12 to 25 % longer.
@pytest.mark.parametrize("rows,keys", [(8, 20000), (4, 40000), (16, 8192), (32, 4096)])
@pytest.mark.parametrize("heads", [32, 64])
def test_splits_of_few_long_rows_fill_the_cus_evenly(heads, rows, keys):
    plan = B.op_attention_decode_plan([keys] * rows, heads, 8, 128, fp8=True)
    wgs = rows * 8 * -(-keys // plan.split_keys(keys))
    assert not 512 < wgs <= 768


# A step over a cache with a scale per token takes half again what another does: a chain of three or more is split.
@pytest.mark.parametrize("lens", [[500], [500] * 8, [500] * 4 + [480]], ids=str)
@pytest.mark.parametrize("heads,hd", [(32, 128), (64, 64)])
def test_short_rows_with_token_scales_are_split(heads, hd, lens):
    assert B.op_attention_decode_plan(lens, heads, 8, hd, fp8=True, per_token=True).n_splits > 1


# Many rows: no split (64 rows x 2048 e4m3 keys 54 us and no combine pass, 2 splits 57 and one).
@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("lens", [[2048] * 64, [900] * 160, [40] * 200, [1] * 1000], ids=lambda v: f"{len(v)}x{v[0]}")
def test_many_rows_are_not_split(lens, fp8):
    assert B.op_attention_decode_plan(lens, 32, 8, 128, fp8=fp8).n_splits == 1


@pytest.mark.parametrize("n", [1, 127, 128, 4096, 10 ** 6])
def test_splits_stay_within_the_limit_of_the_combine_pass(n):
    for rows in (1, 3, 700):
        for fp8 in (False, True):
            plan = B.op_attention_decode_plan([n] * rows, 32, 4, 128, fp8=fp8)
            assert 1 <= plan.n_splits <= min(32, -(-n // 128))


def test_refusals():
    for kw in (dict(n_keys=[]), dict(n_keys=[0]), dict(head_dim=96), dict(n_q_heads=12), dict(n_kv_heads=0)):
        with pytest.raises(Exception):
            B.op_attention_decode_plan(**{**dict(n_keys=[5], n_q_heads=8, n_kv_heads=8, head_dim=64), **kw})


# One or two query heads per KV head over a bf16 cache: the unit that is ahead at the shape (us, vector / matrix: 7.8 / 9.8, 8.8 / 9.8,
# 30.8 / 49, 13 / 21, 23.6 / 28.7, 12.0 / 13.0 in 64-wide heads; 7.9 / 5.9, 21.0 / 18.4, 31.6 / 21.9, 22.2 / 18.4, 28.3 / 23.1).
@pytest.mark.parametrize("lens,shape,unit", [
    ([778], (8, 8, 128), "vector"), ([778], (16, 8, 128), "vector"), ([40] * 200, (32, 32, 128), "vector"), ([40] * 200, (12, 12, 128), "vector"),
    (list(range(500, 4000, 450)), (8, 8, 128), "vector"), ([1600] * 6, (8, 8, 64), "vector"),
    ([100], (8, 8, 128), "matrix"), ([300] * 64, (8, 8, 128), "matrix"), ([20000], (8, 8, 128), "matrix"), ([300] * 64, (16, 8, 128), "matrix"),
    ([1200] * 48, (8, 8, 64), "matrix"), ([778], (16, 8, 64), "matrix")], ids=lambda v: f"{len(v)}x{v[0]}" if isinstance(v, list) else str(v))
def test_unit_of_one_or_two_heads(lens, shape, unit):
    assert B.op_attention_decode_plan(lens, *shape).unit == unit
    for heads in (4, 8):                         # ... and more heads, or e4m3 codes: always the matrix unit
        assert B.op_attention_decode_plan(lens, heads * shape[1], *shape[1:]).unit == "matrix"
    assert B.op_attention_decode_plan(lens, *shape, fp8=True).unit == "matrix"
