"""The plans of the 16-bit products (host arithmetic): every plan can be
launched, and long products of any width take the phased 256 x 256 tile."""

import pytest

from internal import gemm16_partial_bound, plan_gemm16

PHASED = 17
BN = {6: 128, 8: 256, 12: 128, 14: 128, 16: 256, PHASED: 256}

ROWS = [1, 17, 60, 128, 129, 209, 257, 372, 513, 640, 889, 1025, 1500, 2049,
        2300, 2445, 3092, 4097, 6000, 9000, 18020, 70001]
# the 8B-shaped layer (a table of its own), the smallest, odd and large ones
WIDTHS = [(4096, 12288), (128, 64), (384, 1088), (1152, 3072), (2048, 5632),
          (2944, 8192), (5120, 13824), (8192, 22016)]


def _products(d, ffn):
    return ((3 * d, d, True), (d, d, False), (2 * ffn, d, False),
            (d, ffn, False))


@pytest.mark.parametrize("d,ffn", WIDTHS)
def test_every_plan_can_be_launched(d, ffn):
    for N, K, rotary in _products(d, ffn):
        for M in ROWS:
            p = plan_gemm16(M, N, K, rotary)
            assert p.tile in BN and N % BN[p.tile] == 0, (M, N, K, p.tile)
            assert p.ksplit in (1, 2, 3, 4, 5, 6, 8)
            slabs = K // 64
            part = -(-slabs // p.ksplit)
            assert -(-slabs // part) == p.ksplit, "a split without work"
            if p.ksplit > 1:
                assert 4 * p.ksplit * M * N <= gemm16_partial_bound(M, N, K)


@pytest.mark.parametrize("d,ffn", [(3072, 8192), (4608, 12288), (5120, 13824),
                                   (8192, 22016)])
@pytest.mark.parametrize("M", [3000, 4000, 8000])
def test_long_products_take_the_phased_tile(d, ffn, M):
    names = ("qkv", "o", "gu", "dn")
    plans = {n: plan_gemm16(M, *p).tile
             for n, p in zip(names, _products(d, ffn))}
    assert plans["qkv"] == plans["gu"] == PHASED, plans
    if d >= 5120:
        assert plans["dn"] == PHASED, plans
    assert 16 not in plans.values(), plans


@pytest.mark.parametrize("M", [2171, 2300, 2445])
def test_down_projection_keeps_its_split(M):
    # 242 us at 2250 rows, over 261 on the same tile without the split
    p = plan_gemm16(M, 4096, 12288, False)
    assert (p.tile, p.ksplit) == (PHASED, 3)
