"""Which grids the planner gives to the split transform (host only)."""
import pytest

from paper_2409_08090_amd import mils


def odd_part(n):
    while n % 2 == 0:
        n //= 2
    return n


# frequencies whose cheapest split would take 15 residues (n = 15 2^17 .. 15
# 2^21), each of which reads every row when the frequency step leaves none empty
@pytest.mark.parametrize("nf", [1_270_001, 2_550_001, 5_100_001, 10_200_001, 20_300_001])
def test_no_split_of_many_residues(nf):
    d = mils.plan_info(nf // 12, nf, 1e-9)
    assert odd_part(d["n"]) != 15 or d["n"] % 2**17, d


# (and those of up to ten stay: n = R 2^17 .. R 2^21)
@pytest.mark.parametrize("nf,n", [(480_011, 5 << 17), (1_750_001, 9 << 18), (3_500_001, 9 << 19),
                                  (7_000_001, 9 << 20), (9_000_001, 6 << 21),
                                  (16_000_001, 10 << 21)])
def test_split_of_up_to_ten(nf, n):
    assert mils.plan_info(nf // 12, nf, 1e-9)["n"] == n
