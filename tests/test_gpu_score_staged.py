"""Scoring with the query rows staged through LDS: five to sixteen wavefronts, row counts that end inside a read of eight rows, one,
two and three tiles, three that are cut to two, and shapes on either side of what leaves room for it; against the oracle."""
import pytest

from test_gpu_score_tiles import test_against_the_oracle as check

pytestmark = pytest.mark.gpu

CASES = [  # ctx, B, M, Hq, Hkv, last node
    ([16 * 40], 16, 33, 16, 4, 32),                  # 132 rows: five wavefronts, four rows in the last block
    ([64 * 900], 64, 45, 32, 8, 11),                 # 180 rows: six
    ([64 * 100, 64 * 700], 64, 41, 40, 8, 40),       # 205 rows: seven
    ([32 * 2048] * 3, 32, 60, 32, 8, 59),            # 1536 tiles: two a workgroup, at 64 channels three
    ([16 * 1300] * 4, 16, 45, 32, 8, 20),            # 1312 tiles, six wavefronts: three
    ([32 * 2048] * 4 + [1], 32, 57, 32, 8, 0),       # 2560 tiles: four, no room to stage
    ([64 * 250], 64, 60, 40, 8, 30),                 # 300 rows: ten
    ([64 * 250], 64, 128, 32, 8, 127),               # 512 rows: sixteen
]


@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("reduce", ["mean", "max", "last"])
@pytest.mark.parametrize("ctx,B,M,Hq,Hkv,last", CASES)
def test_staged_against_the_oracle(gpu_lib, ctx, B, M, Hq, Hkv, last, reduce, D):
    check(gpu_lib, ctx, B, M, Hq, Hkv, last, reduce, D)
