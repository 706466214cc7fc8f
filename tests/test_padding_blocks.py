"""Which workgroups a GEMM of several launches (k beyond 2^17) has, seen on the CPU: the library runs on a stand-in for the HIP runtime
that records the launches with their grids."""
import json
import re

import pytest

from test_launch_routes import PRODUCTS, STAND_IN, run_on_stand_in

# (m, n, k, N) and the workgroups of a folding launch
CASES = [(64, 100, 200000, 6, 4 * 6),                # one of four blocks of 128 x 128: all four are computed
         (200, 100, 150000, 14, 4 * 14),             # two of four
         (256, 100, 262144, 8, 4 * 8),
         (300, 200, 200000, 15, 6 * 15),             # six of eight: those alone
         (1000, 60, 150000, 16, 16 * 16),            # half of 256 blocks: one each for the compute units
         (1000, 60, 150000, 17, 8 * 17)]             # of 272: those in use


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    stand_in = re.sub(r"strcat\(names, known\[i\]\.name\);", r'sprintf(names + strlen(names), "%s %u", known[i].name, g.x);', STAND_IN)
    assert "g.x" in stand_in
    return run_on_stand_in(tmp_path_factory.mktemp("padding"), PRODUCTS, stand_in, data=json.dumps([("d",) + c[:4] for c in CASES]))


@pytest.mark.parametrize("m,n,k,N,want", CASES)
def test_blocks_of_a_folding_launch(launches, m, n, k, N, want):
    for names in launches["d %d %d %d %d" % (m, n, k, N)]:
        folds = [x for x in names if re.search(r"k_int8_gemmI(Li\d+E){6}Li3E", x)]
        assert len(folds) == -(-k // 131072) - 1 and len(folds) >= 1, names
        assert {int(x.split()[-1]) for x in folds} == {want}, folds
