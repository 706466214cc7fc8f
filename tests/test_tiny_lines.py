"""Where the one-launch form of the smallest products ends by the operands of a compute unit, seen on the CPU: 64 Kp N bytes with tiles of
32 x 32 and 32 Kp N with 16 x 16."""
import json

import pytest

from test_launch_routes import PRODUCTS, run_on_stand_in

# prepared operands: (m, n, k, N) and whether GEMMs and accumulation are one launch
CASES = [(100, 100, 512, 14, True), (100, 100, 512, 15, False),        # 16 x 16: Kp N = 7168 and 7680
         (100, 100, 384, 16, True), (100, 100, 385, 14, True),
         (400, 400, 512, 8, True), (400, 400, 512, 9, False),          # 32 x 32: 4096 and 4608
         (400, 400, 256, 16, True), (400, 400, 257, 11, False),        # 4096 and 4224
         (100, 100, 256, 17, True), (100, 100, 257, 17, False)]        # a second modulus: 512 elements of k in a row


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    return run_on_stand_in(tmp_path_factory.mktemp("lines"), PRODUCTS, data=json.dumps([("d",) + c[:4] for c in CASES]))


@pytest.mark.parametrize("m,n,k,N,one", CASES)
def test_prepared_products_on_both_sides(launches, m, n, k, N, one):
    prepared = launches["d %d %d %d %d" % (m, n, k, N)][2]
    assert ("k_tiny_product" in prepared[0]) == one and len(prepared) == (1 if one else 2), prepared
