"""Kernel and tile of the dX product where the cost tables chose measurably worse ones before: sizes with the measured times of
the candidates beside them (us, the whole backward call with k = 0).  Host queries, no GPU."""
import pytest

import paper_2411_11038_amd as ef

# T, c_in, c_out, dtype, (kernel, tile) as in EFQAT_PLAN_DX_KERNEL and EFQAT_PLAN_DX_TILE
LINEAR = [
    # 256 x 256 tiles of a bf16 copy of dY have no straight-line epilogue: not priced as if they had
    (5888, 5888, 1716, ef.BF16, (1, 192)),        # 175; two stages of 256: 205
    (16384, 2048, 1020, ef.BF16, (0, 128)),       # 105; 119
    (8192, 4096, 4100, ef.BF16, (0, 256)),        # 346; ring of 192: 389
]


@pytest.mark.parametrize("case", LINEAR, ids=str)
def test_dx_plan(case):
    T, c_in, c_out, dtype, want = case
    p = ef.linear_bwd_plan(T, c_in, c_out, 0, dtype)
    assert (p["dx_kernel"], p["dx_tile"]) == want
