"""Kernels and tiles of the products where the cost tables chose measurably worse ones before: sizes with the measured times of
the candidates beside them (us, the whole backward call with k = 0).  Host queries, no GPU."""
import pytest

import paper_2411_11038_amd as ef

# T, c_in, c_out, dtype, (kernel, tile) as in EFQAT_PLAN_DX_KERNEL and EFQAT_PLAN_DX_TILE
LINEAR = [
    # 256 x 256 tiles of a bf16 copy of dY have no straight-line epilogue: not priced as if they had
    (5888, 5888, 1716, ef.BF16, (1, 192)),        # 175; two stages of 256: 205
    (16384, 2048, 1020, ef.BF16, (0, 128)),       # 105; 119
    (8192, 4096, 4100, ef.BF16, (0, 256)),        # 346; ring of 192: 389
    # few K stages under a large dX: bound by memory, more so on 64-wide tiles
    (11474, 7176, 128, ef.BF16, (0, 128)),        # 142; 64: 177
    (16384, 5872, 16, ef.F32, (0, 128)),          # 230; 64: 271
    (15488, 6656, 64, ef.F32, (0, 128)),          # 227; 64: 262
    (15872, 8704, 17, ef.BF16, (0, 128)),         # 207; 64: 256, ring of 128: 245
]


@pytest.mark.parametrize("case", LINEAR, ids=str)
def test_dx_plan(case):
    T, c_in, c_out, dtype, want = case
    p = ef.linear_bwd_plan(T, c_in, c_out, 0, dtype)
    assert (p["dx_kernel"], p["dx_tile"]) == want


def test_dw_plan_of_gathered_codes():
    # two blocks of 128 x 128 a CU, not three: 64-row tiles 582 us, 24 slices of 128-row tiles 616
    p = ef.conv_bwd_plan(64, 47, 47, 512, 384, 2, 2, 1, 1, 192)
    assert (p["dw_operands"], p["dw_tile"]) == (2, 64)


# T, c_in, c_out, rows and columns of a dX tile of a channel-major dY; us on 64 x 128 / 128 x 128 / 128 x 256 / 256 x 256
CHANNEL_MAJOR = [
    (12288, 768, 768, (128, 256)),     # 32.1 / 32.6 / 31.4 / 29.5
    (2048, 3072, 1536, (128, 256)),    # 34.0 / 32.0 / 29.4 / 39.6
    (8192, 768, 1536, (128, 256)),     # 34.0 / 32.1 / 29.6 / 39.8
    (2048, 3072, 8192, (128, 256)),    # 139 / 126 / 105 / 138
    (12288, 3072, 768, (128, 256)),    # 108 / 100 / 85.5 / 102
    (8192, 4096, 4096, (256, 256)),    # 360 / 316 / 250 / 229
    (8192, 11008, 4096, (256, 256)),   # 643, 4 % more on 128 x 256
    (1024, 4096, 3072, (128, 128)),    # 42.1 / 39.6 / 44.4 / 61.8
]


@pytest.mark.parametrize("case", CHANNEL_MAJOR, ids=str)
def test_dx_plan_of_a_channel_major_gradient(case):
    T, c_in, c_out, want = case
    t = ef.linear_bwd_dx_tile(T, c_in, c_out, 0, ef.BF16, ef.DY_CHANNEL_MAJOR)
    assert (t["rows"], t["columns"]) == want


# T, c_in, c_out, k, with a second stream, LDS stages of the ring on 64 x 64 tiles; us with three / eight
RING = [
    (512, 768, 512, 0, False, 3),        # 12.6 / 13.5    short contractions
    (512, 768, 1792, 0, False, 3),       # 17.6 / 17.8
    (512, 768, 2048, 0, False, 8),       # 18.2 / 17.7
    (1000, 777, 4096, 0, False, 8),      # 33.8 / 27.5
    (1024, 1024, 8000, 2000, False, 8),  # 70.6 / 67.0
    (1024, 1024, 8000, 2000, True, 3),   # 64.0 / 72.1    no room for the blocks of the dW product
    (512, 1024, 8000, 2000, True, 8),    # 58.4 / 53.8    ... but where half of the CUs have no dX block
    (512, 1024, 4608, 2304, True, 3),    # 47.7 / 50.1    ... and the contraction is long
    (153, 640, 4608, 2304, True, 8),     # 41.6 / 39.9
    (64, 1024, 4816, 0, False, 3),       # 38.1 / 39.0    rows that are no whole number of lines
    (512, 1024, 8008, 0, False, 3),      # 71.9 / 72.6
    (2000, 333, 4104, 0, False, 8),      # 35.5 / 31.8    ... and tiles over the edge
]


@pytest.mark.parametrize("case", RING, ids=str)
def test_ring_of_dx_tiles(case):
    T, c_in, c_out, k, side, stages = case
    assert ef.linear_bwd_plan(T, c_in, c_out, k)["one_grid"] == 0
    assert ef.linear_bwd_dx_tile(T, c_in, c_out, k, side_stream=side) == dict(rows=64, columns=64, stages=stages)


# tokens, C_in, C_out, columns of a block; us by 16 / 32 / 48 / 64 columns
FEW_TOKENS = [
    (16, 96, 11008, 16),      # 3.7 / 4.2 / 4.7 / 4.4    short rows: one group of 16
    (64, 256, 4112, 16),      # 4.4 / 5.4 / 6.2 / 7.1
    (16, 1024, 4112, 16),     # 4.5 / 4.8 / 5.8 / 5.8
    (64, 192, 8192, 16),      # 4.5 / 5.1 / 6.0 / 6.8
    (16, 333, 11008, 16),     # 6.7 / 8.0 / 8.8 / 9.4    ... not aligned
    (20, 1500, 8192, 16),     # 10.2 / 10.9 / 13.3 / 15.6
    (9, 1136, 11251, 16),     # 4.7 / 5.3 / 5.2 / 5.8      few tokens: three groups pay late
    (5, 2980, 8309, 16),      # 10.1 / 12.0 / 11.6 / 12.7
    (16, 96, 28672, 64),      # 6.4 / 6.5 / 7.8 / 4.9    many columns
    (32, 1024, 32768, 64),    # 18.2 / 15.6 / 14.6 / 12.8
    (16, 4096, 11008, 48),    # 17.1 / 18.3 / 15.8 / 17.7
    (64, 4096, 6000, 32),     # 24.2 / 18.2 / 20.6 / 23.8
    (16, 3001, 28672, 64),    # 58.2 / 51.0 / 53.5 / 43.9
]


@pytest.mark.parametrize("case", FEW_TOKENS, ids=str)
def test_columns_of_a_block_of_few_tokens(case):
    T, c_in, c_out, columns = case
    assert ef.linear_fwd_plan(T, c_in, c_out) == dict(few_tokens=1, columns=columns)
