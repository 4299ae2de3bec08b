"""dX of a channel-major dY on 128 x 256 tiles: one and several rounds of blocks, whole and ragged K stages, fp32 x and bf16, against the
tiles of 192 on a token-major copy, which add the same products in the same order (bit for bit)."""
import pytest
import torch

import paper_2411_11038_amd as ef

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("size", [(8192, 1024, 1024), (8192, 1024, 1000), (4096, 2048, 520), (4096, 2048, 4096), (16384, 1024, 300),
                                  (12288, 3072, 72), (12288, 768, 8), (7936, 1024, 200)], ids=str)
@pytest.mark.parametrize("x_dt", (torch.bfloat16, torch.float32), ids=("bf16", "f32"))
def test_against_tiles_of_192(size, x_dt):
    T, c_in, c_out = size
    assert ef.linear_bwd_plan(T, c_in, c_out, 0, ef.BF16, ef.DY_CHANNEL_MAJOR)["dx_tile"] == 128
    g = torch.Generator(device="cuda")
    g.manual_seed(c_out)
    x = torch.randn(T, c_in, generator=g, device="cuda").to(x_dt)
    w = torch.randn(c_out, c_in, generator=g, device="cuda") * 0.05
    dy = torch.randn(c_out, T, generator=g, device="cuda").bfloat16()
    fx = ef.fakequant_fwd(x, ef.ACT_PER_TENSOR_ASYM, 8)
    fx["scale"] *= 0.6                                 # some are clipped
    ef.fakequant_fwd(x, ef.ACT_PER_TENSOR_ASYM, 8, init_minmax=False, out=fx)
    fw = ef.fakequant_fwd(w, ef.W_PER_ROW_SYM, 8)
    args = (dy, fx["codes"], fx["clip_bits"], x, fx["scale"], fx["zero_point"], fw["codes"], fw["clip_bits"], w, fw["scale"], None)
    got = ef.linear_bwd(*args, dy_layout=ef.DY_CHANNEL_MAJOR)
    want = ef.linear_bwd(*args, dy_layout=ef.DY_CHANNEL_MAJOR, dx_kernel=ef.DX_KERNEL_BF16_PINNED)
    assert torch.equal(got["dx"], want["dx"])
    for n in ("ds_x", "dz_x"):                         # summed in another order of tiles
        assert (got[n] - want[n]).abs() <= 1e-3 * (want[n].abs() + want["dx"].float().norm())
