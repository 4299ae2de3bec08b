"""bf16 copy of a token-major dY whose rows are no whole number of chunks: its padding is zero and every value in its place, so that dX has the bits
of the same call with the channels filled up by channels of weight zero and gradient zero."""
import pytest
import torch

import paper_2411_11038_amd as ef

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt", (torch.bfloat16, torch.float32), ids=("bf16", "f32"))
@pytest.mark.parametrize("T", (1, 37, 700, 9001))      # one to 64 lanes to a row, several trips
@pytest.mark.parametrize("c_out", tuple(range(1, 18)) + (63, 257, 505, 509, 514, 519, 1031, 2050, 4099))
def test_same_bits_as_filled_up(c_out, T, dt):
    c_in, full = 64, (c_out + 7) // 8 * 8
    g = torch.Generator(device="cuda")
    g.manual_seed(T + c_out)
    x = torch.randn(T, c_in, generator=g, device="cuda").to(dt)
    w = torch.zeros(full, c_in, device="cuda")
    w[:c_out] = torch.randn(c_out, c_in, generator=g, device="cuda") * 0.05
    dy = torch.zeros(T, full, device="cuda", dtype=dt)
    dy[:, :c_out] = torch.randn(T, c_out, generator=g, device="cuda").to(dt)
    fx = ef.fakequant_fwd(x, ef.ACT_PER_TENSOR_ASYM, 8)
    dx = []
    for n in (c_out, full):
        wn = w[:n].contiguous()
        fw = ef.fakequant_fwd(wn, ef.W_PER_ROW_SYM, 8)
        dx.append(ef.linear_bwd(dy[:, :n].contiguous(), fx["codes"], fx["clip_bits"], x, fx["scale"], fx["zero_point"], fw["codes"],
                                fw["clip_bits"], wn, fw["scale"], None, dx_kernel=ef.DX_KERNEL_BF16_PINNED)["dx"])
    assert torch.equal(dx[0], dx[1])
