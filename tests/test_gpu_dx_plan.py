"""The choice of the dX kernel: calls whose workspace or weight codes do not fit the first plan take the wide one, and the tiles
of 64 against the others at sizes around them."""
import pytest
import torch

import paper_2411_11038_amd as ef

pytestmark = pytest.mark.gpu


def _linear(T, c_in, c_out, dt, w_off=0, ws=None, kernel=0):
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    x = torch.randn(T, c_in, generator=g, device="cuda").to(dt)
    w = torch.randn(c_out, c_in, generator=g, device="cuda") * 0.05
    dy = torch.randn(T, c_out, generator=g, device="cuda").to(dt)
    fx = ef.fakequant_fwd(x, ef.ACT_PER_TENSOR_ASYM, 8)
    fw = ef.fakequant_fwd(w, ef.W_PER_ROW_SYM, 8)
    codes = torch.empty(fw["codes"].numel() + 16, dtype=torch.int8, device="cuda")[w_off:w_off + fw["codes"].numel()].view(c_out, c_in)
    codes.copy_(fw["codes"])
    idx, _ = ef.channel_select(w, max(1, c_out // 4))
    return ef.linear_bwd(dy, fx["codes"], fx["clip_bits"], x, fx["scale"], fx["zero_point"], codes, fw["clip_bits"], w,
                         fw["scale"], idx, ws=ws, dx_kernel=kernel)


def _same(a, b, exact_dx=True):
    # every dX kernel adds the same bf16 products in the order of K in fp32; dS_x is summed in another order of tiles
    assert torch.equal(a["dx"], b["dx"]) if exact_dx else (a["dx"] - b["dx"]).abs().max() <= 2.0 ** -7 * a["dx"].abs().max()
    # dW: fp32 sums of the same exact terms, cut into other slices (the bound of bwd_checks.py for that)
    assert (a["dw"] - b["dw"]).abs().max() <= 2e-4 * a["dw"].abs().max()
    for n in ("ds_x", "dz_x"):
        assert (a[n] - b[n]).abs() <= 1e-3 * (a[n].abs() + a["dx"].float().norm())


@pytest.mark.parametrize("dt", (torch.bfloat16, torch.float32), ids=("bf16", "f32"))
def test_smaller_workspaces(dt):
    """What a call needed before there were tiles of 64 and short slices is still taken."""
    T, c_in, c_out = 2000, 264, 64
    need = ef.lib().efqat_linear_bwd_workspace_bytes(T, c_in, c_out, 16, ef.BF16 if dt == torch.bfloat16 else ef.F32, 0)
    full = _linear(T, c_in, c_out, dt, ws=torch.empty(need, dtype=torch.uint8, device="cuda"))
    taken = 0
    for less in range(need - 256, 0, -256):
        try:
            got = _linear(T, c_in, c_out, dt, ws=torch.empty(less, dtype=torch.uint8, device="cuda"))
        except ef.EfqatError as e:
            assert e.code == -6
            break
        _same(full, got)
        taken += 1
    assert taken > 0


def test_unaligned_weight_codes_where_tiles_of_256_would_read_them():
    T, c_in, c_out = 8448, 1536, 496
    assert ef.lib().efqat_linear_bwd_weight_operand_bytes(T, c_in, c_out, ef.BF16, 0) == 0       # read as they lie
    _same(_linear(T, c_in, c_out, torch.bfloat16), _linear(T, c_in, c_out, torch.bfloat16, w_off=1))


@pytest.mark.parametrize("size", [(64, 64, 64), (63, 65, 8), (129, 128, 192), (640, 192, 136), (65, 1000, 4096), (1, 4096, 520)], ids=str)
@pytest.mark.parametrize("dt", (torch.bfloat16, torch.float32), ids=("bf16", "f32"))
def test_small_tiles_against_tiles_of_192(size, dt):
    _same(_linear(*size, dt), _linear(*size, dt, kernel=ef.DX_KERNEL_BF16_PINNED))
