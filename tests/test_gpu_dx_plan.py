"""The choice of the dX kernel: calls whose workspace or weight codes do not fit the first plan take the wide one, and the tiles
of 64 against the others at sizes around them."""
import pytest
import torch

import paper_2411_11038_amd as ef

pytestmark = pytest.mark.gpu


def _linear(T, c_in, c_out, dt, w_off=0, ws=None, kernel=0, operand=None):
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
                         fw["scale"], idx, ws=ws, dx_kernel=kernel, w_operand=operand)


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


# A layer whose tiles of 256 read the weight codes has no operand made beforehand: a buffer handed over is ignored, also where the
# call falls back to tiles that multiply by W_q^T.  The buffer is as large as W_q^T would be and holds no number.
@pytest.mark.parametrize("less", (False, True), ids=("unaligned codes", "smallest workspace"))
def test_operand_of_a_layer_that_has_none(less):
    T, c_in, c_out, k = 8448, 1536, 496, 124
    L = ef.lib()
    assert L.efqat_linear_bwd_weight_operand_bytes(T, c_in, c_out, ef.BF16, 0) == 0
    need = L.efqat_linear_bwd_workspace_bytes(T, c_in, c_out, k, ef.BF16, 0)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    if less:
        lo, hi = 0, need // 256                        # the smallest workspace that is taken, in units of 256 bytes
        while hi - lo > 1:
            mid = (lo + hi) // 2
            try:
                _linear(T, c_in, c_out, torch.bfloat16, ws=ws[:mid * 256])
                hi = mid
            except ef.EfqatError as e:
                assert e.code == -6
                lo = mid
        assert hi * 256 < need
        ws = ws[:hi * 256]
    off = 0 if less else 1
    want = _linear(T, c_in, c_out, torch.bfloat16, w_off=off, ws=ws)
    bad = torch.full(((c_in * c_out * 2 + 256) // 2,), float("nan"), dtype=torch.bfloat16, device="cuda").view(torch.uint8)
    got = _linear(T, c_in, c_out, torch.bfloat16, w_off=off, ws=ws, operand=bad)
    for n in ("dx", "dw", "ds_w", "ds_x", "dz_x"):
        assert torch.equal(got[n], want[n]), n


@pytest.mark.parametrize("size", [(64, 64, 64), (63, 65, 8), (129, 128, 192), (640, 192, 136), (65, 1000, 4096), (1, 4096, 520)], ids=str)
@pytest.mark.parametrize("dt", (torch.bfloat16, torch.float32), ids=("bf16", "f32"))
def test_small_tiles_against_tiles_of_192(size, dt):
    _same(_linear(*size, dt), _linear(*size, dt, kernel=ef.DX_KERNEL_BF16_PINNED))
