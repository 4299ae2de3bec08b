"""dS_x and dZ_x where products, sums or inputs are infinite or undefined, on every form of the dX epilogue: dZ_x = -S sum of the products of
clipped activations, undefined where a product of any activation is, and untouched by an overflow of the sum of dS_x alone."""
import pytest
import torch

import paper_2411_11038_amd as ef

pytestmark = pytest.mark.gpu

TOK, CHAN = ef.DY_TOKEN_MAJOR, ef.DY_CHANNEL_MAJOR
# T, c_in, c_out, type of x, layout of dY, dX kernel asked for; kernel and tile that it takes
SIZES = [
    (3264, 3072, 576, "bf16", TOK, ef.DX_KERNEL_BF16_PINNED, (1, 192)),  # whole tiles, more than one a CU: inputs requested in the
    (3264, 3072, 648, "bf16", TOK, ef.DX_KERNEL_BF16_PINNED, (1, 192)),  # first stages, nine of them and a ragged eleventh
    (384, 384, 640, "bf16", TOK, ef.DX_KERNEL_BF16_PINNED, (1, 192)),    # ... in the last ones
    (384, 384, 72, "bf16", TOK, ef.DX_KERNEL_BF16_PINNED, (1, 192)),
    (400, 200, 72, "bf16", TOK, ef.DX_KERNEL_BF16_PINNED, (1, 192)),
    (384, 384, 72, "f32", TOK, ef.DX_KERNEL_BF16_PINNED, (1, 192)),
    (1024, 512, 64, "bf16", TOK, ef.DX_KERNEL_INT8, (2, 256)),
    (256, 256, 64, "bf16", TOK, ef.DX_KERNEL_INT8, (2, 128)),
    (200, 208, 64, "f32", TOK, ef.DX_KERNEL_INT8, (2, 128)),
    (150, 200, 512, "bf16", TOK, ef.DX_KERNEL_AUTO, (1, 64)),
    (256, 256, 64, "f32", TOK, ef.DX_KERNEL_AUTO, (0, 64)),
    (4096, 2048, 27, "bf16", TOK, ef.DX_KERNEL_AUTO, (0, 128)),
    (2048, 2048, 386, "bf16", TOK, ef.DX_KERNEL_AUTO, (1, 128)),
    (256, 256, 256, "bf16", CHAN, ef.DX_KERNEL_AUTO, (2, 64)),
    (8192, 1024, 1000, "bf16", CHAN, ef.DX_KERNEL_AUTO, (2, 128)),
    (8192, 1024, 1000, "f32", CHAN, ef.DX_KERNEL_AUTO, (2, 128)),
    (8912, 1328, 623, "bf16", CHAN, ef.DX_KERNEL_AUTO, (2, 256)),
    (2528, 784, 1000, "bf16", CHAN, ef.DX_KERNEL_AUTO, (2, 128)),        # up to 256 tiles: the mask in every chunk
    (1528, 1328, 1000, "f32", CHAN, ef.DX_KERNEL_AUTO, (2, 128)),
]
S, Z = 0.02, 128.0


@pytest.mark.parametrize("what", ("clipped", "in_range", "overflow", "nan_in_x"))
@pytest.mark.parametrize("size", SIZES, ids=lambda s: "-".join(map(str, s[:6])))
def test_sums(size, what):
    T, c_in, c_out, kind, layout, dxk, plan = size
    p = ef.linear_bwd_plan(T, c_in, c_out, 0, ef.BF16, layout, dxk)
    assert (p["dx_kernel"], p["dx_tile"]) == plan
    g = torch.Generator(device="cuda")
    g.manual_seed(T + c_in + c_out)
    x = (torch.randn(T, c_in, generator=g, device="cuda") * 0.5).clamp(-2, 2).to(torch.bfloat16 if kind == "bf16" else torch.float32)
    w = torch.randn(c_out, c_in, generator=g, device="cuda") * 0.05
    w[0] = w[0].abs() + 0.01                           # every code of the first channel is positive
    w[0, 2] = 0.1
    dy = torch.randn(T, c_out, generator=g, device="cuda").bfloat16()
    rows = [37, T - 1]                                 # the last one lies in an edge tile where there are any
    dy[rows] = 0
    x[5, 3] = 10.0                                     # clipped, an ordinary product
    x[T - 2, c_in - 1] = -10.0
    if what in ("clipped", "in_range"):
        dy[rows, 0] = float("inf")                     # products of these rows: inf
        if what == "clipped":
            x[rows] = 10.0
    elif what == "overflow":                           # products of 2e36 to 5e37, that of column 2 times code - Z = 127 more than fp32 holds
        dy[rows, 0] = 2e38
        x[rows, 2] = 10.0
    fx = dict(ef.fakequant_fwd(x, ef.ACT_PER_TENSOR_ASYM, 8))
    fx["scale"].fill_(S)
    fx["zero_point"].fill_(Z)
    ef.fakequant_fwd(x, ef.ACT_PER_TENSOR_ASYM, 8, init_minmax=False, out=fx)
    fw = ef.fakequant_fwd(w, ef.W_PER_ROW_SYM, 8)
    clipped = (x.double() / S).round() + Z
    clipped = (clipped < 0) | (clipped > 255)
    if what == "nan_in_x":                             # in range by its mask bit
        x[7, c_in - 2] = float("nan")
    out = ef.linear_bwd((dy if layout == TOK else dy.T.contiguous()), fx["codes"], fx["clip_bits"], x, fx["scale"], fx["zero_point"],
                        fw["codes"], fw["clip_bits"], w, fw["scale"], None, dy_layout=layout, dx_kernel=dxk)
    dx, ds, dz = out["dx"].float(), out["ds_x"].item(), out["dz_x"].item()
    assert (dx[clipped] == 0).all()
    wq = (fw["codes"].float() * fw["scale"][:, None]).bfloat16().double()
    where = clipped.any(dim=1).nonzero().flatten()
    terms = (dy[where].double() @ wq)[clipped[where]]
    if what == "clipped":
        assert ds == float("inf") and dz == float("-inf")
    elif what == "in_range":
        assert not (abs(ds) < float("inf")) and dz != dz and (dx[rows] == float("inf")).all()
    else:
        assert ds == float("inf") if what == "overflow" else ds != ds
        # fp32 sums of products of bf16 values: 2^-24 an addition, c_out of them in a product and a handful behind it
        assert abs(dz + S * terms.sum().item()) <= 2.0 ** -24 * (c_out + 64) * S * (
            (dy[where].double().abs() @ wq.abs())[clipped[where]].sum().item())
