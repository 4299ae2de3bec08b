"""The fused epilogue of the dX product at the edges of its tiles: rows and columns that end inside a tile, a wavefront or an
8-column chunk, widths that are no multiple of anything, matrices of fewer than 8 elements, x / codes / dX at element
alignment, fp32 and bf16 x and dX in every combination, on each dX kernel."""
import pytest
import torch

import paper_2411_11038_amd as ef

pytestmark = pytest.mark.gpu

# T, c_in, c_out, dX kernel
CASES = [(1, 1, 3, 0), (3, 2, 5, 0), (1, 7, 9, 0), (1, 8, 8, 0), (2, 5, 64, 0), (33, 9, 70, 0), (64, 64, 64, 0), (65, 65, 40, 0),
         (127, 129, 72, 0), (128, 128, 128, 0), (129, 136, 200, 0), (257, 31, 64, 0), (300, 777, 131, 0), (191, 193, 64, 3),
         (385, 200, 72, 3), (260, 528, 64, 2), (1030, 784, 136, 2), (2100, 2056, 64, 1), (4100, 1544, 72, 0)]


def _call(T, c_in, c_out, xt, dxt, kernel, off, layout):
    g = torch.Generator(device="cuda")
    g.manual_seed(T + c_in)

    def place(t):                                     # the same values, `off` elements behind a 256-byte boundary
        b = torch.empty(t.numel() + 16, dtype=t.dtype, device="cuda")
        v = b[off:off + t.numel()].view(t.shape)
        v.copy_(t)
        return v

    x = place(torch.randn(T, c_in, generator=g, device="cuda").to(xt))
    w = torch.randn(c_out, c_in, generator=g, device="cuda") * 0.05
    dy = torch.randn(T, c_out, generator=g, device="cuda").to(torch.bfloat16)
    fx = ef.fakequant_fwd(x, ef.ACT_PER_TENSOR_ASYM, 8)
    fx = ef.fakequant_fwd(x, ef.ACT_PER_TENSOR_ASYM, 8, init_minmax=False, scale=fx["scale"] * 0.6, zero_point=fx["zero_point"])
    fw = ef.fakequant_fwd(w, ef.W_PER_ROW_SYM, 8)
    codes = place(fx["codes"])
    buf = torch.full((T * c_in + 32,), 77.0, dtype=dxt, device="cuda")
    dx = buf[8 + off:8 + off + T * c_in].view(T, c_in)
    out = dict(dx=dx, dw=None, ds_w=None, ds_x=torch.empty(1, device="cuda"), dz_x=torch.empty(1, device="cuda"))
    ef.linear_bwd(dy.t().contiguous() if layout else dy, codes, fx["clip_bits"], x, fx["scale"], fx["zero_point"], fw["codes"],
                  fw["clip_bits"], w, fw["scale"], None, dy_layout=layout, dx_kernel=kernel, out=out)
    assert (buf[:8 + off] == 77).all() and (buf[8 + off + T * c_in:] == 77).all()      # nothing beside dX is written
    return dx, out["ds_x"], out["dz_x"], dy, x, fx, fw


@pytest.mark.parametrize("case", CASES, ids=str)
@pytest.mark.parametrize("xt", (torch.bfloat16, torch.float32), ids=("xbf16", "xf32"))
def test_dx_edges(case, xt):
    T, c_in, c_out, kernel = case
    for dxt in (torch.bfloat16, torch.float32):
        for layout in ((0, 1) if kernel == 0 else (0,)):
            dx, dsx, dzx, dy, x, fx, fw = _call(T, c_in, c_out, xt, dxt, kernel, 0, layout)
            words = fx["clip_bits"].view(T, -1)
            inr = ((words[:, :, None] >> torch.arange(32, device="cuda", dtype=torch.int32)) & 1).bool().view(T, -1)[:, :c_in]
            s, z = fx["scale"].double(), fx["zero_point"].double().round()
            dxq = dy.double() @ (fw["codes"].double() * fw["scale"].double()[:, None])
            ref = torch.where(inr, dxq, torch.zeros_like(dxq))
            assert not dx[~inr].any()
            # one bf16 rounding of each weight (2^-9 of a term, terms of independent sign), one of a bf16 result
            scale = (dy.double().abs() @ (fw["codes"].double().abs() * fw["scale"].double()[:, None])).max()
            assert (dx.double() - ref).abs().max() <= 2.0 ** -8 * scale
            q = fx["codes"].double() - z
            gs = torch.where(inr, q - x.double() / s, q)
            # the same rounding carried into the sums: the bound of bwd_checks.py, at least one term's worth
            assert (dsx.double() - (dxq * gs).sum()).abs() <= 1e-2 * (dxq * gs).norm() + 2.0 ** -8 * scale * gs.abs().max()
            want = -s * dxq[~inr].sum()
            assert (dzx.double() - want).abs() <= 2e-2 * s * (dxq[~inr].norm() + scale / 8)
            if layout == 0:
                got = _call(T, c_in, c_out, xt, dxt, kernel, 1, layout)[:3]
                assert torch.equal(got[0], dx) and torch.equal(got[1], dsx) and torch.equal(got[2], dzx)
