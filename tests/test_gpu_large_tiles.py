"""Layers large enough for products on tiles of 128 rows and more, and for the ring on 64, with whole tiles, ragged rows and
ragged (also odd) columns: linear layers, convolutions gathered at stride 1 and by stride phase, against the same products in
double precision.  The plan of every size is asserted, so that other cost tables cannot send it elsewhere unseen.  Bounds:
tests/bwd_checks.py."""
import pytest
import torch

import paper_2411_11038_amd as ef
from bwd_checks import EXACT_TOL, GEMM_RMS, GEMM_TOL, QP_SUM_TOL

pytestmark = pytest.mark.gpu

# N, H, W, c_in, c_out, kernel, stride, k, type of x and dY; kernel (0 two LDS stages, 1 ring) and tile of dX; tile of dW
CONV = [
    (44, 28, 24, 256, 64, 2, 1, 3, "bf16", (0, 128), 64),        # whole tiles: the straight-line epilogue
    (60, 22, 23, 199, 64, 2, 1, 3, "bf16", (0, 128), 64),
    (56, 39, 30, 96, 64, 2, 1, 3, "f32", (0, 128), 64),
    (42, 32, 36, 192, 64, 2, 1, 3, "bf16", (0, 192), 64),        # whole tiles
    (38, 36, 33, 154, 64, 3, 1, 3, "bf16", (0, 192), 64),
    (24, 33, 31, 373, 64, 2, 1, 16, "f32", (0, 192), 64),
    (14, 16, 36, 512, 64, 5, 1, 3, "bf16", (1, 128), 64),        # whole tiles
    (30, 23, 45, 83, 256, 3, 1, 64, "bf16", (1, 128), 64),
    (56, 14, 41, 72, 256, 3, 1, 12, "f32", (1, 128), 64),
    (24, 40, 34, 256, 128, 3, 2, 32, "bf16", (0, 128), 64),
    (61, 24, 44, 98, 64, 5, 3, 16, "bf16", (0, 128), 64),
    (51, 8, 40, 475, 64, 3, 2, 3, "f32", (0, 128), 64),
    (32, 12, 25, 384, 512, 5, 2, 128, "bf16", (1, 128), 128),
    (63, 26, 17, 93, 512, 5, 2, 128, "bf16", (1, 128), 128),
    (56, 13, 40, 80, 512, 5, 2, 128, "f32", (1, 128), 128),
]
# T, c_in, c_out, k, type of x and dY, layout; kernel (2: int8 weight codes) and tile of dX; operands (1 token major, 3 staged,
# 4 rows of a channel-major dY) and tile of dW
LINEAR = [
    (4096, 1929, 72, 72, "f32", 0, (0, 128), (3, 64)),
    (2280, 3399, 72, 72, "bf16", 1, (0, 128), (3, 64)),
    (4096, 2048, 27, 1, "bf16", 0, (0, 128), (1, 64)),           # whole tiles
    (3536, 3536, 405, 405, "f32", 1, (0, 256), (3, 128)),
    (4096, 2147, 711, 711, "bf16", 0, (0, 256), (3, 128)),
    (2048, 4608, 1485, 371, "bf16", 0, (0, 256), (1, 128)),      # whole tiles
    (3072, 1152, 577, 577, "f32", 1, (1, 128), (3, 128)),        # whole tiles
    (6174, 519, 608, 608, "bf16", 0, (1, 128), (3, 128)),
    (2048, 2048, 386, 386, "bf16", 0, (1, 128), (1, 128)),       # whole tiles
    (3072, 2997, 196, 196, "f32", 0, (1, 192), (3, 128)),
    (7619, 1122, 203, 203, "bf16", 0, (1, 192), (3, 128)),
    (346, 1091, 2272, 568, "f32", 0, (1, 64), (3, 64)),
    (304, 2191, 1590, 397, "bf16", 1, (1, 64), (3, 64)),
    (1536, 4768, 21, 21, "bf16", 1, (2, 128), (4, 64)),
    (8912, 1328, 623, 623, "bf16", 1, (2, 256), (4, 128)),
    (4096, 3136, 264, 264, "bf16", 0, (2, 256), (1, 64)),
    (414, 4096, 2080, 2080, "bf16", 0, (1, 64), (1, 256)),
    (359, 4260, 1960, 1960, "bf16", 0, (1, 64), (3, 192)),
    (481, 4857, 1779, 1779, "bf16", 0, (1, 128), (3, 256)),
    (424, 4432, 2288, 2288, "f32", 1, (1, 64), (3, 256)),
    (472, 4224, 1952, 1952, "bf16", 1, (2, 128), (4, 256)),
]


def _check(x, w, dy, k, stride, pad, layout):
    """One backward call on NHWC x and OHWI w (a linear layer: 1 x 1 pixels) with clipped elements; dy NHWC."""
    N, H, W, c_in = x.shape
    c_out, ks = w.shape[:2]
    Ho, Wo = dy.shape[1:3]
    kind = "bf16" if x.dtype == torch.bfloat16 else "f32"
    x2, w2 = x.view(-1, c_in), w.view(c_out, -1)
    fx, fw = ef.fakequant_fwd(x2, ef.ACT_PER_TENSOR_ASYM, 8), ef.fakequant_fwd(w2, ef.W_PER_ROW_SYM, 8)
    fx = ef.fakequant_fwd(x2, ef.ACT_PER_TENSOR_ASYM, 8, init_minmax=False, scale=fx["scale"] * 0.7, zero_point=fx["zero_point"])
    fw = ef.fakequant_fwd(w2, ef.W_PER_ROW_SYM, 8, init_minmax=False, scale=fw["scale"] * 0.7)
    idx, _ = ef.channel_select(w2, k)
    if H * W > 1:
        out = ef.conv_bwd(dy, fx["codes"].view(x.shape), fx["clip_bits"], x, fx["scale"], fx["zero_point"], fw["codes"].view(w.shape),
                          fw["clip_bits"], w, fw["scale"], idx, stride=stride, pad=pad)
    else:
        dy2 = dy.view(N, c_out)
        out = ef.linear_bwd(dy2.t().contiguous() if layout else dy2, fx["codes"], fx["clip_bits"], x2, fx["scale"], fx["zero_point"],
                            fw["codes"], fw["clip_bits"], w2, fw["scale"], idx, dy_layout=layout)

    mask = lambda bits, cols: ((bits[:, :, None] >> torch.arange(32, device="cuda", dtype=torch.int32)) & 1).view(bits.shape[0], -1)[:, :cols] == 1
    sx, code = fx["scale"].double(), fx["codes"].double().view(x.shape) - fx["zero_point"].double().round()
    wq = (fw["codes"].double() * fw["scale"].double()[:, None]).view(w.shape)
    dyd, xq = dy.double().view(-1, c_out), torch.zeros(N, H + 2 * pad, W + 2 * pad, c_in, dtype=torch.float64, device="cuda")
    xq[:, pad:pad + H, pad:pad + W] = sx * code
    dxq, dw = torch.zeros_like(xq), torch.empty(k, ks, ks, c_in, dtype=torch.float64, device="cuda")
    sel = dyd[:, idx.long()].t().contiguous()
    for i in range(ks):
        for j in range(ks):
            at = (slice(None), slice(i, i + stride * (Ho - 1) + 1, stride), slice(j, j + stride * (Wo - 1) + 1, stride))
            dxq[at] += (dyd @ wq[:, i, j].contiguous()).view(N, Ho, Wo, c_in)
            dw[:, i, j] = sel @ xq[at].reshape(-1, c_in)
    dxq = dxq[:, pad:pad + H, pad:pad + W]
    xm, wm = mask(fx["clip_bits"], c_in).view(x.shape), mask(fw["clip_bits"], w2.shape[1]).view(w.shape)[idx.long()]
    assert 0 < int((~xm).sum()) < xm.numel() // 10

    def close(got, ref, tol, rms=None):
        err = got.double().view(ref.shape) - ref
        assert err.abs().max() <= tol * ref.abs().max()
        assert rms is None or err.norm() <= rms * ref.norm()

    assert not out["dx"].view(x.shape)[~xm].any() and not out["dw"].view(wm.shape)[~wm].any()
    close(out["dx"], dxq * xm, GEMM_TOL, GEMM_RMS + (4e-3 if kind == "bf16" else 0.0))
    close(out["dw"], dw * wm, EXACT_TOL if kind == "bf16" else GEMM_TOL)
    gs = torch.where(xm, code - x.double() / sx, code)
    assert (out["ds_x"].double() - (dxq * gs).sum()).abs() <= QP_SUM_TOL * (dxq * gs).norm()
    clipped, rms2 = dxq[~xm], (dxq ** 2).mean()
    assert (out["dz_x"].double() + sx * clipped.sum()).abs() <= QP_SUM_TOL * sx * torch.maximum(clipped ** 2, rms2).sum().sqrt()


def _normal(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return lambda *shape: torch.randn(*shape, generator=g, device="cuda")


@pytest.mark.parametrize("case", CONV, ids=lambda c: "%dx%dx%d_%d-%d_k%ds%d_%s_%d" % (*c[:7], c[8], c[9][1]))
def test_conv_tiles(case):
    N, H, W, c_in, c_out, ks, stride, k, kind, dx_plan, dw_tile = case
    pad, dt, normal = ks // 2, torch.bfloat16 if kind == "bf16" else torch.float32, _normal(N)
    p = ef.conv_bwd_plan(N, H, W, c_in, c_out, ks, ks, stride, pad, k, ef.BF16 if kind == "bf16" else ef.F32)
    assert (p["dx_kernel"], p["dx_tile"]) == dx_plan and p["dx_rows"] == (1 if stride == 1 else 2) and not p["one_grid"], p
    assert p["dw_tile"] == dw_tile, p
    Ho, Wo = (H + 2 * pad - ks) // stride + 1, (W + 2 * pad - ks) // stride + 1
    _check(normal(N, H, W, c_in).to(dt), normal(c_out, ks, ks, c_in) * 0.05, normal(N, Ho, Wo, c_out).to(dt), k, stride, pad, 0)


@pytest.mark.parametrize("case", LINEAR, ids=lambda c: "%dx%d-%d_%s_L%d_%d_%d" % (*c[:3], c[4], c[5], c[6][1], c[7][1]))
def test_linear_tiles(case):
    T, c_in, c_out, k, kind, layout, dx_plan, dw_plan = case
    dt, normal = torch.bfloat16 if kind == "bf16" else torch.float32, _normal(T)
    p = ef.linear_bwd_plan(T, c_in, c_out, k, ef.BF16 if kind == "bf16" else ef.F32, layout)
    assert (p["dx_kernel"], p["dx_tile"]) == dx_plan and (p["dw_operands"], p["dw_tile"]) == dw_plan and not p["one_grid"], p
    _check(normal(T, 1, 1, c_in).to(dt), normal(c_out, 1, 1, c_in) * 0.05, normal(T, 1, 1, c_out).to(dt), k, 1, 0, layout)
