"""Second pass of the weight gradient over rows of any width and alignment (four columns a lane, the last lane of a ragged row starting
earlier): gradients, scale gradients and the fused optimizer step against double precision, widths around the trips of every
block size; frozen rows keep their bits."""
import numpy as np
import pytest
import torch

import paper_2411_11038_amd as ef
from tests.gpu_util import clip_words

pytestmark = pytest.mark.gpu


def _off(t, off):
    buf = torch.empty(t.numel() + 4, dtype=t.dtype, device="cuda")
    v = buf[off:off + t.numel()].view(t.shape)
    v.copy_(t)
    return v


@pytest.mark.parametrize("off", (0, 1))
@pytest.mark.parametrize("c_in", (1, 2, 3, 4, 5, 7, 64, 1021, 1024, 1027, 1500, 2045, 2048, 2051, 4101))
def test_rows(c_in, off):
    T, c_out, k = 200, 24, 7
    g = torch.Generator(device="cuda")
    g.manual_seed(c_in)
    x = torch.randn(T, c_in, generator=g, device="cuda").bfloat16()
    w = _off(torch.randn(c_out, c_in, generator=g, device="cuda") * 0.05, off)
    dy = (torch.randn(T, c_out, generator=g, device="cuda") / T).bfloat16()
    fx = ef.fakequant_fwd(x, ef.ACT_PER_TENSOR_ASYM, 8)
    fw = ef.fakequant_fwd(w, ef.W_PER_ROW_SYM, 4)
    fw["scale"] *= 0.8                                 # some are clipped
    ef.fakequant_fwd(w, ef.W_PER_ROW_SYM, 4, init_minmax=False, out=fw)
    idx, _ = ef.channel_select(w, k)
    args = (dy, fx["codes"], fx["clip_bits"], x, fx["scale"], fx["zero_point"], fw["codes"], fw["clip_bits"])
    got = ef.linear_bwd(*args, w, fw["scale"], idx)
    # dY and code - Z are exact in bf16: what differs is the order of fp32 sums (the bound of bwd_checks.py)
    rows = idx.long()
    dwq = (dy.double()[:, rows].T @ (fx["codes"].double() - fx["zero_point"].double().round())) * fx["scale"].double()
    bits = torch.from_numpy(np.unpackbits(clip_words(fw["clip_bits"]).reshape(c_out, -1).view(np.uint8), axis=1, bitorder="little")
                            [:, :c_in].astype(bool)).cuda()[rows]
    want = torch.where(bits, dwq, torch.zeros_like(dwq))
    assert (got["dw"].double() - want).abs().max() <= 2e-4 * dwq.abs().max()
    code, s = fw["codes"].double()[rows], fw["scale"].double()[rows, None]
    terms = dwq * torch.where(bits, code - w.double()[rows] / s, code)
    # per row: 1e-5 of the 2-norm of its terms for the sums, 2^-18 of |dW_q| for the rounding of w / S_w (bwd_checks.py)
    bound = 1e-5 * terms.norm(dim=1) + 2.0 ** -18 * dwq.abs().sum(dim=1) + 2e-4 * dwq.abs().max() * c_in ** 0.5
    assert ((got["ds_w"].double() - terms.sum(dim=1)).abs() <= bound).all()

    w1, mom = _off(w, off), _off(torch.randn(c_out, c_in, generator=g, device="cuda"), off)
    w0, m0 = w1.clone(), mom.clone()
    step = dict(lr_w=0.1, momentum=0.9, weight_decay=0.01, mom_w=mom, lr_s=1e-3, adam_m=torch.zeros(c_out, device="cuda"),
                adam_v=torch.zeros(c_out, device="cuda"), adam_t=torch.zeros(c_out, dtype=torch.int32, device="cuda"))
    ef.linear_bwd(*args, w1, fw["scale"].clone(), idx, step=step)
    grad = got["dw"].double()
    m = 0.9 * m0.double()[rows] + grad + 0.01 * w0.double()[rows]
    new = w0.double()[rows] - 0.1 * m
    frozen = torch.ones(c_out, dtype=torch.bool, device="cuda")
    frozen[rows] = False
    # formed in fp32: 2e-6 of the value, 2^-22 of what was added
    assert ((mom.double()[rows] - m).abs() <= 2e-6 * m.abs() + 2.0 ** -22 * (m0.double()[rows].abs() + grad.abs())).all()
    assert ((w1.double()[rows] - new).abs() <= 2e-6 * new.abs() + 2.0 ** -22 * (w0.double()[rows].abs() + m.abs())).all()
    assert torch.equal(w1[frozen], w0[frozen]) and torch.equal(mom[frozen], m0[frozen])
