"""Second pass of the weight gradient over rows of any width and alignment (four columns a lane, the last lane of a ragged row starting
earlier): gradients, scale gradients and the fused optimizer step against double precision.  Few rows: widths around one and several
trips of each block size, one slice and two, and every number of slices that the batches of 8, 4, 3, 2 and 1 take apart in another way;
many rows: one and several trips of 256 threads, aligned and not.  Frozen rows keep their bits."""
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
    _check(200, c_in, 24, 7, off)


# T, c_in; slices
FEW_ROWS = [(384, 64, 3), (512, 64, 4), (640, 64, 5), (1000, 64, 8), (1500, 64, 12), (2100, 64, 11), (3000, 64, 16),
            (512, 1021, 3), (1000, 1021, 6), (1500, 1021, 8), (2100, 1500, 9), (384, 2048, 3), (2100, 2051, 7), (6000, 2051, 12)]


@pytest.mark.parametrize("off", (0, 1))
@pytest.mark.parametrize("case", FEW_ROWS, ids=str)
def test_slices_of_few_rows(case, off):
    T, c_in, slices = case
    assert ef.linear_bwd_plan(T, c_in, 24, 7)["dw_slices"] == slices
    _check(T, c_in, 24, 7, off)


MANY_ROWS = [(200, 777, 1), (2100, 777, 3), (6000, 1027, 11), (2100, 1028, 3), (6000, 2050, 6), (2100, 1536, 3), (6000, 1024, 6)]


@pytest.mark.parametrize("off", (0, 1))
@pytest.mark.parametrize("case", MANY_ROWS, ids=str)
def test_many_rows(case, off):
    T, c_in, slices = case
    assert ef.linear_bwd_plan(T, c_in, 600, 520)["dw_slices"] == slices
    _check(T, c_in, 600, 520, off)


def _check(T, c_in, c_out, k, off):
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
    # per row (bwd_checks.py): fp32 sums within 1e-5 of the 2-norm of their terms, those of the row and the products in each of them,
    # and 2^-18 of |dW_q| for the rounding of w / S_w
    inner = ((dy.double()[:, rows] ** 2).T @ (fx["codes"].double() - fx["zero_point"].double().round()) ** 2).sqrt() * fx["scale"].double()
    weight = torch.where(bits, code - w.double()[rows] / s, code)
    bound = 1e-5 * (terms.norm(dim=1) + (inner * weight).norm(dim=1)) + 2.0 ** -18 * dwq.abs().sum(dim=1)
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
    # formed in fp32: 2e-6 of the value, 2^-22 of what was added; the weights carry the momentum's error times the learning rate, which
    # counts where the momentum is small because its terms cancel
    err_m = 2e-6 * m.abs() + 2.0 ** -22 * (m0.double()[rows].abs() + grad.abs())
    assert ((mom.double()[rows] - m).abs() <= err_m).all()
    err_w = 2e-6 * new.abs() + 2.0 ** -22 * (w0.double()[rows].abs() + m.abs()) + 0.1 * err_m
    assert ((w1.double()[rows] - new).abs() <= err_w).all()
    assert torch.equal(w1[frozen], w0[frozen]) and torch.equal(mom[frozen], m0[frozen])
