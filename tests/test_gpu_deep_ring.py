"""dX of few 64 x 64 tiles: on a ring of eight stages from 32 K stages on (linear layers), every remainder of the ring's rounds, whole and
ragged last stages; shorter contractions on the ring of three or, below seven stages, without a ring.  Against the tiles of 192, which
add the same products in the same order: dX bit for bit, the sums of dS_x and dZ_x in another order.  Convolutions of few tiles, on the
ring of three, against double precision."""
import numpy as np
import pytest
import torch

import paper_2411_11038_amd as ef
from tests.gpu_util import clip_words

pytestmark = pytest.mark.gpu


def _in_range(fx, cols):
    """The range made from the data can clip its own ends: dX is 0 there."""
    words = clip_words(fx["clip_bits"])
    bits = np.unpackbits(words.reshape(-1, words.shape[-1]).view(np.uint8), axis=1, bitorder="little")[:, :cols]
    return torch.from_numpy(bits.astype(np.float64)).cuda()


@pytest.mark.parametrize("dt", (torch.bfloat16, torch.float32), ids=("bf16", "f32"))
@pytest.mark.parametrize("c_out", (8, 64, 72, 392, 448, 504, 512, 520, 960, 1016, 1032, 1088, 1536, 2040) +
                         tuple(range(2048, 2624, 64)) + tuple(range(4040, 4616, 64)))
def test_against_tiles_of_192(c_out, dt):
    T, c_in = (150, 200) if c_out < 4000 else (500, 520)   # ragged rows of dY take eight stages on 64 tiles and more only
    tile = ef.linear_bwd_dx_tile(T, c_in, c_out, 0, ef.BF16 if dt == torch.bfloat16 else ef.F32)
    assert tile["rows"] == 64 and (tile["stages"] == 8 if c_out >= 2041 else tile["stages"] in (2, 3))
    g = torch.Generator(device="cuda")
    g.manual_seed(c_out)
    x = torch.randn(T, c_in, generator=g, device="cuda").to(dt)
    w = torch.randn(c_out, c_in, generator=g, device="cuda") * 0.05
    dy = torch.randn(T, c_out, generator=g, device="cuda").to(dt)
    fx = ef.fakequant_fwd(x, ef.ACT_PER_TENSOR_ASYM, 8)
    fx["scale"] *= 0.3                                 # a fifth is clipped
    ef.fakequant_fwd(x, ef.ACT_PER_TENSOR_ASYM, 8, init_minmax=False, out=fx)
    fw = ef.fakequant_fwd(w, ef.W_PER_ROW_SYM, 8)
    args = (dy, fx["codes"], fx["clip_bits"], x, fx["scale"], fx["zero_point"], fw["codes"], fw["clip_bits"], w, fw["scale"], None)
    got = [ef.linear_bwd(*args, dx_kernel=k) for k in (ef.DX_KERNEL_AUTO, ef.DX_KERNEL_BF16_PINNED)]
    inr, full = _in_range(fx, c_in), dy.double() @ (fw["codes"].double() * fw["scale"].double()[:, None])
    ref = (full * inr).float()
    assert torch.equal(got[0]["dx"], got[1]["dx"])
    # W_q (and a fp32 dY) rounded to bf16, dX to its type: the bound of bwd_checks.py
    assert (got[0]["dx"].float() - ref).abs().max() <= 2e-2 * ref.abs().max()
    # fp32 sums in two orders: 1e-5 of the 2-norm of their terms (bwd_checks.py)
    q, s = fx["codes"].double() - fx["zero_point"].double().round(), fx["scale"].double()
    terms = dict(ds_x=full * (q - inr * x.double() / s), dz_x=s * full * (1 - inr))
    for n, t in terms.items():
        assert (got[0][n].double() - got[1][n].double()).abs() <= 1e-5 * t.norm()


@pytest.mark.parametrize("size", [(2, 9, 7, 64, 3), (1, 14, 14, 192, 3), (4, 5, 5, 128, 5), (8, 7, 7, 512, 3)], ids=str)
def test_convolutions(size):
    N, H, W, c_out, kernel = size
    c_in, pad = 96, kernel // 2
    g = torch.Generator(device="cuda")
    g.manual_seed(N)
    x = torch.randn(N, H, W, c_in, generator=g, device="cuda").abs().bfloat16()
    w = torch.randn(c_out, kernel, kernel, c_in, generator=g, device="cuda") * 0.05
    dy = torch.randn(N, H, W, c_out, generator=g, device="cuda").bfloat16()
    fx = ef.fakequant_fwd(x, ef.ACT_PER_TENSOR_ASYM, 8)
    fw = ef.fakequant_fwd(w.view(c_out, -1), ef.W_PER_ROW_SYM, 8)
    got = ef.conv_bwd(dy.view(-1, c_out), fx["codes"].view(N, H, W, c_in), fx["clip_bits"], x, fx["scale"], fx["zero_point"],
                      fw["codes"].view(w.shape), fw["clip_bits"], w, fw["scale"], None, pad=pad)["dx"]
    wq = (fw["codes"].double() * fw["scale"].double()[:, None]).view(w.shape).permute(0, 3, 1, 2).cpu()
    ref = torch.nn.functional.conv_transpose2d(dy.double().permute(0, 3, 1, 2).cpu(), wq, padding=pad).permute(0, 2, 3, 1).cuda()
    ref = ref * _in_range(fx, c_in).view(ref.shape)
    assert (got.double().view(ref.shape) - ref).abs().max() <= 2e-2 * ref.abs().max()
