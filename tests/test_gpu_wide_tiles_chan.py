"""dX of a channel-major dY on 128 x 256 tiles: one and several rounds of blocks, the last one whole and partly filled, whole and ragged K
stages, fp32 x and bf16, few and many clipped elements, against the tiles of 192 on a token-major copy, which add the same products in
the same order: dX bit for bit, dS_x and dZ_x in another order of the sums."""
import numpy as np
import pytest
import torch

import paper_2411_11038_amd as ef
from tests.gpu_util import clip_words

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("size", [(8192, 1024, 1024), (8192, 1024, 1000), (4096, 2048, 520), (4096, 2048, 4096), (16384, 1024, 300),
                                  (12288, 3072, 72), (12288, 768, 8), (12160, 1024, 200)], ids=str)
@pytest.mark.parametrize("x_dt", (torch.bfloat16, torch.float32), ids=("bf16", "f32"))
@pytest.mark.parametrize("tighter", (0.6, 0.3))        # one in some hundred elements is clipped: most chunks leave the mask out; a ninth
def test_against_tiles_of_192(size, x_dt, tighter):
    T, c_in, c_out = size
    tile = ef.linear_bwd_dx_tile(T, c_in, c_out, 0, ef.BF16, ef.DY_CHANNEL_MAJOR)
    assert (tile["rows"], tile["columns"]) == (128, 256)
    g = torch.Generator(device="cuda")
    g.manual_seed(c_out)
    x = torch.randn(T, c_in, generator=g, device="cuda").to(x_dt)
    w = torch.randn(c_out, c_in, generator=g, device="cuda") * 0.05
    dy = torch.randn(c_out, T, generator=g, device="cuda").bfloat16()
    fx = ef.fakequant_fwd(x, ef.ACT_PER_TENSOR_ASYM, 8)
    fx["scale"] *= tighter
    ef.fakequant_fwd(x, ef.ACT_PER_TENSOR_ASYM, 8, init_minmax=False, out=fx)
    fw = ef.fakequant_fwd(w, ef.W_PER_ROW_SYM, 8)
    args = (dy, fx["codes"], fx["clip_bits"], x, fx["scale"], fx["zero_point"], fw["codes"], fw["clip_bits"], w, fw["scale"], None)
    got = ef.linear_bwd(*args, dy_layout=ef.DY_CHANNEL_MAJOR)
    want = ef.linear_bwd(*args, dy_layout=ef.DY_CHANNEL_MAJOR, dx_kernel=ef.DX_KERNEL_BF16_PINNED)
    assert torch.equal(got["dx"], want["dx"])
    # fp32 sums of the same terms in two orders: 1e-5 of the 2-norm of the terms (bwd_checks.py)
    bits = np.unpackbits(clip_words(fx["clip_bits"]).reshape(T, -1).view(np.uint8), axis=1, bitorder="little")[:, :c_in]
    inr = torch.from_numpy(bits).cuda().bool()
    full = dy.float().t().contiguous() @ (fw["codes"].float() * fw["scale"][:, None])
    q = fx["codes"].float() - fx["zero_point"].round()
    terms = dict(ds_x=full * torch.where(inr, q - x.float() / fx["scale"], q), dz_x=fx["scale"] * full * ~inr)
    for n, t in terms.items():
        norm = t.double().norm()
        assert norm > 0 and (got[n].double() - want[n].double()).abs() <= 1e-5 * norm
