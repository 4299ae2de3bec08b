"""Codes and masks of rows that start at any element: whole chunks of 8 are one vector access whatever their alignment, the chunk
that ends a row is not; views one to three elements into their storage, inputs and outputs alike, bit for bit against the oracle."""
import numpy as np
import pytest
import torch

import paper_2411_11038_amd as ef
from oracle import efqat_oracle as orc
from tests.gpu_util import clip_words, pack_mask

pytestmark = pytest.mark.gpu


def _view(t, off):
    """t's values `off` elements into a larger buffer, whose other elements are returned too."""
    buf = torch.full((t.numel() + off + 8,), 77, dtype=t.dtype, device="cuda")
    buf[off:off + t.numel()] = t.flatten()
    return buf, buf[off:off + t.numel()].view(t.shape)


@pytest.mark.parametrize("off", (0, 1, 3))
@pytest.mark.parametrize("size", [(1, 8), (3, 7), (5, 9), (4, 15), (9, 64), (2, 513), (33, 777), (3, 1031)], ids=str)
@pytest.mark.parametrize("kind", ("bf16", "f32"))
def test_activation_codes(size, kind, off):
    rows, cols = size
    dt = torch.bfloat16 if kind == "bf16" else torch.float32
    X = torch.from_numpy(np.random.default_rng(cols).standard_normal(size).astype(np.float32)).to(dt)
    _, x = _view(X.cuda(), off)
    cbuf, codes = _view(torch.zeros(size, dtype=torch.uint8, device="cuda"), off)
    qbuf, xq = _view(torch.zeros(size, dtype=torch.bfloat16, device="cuda"), off)
    got = ef.fakequant_fwd(x, ef.ACT_PER_TENSOR_ASYM, 8, out=dict(codes=codes, xq=xq))
    V = X.float().numpy()
    s, z = orc.act_qparams_minmax(V, 8)
    want, mask, wq = orc.fakequant_act(V, s, z, 8)
    assert got["scale"].item() == float(s) and got["zero_point"].item() == float(z)
    assert np.array_equal(codes.cpu().numpy().astype(np.int64), want.astype(np.int64))
    assert np.array_equal(clip_words(got["clip_bits"]).reshape(rows, -1), pack_mask(mask))
    assert np.abs(xq.float().cpu().numpy() - wq).max() <= 2.0 ** -8 * np.abs(wq).max()
    for buf in (cbuf, qbuf):                           # nothing beside the rows was written
        assert (buf[:off] == 77).all() and (buf[off + rows * cols:] == 77).all()


@pytest.mark.parametrize("size", [(3, 16385), (2, 16391), (2, 16400)], ids=str)
def test_weight_rows_beyond_the_registers(size):
    W = (np.random.default_rng(size[1]).standard_normal(size) * 0.02).astype(np.float32)
    W[:, -1] = np.float32(0.5)                         # the largest in the chunk that ends a row
    _, w = _view(torch.from_numpy(W).cuda(), 1)
    got = ef.fakequant_fwd(w, ef.W_PER_ROW_SYM, 8)
    sw = orc.weight_scale_minmax(W, 8)
    want, mask, _ = orc.fakequant_weight(W, sw, 8)
    assert np.array_equal(got["scale"].cpu().numpy(), sw)
    assert np.array_equal(got["codes"].cpu().numpy().astype(np.int64), want.astype(np.int64))
    assert np.array_equal(clip_words(got["clip_bits"]).reshape(size[0], -1), pack_mask(mask))
