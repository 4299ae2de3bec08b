"""The weight quantizer with the row in registers, over row lengths around its chunks of 8, mask words and wavefronts, rows off
the vector alignment, few and many rows, scales from the data and given: codes, masks, scales bit for bit against the oracle,
importances in double precision."""
import numpy as np
import pytest
import torch

import paper_2411_11038_amd as ef
from oracle import efqat_oracle as orc
from tests.gpu_util import clip_words, pack_mask

pytestmark = pytest.mark.gpu

SIZES = [(1, 1), (3, 7), (5, 8), (4, 9), (7, 31), (6, 32), (9, 33), (130, 511), (5, 513), (64, 777), (3, 2047), (2, 2049), (4099, 65),
         (4097, 512), (4097, 515), (33, 4096), (5, 4099), (3, 8200), (2, 16383), (2, 16384), (2, 16390)]


@pytest.mark.parametrize("size", SIZES, ids=str)
@pytest.mark.parametrize("off", (0, 1), ids=("aligned", "unaligned"))
def test_weight_rows(size, off):
    rows, cols = size
    rng = np.random.default_rng(rows * 7 + cols)
    W = (rng.standard_normal((rows, cols)) * 0.02).astype(np.float32)
    if rows > 2:
        W[1] = 0.0                                     # an all-zero row: scale 1
    wd = torch.empty(rows * cols + 4, device="cuda")[off:off + rows * cols].view(rows, cols)
    wd.copy_(torch.from_numpy(W))
    k = max(1, rows // 3)
    for bits in (4, 8):
        got = ef.weight_quant_select(wd, bits, k)
        sw = orc.weight_scale_minmax(W, bits)
        assert np.array_equal(got["scale"].cpu().numpy(), sw)
        imp = orc.channel_importance(W)
        assert np.abs(got["scores"].cpu().numpy() - imp).max() <= 1e-12 * imp.max()
        for shrink in (1.0, 0.7):
            if shrink != 1.0:                          # given scales: some values are clipped
                sw = (sw * np.float32(shrink)).astype(np.float32)
                got = ef.weight_quant_select(wd, bits, k, init_minmax=False, out=dict(got, scale=torch.from_numpy(sw).cuda()))
                assert np.abs(got["scores"].cpu().numpy() - imp).max() <= 1e-12 * imp.max()
            codes, mask, _ = orc.fakequant_weight(W, sw, bits)
            assert np.array_equal(got["codes"].cpu().numpy().astype(np.int64), codes.astype(np.int64))
            assert np.array_equal(clip_words(got["clip_bits"]).reshape(rows, -1), pack_mask(mask))
            assert got["idx"].cpu().numpy().tolist() == orc.top_k_channels(got["scores"].cpu().numpy(), k).tolist()
