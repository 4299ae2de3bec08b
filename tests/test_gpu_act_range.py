"""Range, scale, zero point and codes of an activation tensor, every block of the second kernel making the range from the
partial ones for itself, or a launch between the two: tensors of less than a block up to more chunks than the grid takes at once, both kernels, bit for
bit against the oracle; the range's ends in the first, the last and an inner element."""
import numpy as np
import pytest
import torch

import paper_2411_11038_amd as ef
from oracle import efqat_oracle as orc
from tests.gpu_util import act_tensor, clip_words, pack_mask

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ("bf16", "f32"))
@pytest.mark.parametrize("size", [(1, 1), (1, 7), (1, 32), (5, 96), (128, 32), (129, 32), (257, 160), (255, 33), (1000, 1000),
                                  (4096, 1024), (4097, 1024), (6145, 1024), (8194, 1056),
                                  # ragged rows on both sides of the 10240 segments, short (a launch for the range) and not, and
                                  # more segments than the blocks take at once
                                  (10240, 9), (10244, 9), (5122, 513), (10244, 300), (16388, 300), (5463, 1337)], ids=str)
def test_act_range(size, kind):
    rows, cols = size
    rng = np.random.default_rng(rows + cols)
    x = rng.standard_normal(rows * cols).astype(np.float32)
    for place in ((0, -1), (-1, 0), (rows * cols // 2, rows * cols // 3)):
        x[place[0]] = 6.5
        x[place[1]] = -5.25
        X = torch.from_numpy(x.reshape(rows, cols)).to(torch.bfloat16 if kind == "bf16" else torch.float32).float().numpy()
        got = ef.fakequant_fwd(act_tensor(X, kind), ef.ACT_PER_TENSOR_ASYM, 8)
        sx, zx = orc.act_qparams_minmax(X, 8)
        assert got["scale"].item() == float(sx) and got["zero_point"].item() == float(zx)
        codes, mask, _ = orc.fakequant_act(X, sx, zx, 8)
        assert np.array_equal(got["codes"].cpu().numpy().astype(np.int64), codes.astype(np.int64))
        assert np.array_equal(clip_words(got["clip_bits"]).reshape(rows, -1), pack_mask(mask))
        x[place[0]] = x[place[1]] = 0.0
