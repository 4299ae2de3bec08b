"""Convolutions whose dX product gathers dY by stride phase (strides 2 to 4) or from a copy padded to whole 64-channel
stages, against the oracle: phases with different tap counts and without taps, images smaller than the stride, ragged last
tiles of a phase, one and several column tiles, both dY layouts.  These sizes run on 64 x 64 tiles beside dW; the larger tiles:
test_gpu_large_tiles.py."""
import numpy as np
import pytest
import torch

import paper_2411_11038_amd as ef
from tests.test_gpu_parity import _conv_case

pytestmark = pytest.mark.gpu

CASES = [
    # N, H, W, c_in, c_out, kh, kw, stride, pad, kind, w_bits, shrink, (num, den), layout, scatter
    (2, 8, 8, 32, 64, 1, 1, 2, 0, "bf16", 8, 0.8, (1, 4), 0, False),      # three phases of four have no tap: dX = 0
    (2, 9, 7, 32, 64, 3, 3, 2, 1, "bf16", 4, 0.8, (1, 4), 0, False),      # 4 / 2 / 2 / 1 taps, odd image
    (3, 9, 8, 128, 64, 3, 3, 2, 1, "f32", 8, 0.8, (1, 2), 0, True),
    (2, 9, 8, 20, 128, 2, 3, 2, 2, "bf16", 8, 0.8, (1, 3), 1, False),     # two K stages per tap, ragged c_in, padding 2
    (1, 2, 1, 16, 64, 2, 1, 3, 0, "bf16", 8, 1.0, (1, 1), 0, False),      # image smaller than the stride
    (2, 11, 10, 48, 64, 5, 4, 3, 2, "bf16", 8, 0.8, (1, 4), 0, False),
    (2, 13, 9, 24, 64, 3, 5, 4, 1, "f32", 8, 0.8, (1, 4), 1, False),      # 16 phases, some without taps
    (2, 12, 12, 16, 64, 3, 3, 5, 1, "bf16", 8, 0.8, (1, 4), 0, False),    # beyond the rule: im2col matrix
    (40, 29, 31, 136, 64, 3, 3, 2, 1, "bf16", 8, 0.8, (1, 4), 0, False),  # 563 row tiles x 3, the dW product beside them
    # stride 1 and 2 on padded channel counts
    (2, 9, 7, 32, 40, 3, 3, 1, 1, "bf16", 4, 0.8, (1, 4), 0, False),
    (2, 9, 7, 32, 97, 3, 3, 1, 1, "bf16", 8, 0.8, (1, 4), 0, False),      # rows of dY not 16-byte aligned
    (2, 9, 7, 128, 72, 3, 3, 2, 1, "bf16", 8, 0.8, (1, 1), 0, False),     # every channel: compaction from the dY itself
    (2, 9, 8, 32, 33, 3, 3, 2, 1, "f32", 8, 0.8, (1, 4), 1, False),
    (1, 5, 6, 8, 31, 3, 3, 1, 1, "bf16", 8, 0.8, (1, 4), 0, False),       # 31 channels: not worth padding to 64
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "N%d_%dx%d_%d-%d_k%dx%d_s%dp%d_%s_L%d" % (
    c[0], c[1], c[2], c[3], c[4], c[5], c[6], c[7], c[8], c[9], c[13]))
def test_conv_bwd_gathered_dx(case):
    _conv_case(case)


def _draw(seed):
    rng = np.random.default_rng(7100 + seed)
    kh, kw, stride, pad = (int(rng.integers(*r)) for r in ((1, 6), (1, 6), (1, 5), (0, 4)))
    H, W = (int(rng.integers(6, 15)) for _ in range(2))         # never an image that no tap reaches
    c_in = int(rng.choice([rng.integers(1, 140), 16, 64, 128]))
    c_out = int(rng.choice([rng.integers(20, 200), 64, 128, 192]))
    return (int(rng.integers(1, 4)), H, W, c_in, c_out, kh, kw, stride, pad, ["bf16", "f32"][int(rng.integers(0, 2))],
            [8, 4][int(rng.integers(0, 2))], [1.0, 0.7][int(rng.integers(0, 2))],
            [(0, 1), (1, 7), (1, 3), (1, 1)][int(rng.integers(0, 4))], int(rng.integers(0, 2)), bool(rng.integers(0, 2)))


@pytest.mark.parametrize("seed", range(20))
def test_conv_bwd_gathered_dx_drawn(seed):
    _conv_case(_draw(seed))


# K stages beyond what the tile loads take apart exactly: 2^14 channel stages times 4 x 5 taps go through the im2col matrix.
# fp32 dX against a product in 64 bits of the same quantised operands; each operand is rounded to bf16 once (2^-8), the
# terms are independent, so the error of a sum stays within a few times that of its 2-norm.
def test_a_million_channels():
    c_out, c_in, KH, KW, H, W, pad = 1 << 20, 8, 4, 5, 4, 5, 1
    g = torch.Generator(device="cuda")
    g.manual_seed(9)
    Ho, Wo = H + 2 * pad - KH + 1, W + 2 * pad - KW + 1
    dy = torch.randn((1, Ho, Wo, c_out), generator=g, device="cuda")
    w = torch.randint(-127, 128, (c_out, KH, KW, c_in), generator=g, device="cuda", dtype=torch.int8)
    sw = torch.rand(c_out, generator=g, device="cuda") + 0.5
    x = torch.zeros((1, H, W, c_in), device="cuda")
    fx = ef.fakequant_fwd(x.view(H * W, c_in), ef.ACT_PER_TENSOR_ASYM, 8, init_minmax=False,
                          scale=torch.ones(1, device="cuda"), zero_point=torch.full((1,), 128.0, device="cuda"))
    out = ef.conv_bwd(dy, fx["codes"].view(1, H, W, c_in), fx["clip_bits"], x, fx["scale"], fx["zero_point"], w, None,
                      torch.empty(1, device="cuda"), sw, None, stride=1, pad=pad)
    ref = torch.zeros((H + 2 * pad, W + 2 * pad, c_in), dtype=torch.float64, device="cuda")
    rows = dy.double().view(Ho * Wo, c_out)
    for kh in range(KH):
        for kw in range(KW):
            part = rows @ (w[:, kh, kw].double() * sw.double()[:, None])
            ref[kh:kh + Ho, kw:kw + Wo] += part.view(Ho, Wo, c_in)
    ref = ref[pad:pad + H, pad:pad + W]
    assert (out["dx"][0].double() - ref).norm() <= 2.0 ** -7 * ref.norm()
