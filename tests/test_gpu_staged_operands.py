"""The one launch that lays out every operand the products cannot read as it lies (k_prep), against the oracle: each
combination of its parts, at the edges of its 64 x 64 tiles and 4-wide loads."""
import pytest

from tests.bwd_checks import check_backward
from tests.test_gpu_parity import _conv_case, _run_linear
from workloads import synth

pytestmark = pytest.mark.gpu

# T, c_in, c_out, kind, (num, den), layout
LINEAR = [
    (1, 1, 1, "bf16", (1, 1), 0),
    (63, 65, 64, "f32", (1, 4), 0),        # copy of dY, W_q^T, codes and selected columns
    (64, 63, 129, "bf16", (1, 1), 0),      # every channel, still through the selection
    (65, 68, 128, "bf16", (1, 3), 0),      # dY in place, 4-wide loads of codes and weights
    (129, 64, 65, "f32", (1, 4), 1),       # channel major: rows of dY, dY transposed
    (66, 63, 64, "bf16", (1, 2), 1),       # rows of dY not 16-byte aligned
    (64, 66, 72, "bf16", (1, 4), 1),       # rows of dY in place for dW, transposed for dX
    (65, 63, 64, "f32", (0, 1), 1),        # nothing selected
    (1031, 40, 24, "f32", (1, 4), 1),      # few selected rows of several 512-column segments, the last one ragged
    (512, 16, 33, "f32", (1, 1), 1),       # rows of one whole segment
    (65, 24, 515, "bf16", (1, 4), 0),      # copy of dY: two segments a row
    (16500, 9, 9, "f32", (1, 3), 0),       # more rows than blocks
]


@pytest.mark.parametrize("case", LINEAR, ids=str)
def test_linear_bwd_staged_operands(case):
    T, c_in, c_out, kind, (num, den), layout = case
    X, W, dY = synth.linear_layer(8200 + T + c_in, T, c_in, c_out, act_dtype=kind)
    out, ref, idx, idx_ref, _, _, qp = _run_linear(X, W, dY, kind, 8, 8, 0.8, num, den, layout, False)
    check_backward(out, ref, idx, idx_ref, X, W, qp, kind, False, kind == "bf16", W.shape)


CONV = [
    # N, H, W, c_in, c_out, kh, kw, stride, pad, kind, w_bits, shrink, (num, den), layout, scatter
    (2, 7, 5, 65, 64, 3, 2, 1, 1, "bf16", 8, 0.8, (1, 4), 0, False),
    (2, 8, 8, 64, 31, 3, 3, 2, 1, "f32", 8, 0.8, (1, 2), 0, True),
    (2, 8, 7, 128, 33, 2, 3, 1, 1, "f32", 8, 0.8, (1, 3), 1, False),
]


@pytest.mark.parametrize("case", CONV, ids=str)
def test_conv_bwd_staged_operands(case):
    _conv_case(case)
