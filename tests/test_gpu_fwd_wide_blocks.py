"""Int8 forward product of few tokens where a block takes one to four groups of 16 weight rows: columns that end inside a group or leave
whole groups of the last block empty, rows of K that end inside a step, against exact integer arithmetic."""
import pytest
import torch

import paper_2411_11038_amd as ef

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("c_out", (4100, 6001, 8191, 8193, 11009, 12305, 16385, 28673))
@pytest.mark.parametrize("T", (1, 5, 16, 17, 32, 33, 64))
@pytest.mark.parametrize("long", (False, True), ids=("short", "long"))   # short rows take wide blocks for many columns only
def test_against_integer_arithmetic(T, c_out, long):
    c_in = (2083 if T % 2 else 1552) if long else 83 if T % 2 else 528
    g = torch.Generator(device="cuda")
    g.manual_seed(T * c_out)
    x = torch.randint(0, 256, (T, c_in), generator=g, device="cuda", dtype=torch.uint8)
    w = torch.randint(-127, 128, (c_out, c_in), generator=g, device="cuda", dtype=torch.int8)
    sx = torch.tensor([0.013], device="cuda")
    sw = torch.rand(c_out, generator=g, device="cuda") * 0.01 + 0.001
    y = torch.full((T * c_out + 64,), 7.0, device="cuda")
    got = ef.linear_fwd(x, sx, torch.tensor([117.0], device="cuda"), w, sw, out=y[:T * c_out].view(T, c_out))
    ref = ((x.double() - 117) @ w.double().t()).float() * (sx * sw)[None, :]   # exact integers, two fp32 roundings in this order
    assert torch.equal(got, ref)
    assert (y[T * c_out:] == 7.0).all()
