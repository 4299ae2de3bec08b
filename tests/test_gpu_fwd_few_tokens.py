"""Int8 forward product at the token counts where its kernel changes (16, 32, 64 and beyond) and at row lengths that end
inside a 16-byte fragment, a 64-byte step or a wavefront's slice of K, against exact integer arithmetic."""
import numpy as np
import pytest
import torch

import paper_2411_11038_amd as ef
from tests.gpu_util import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("c_in,c_out", [(1, 1), (15, 17), (64, 16), (65, 100), (511, 33), (512, 64), (1003, 515), (4096, 48),
                                        (96, 8192), (100, 8209)])
@pytest.mark.parametrize("T", [1, 16, 17, 32, 33, 64, 65])
def test_forward_matches_integer_arithmetic(T, c_in, c_out):
    r = np.random.default_rng(1000 * T + c_in)
    x = r.integers(0, 256, (T, c_in)).astype(np.uint8)
    w = r.integers(-127, 128, (c_out, c_in)).astype(np.int8)
    sx, z = np.float32(0.013), np.float32(117.0)
    sw = (r.random(c_out) * 0.01 + 0.001).astype(np.float32)
    got = ef.linear_fwd(dev(x), dev(np.array([sx])), dev(np.array([z])), dev(w), dev(sw), y_dtype=torch.float32)
    torch.cuda.synchronize()
    sums = (x.astype(np.int64) - 117) @ w.astype(np.int64).T
    ref = sums.astype(np.float32) * (sx * sw)[None, :]            # two fp32 roundings, in this order
    # the sums are exact integers: only the roundings of the scale product and of the result are left (2^-24 each)
    assert np.abs(got.cpu().numpy() - ref).max() <= 2.0 ** -22 * np.abs(ref).max()


# more tokens, with sizes that take each of the four tiles and end inside a tile, a 16-byte store and a K stage; the zero
# point of 1e6 needs sums of more than 32 bits
@pytest.mark.parametrize("z", [117.0, 1.0e6])
@pytest.mark.parametrize("T,c_in,c_out", [(65, 100, 70), (200, 48, 129), (2000, 1003, 1900), (1100, 4112, 4088), (3000, 1536, 6000),
                                          (8000, 4096, 4100), (16385, 64, 520)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_forward_tiles_match_integer_arithmetic(T, c_in, c_out, z, dtype):
    g = torch.Generator(device="cuda")
    g.manual_seed(T)
    x = torch.randint(0, 256, (T, c_in), generator=g, device="cuda", dtype=torch.uint8)
    w = torch.randint(-127, 128, (c_out, c_in), generator=g, device="cuda", dtype=torch.int8)
    sx = torch.tensor([0.013], device="cuda")
    sw = torch.rand(c_out, generator=g, device="cuda") * 0.01 + 0.001
    got = ef.linear_fwd(x, sx, torch.tensor([z], device="cuda"), w, sw, y_dtype=dtype)
    sums = (x.double() - z) @ w.double().t()                      # integers below 2^53: exact in any order
    ref = sums.float() * (sx * sw)[None, :]                       # the same two roundings
    assert torch.equal(got, ref.to(dtype))


def test_more_columns_than_one_grid_dimension_holds():
    c_out = (1 << 27) + 5                                         # 16 columns and 512 threads a block: beyond 2^32 threads
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    x = torch.tensor([[201]], dtype=torch.uint8, device="cuda")
    w = torch.randint(-127, 128, (c_out, 1), generator=g, device="cuda", dtype=torch.int8)
    sx, sw = torch.tensor([0.013], device="cuda"), torch.rand(c_out, generator=g, device="cuda")
    got = ef.linear_fwd(x, sx, torch.tensor([117.0], device="cuda"), w, sw, y_dtype=torch.float32)
    assert torch.equal(got[0], (84.0 * w[:, 0].float()) * (sx * sw))
