"""Both products of a layer in one grid against the same blocks in two launches (what timing by class asks for), bit for bit:
operands read as they lie and staged, both K loops, linear layers and convolutions of both kinds, more blocks than places on
the chip, a second stream, replays of a captured call."""
import pytest
import torch

import paper_2411_11038_amd as ef

pytestmark = pytest.mark.gpu

KEYS = ("dx", "dw", "ds_w", "ds_x", "dz_x")
# T, c_in, c_out, k
LINEAR = [(64, 64, 64, 16), (65, 80, 72, 72), (1, 16, 8, 1), (300, 72, 520, 1), (129, 777, 65, 40), (96, 31, 4100, 30), (2048, 512, 512, 100),
          (4000, 320, 136, 130), (16000, 48, 40, 7), (72, 80, 33, 5), (8, 16, 8, 8), (1000, 144, 200, 200)]
# N, H, c_in, c_out, kernel, stride, k
CONV = [(2, 9, 128, 64, 3, 1, 10), (2, 9, 72, 64, 3, 1, 64), (3, 8, 128, 40, 3, 2, 20), (2, 9, 20, 128, 5, 2, 3), (1, 7, 256, 64, 1, 2, 64),
        (40, 14, 128, 128, 3, 1, 32), (33, 15, 64, 64, 3, 2, 16), (128, 9, 128, 64, 5, 1, 64), (6, 20, 128, 128, 5, 2, 32)]


def _plan(size, dt, layout):
    code = ef.BF16 if dt == torch.bfloat16 else ef.F32
    if len(size) == 4:
        return ef.linear_bwd_plan(*size, code, layout)
    N, H, c_in, c_out, kernel, stride, k = size
    return ef.conv_bwd_plan(N, H, H, c_in, c_out, kernel, kernel, stride, kernel // 2, k, code, layout)


def _linear(size, dt, layout):
    T, c_in, c_out, k = size
    g = torch.Generator(device="cuda")
    g.manual_seed(T)
    x = torch.randn(T, c_in, generator=g, device="cuda").to(dt)
    w = torch.randn(c_out, c_in, generator=g, device="cuda") * 0.05
    dy = torch.randn(T, c_out, generator=g, device="cuda").to(dt)
    fx, fw = ef.fakequant_fwd(x, ef.ACT_PER_TENSOR_ASYM, 8), ef.fakequant_fwd(w, ef.W_PER_ROW_SYM, 8)
    idx, _ = ef.channel_select(w, k)
    dy = dy.t().contiguous() if layout else dy
    return lambda **kw: ef.linear_bwd(dy, fx["codes"], fx["clip_bits"], x, fx["scale"], fx["zero_point"], fw["codes"],
                                      fw["clip_bits"], w, fw["scale"], idx, dy_layout=layout, **kw)


def _conv(size, dt, layout):
    N, H, c_in, c_out, kernel, stride, k = size
    g = torch.Generator(device="cuda")
    g.manual_seed(N)
    pad = kernel // 2
    Ho = (H + 2 * pad - kernel) // stride + 1
    x = torch.randn(N, H, H, c_in, generator=g, device="cuda").to(dt)
    w = torch.randn(c_out, kernel, kernel, c_in, generator=g, device="cuda") * 0.05
    dy = torch.randn(N * Ho * Ho, c_out, generator=g, device="cuda").to(dt)
    fx, fw = ef.fakequant_fwd(x.view(-1, c_in), ef.ACT_PER_TENSOR_ASYM, 8), ef.fakequant_fwd(w.view(c_out, -1), ef.W_PER_ROW_SYM, 8)
    idx, _ = ef.channel_select(w.view(c_out, -1), k)
    dy = dy.t().contiguous() if layout else dy
    return lambda **kw: ef.conv_bwd(dy, fx["codes"].view(N, H, H, c_in), fx["clip_bits"], x, fx["scale"], fx["zero_point"],
                                    fw["codes"].view(c_out, kernel, kernel, c_in), fw["clip_bits"], w, fw["scale"], idx,
                                    stride=stride, pad=pad, dy_layout=layout, **kw)


def test_every_form_of_the_shared_grid_is_reached():
    got = set()
    for size in LINEAR + CONV:
        for dt in (torch.bfloat16, torch.float32):
            for layout in (0, 1):
                p = _plan(size, dt, layout)
                got.add((p["dx_kernel"], p["dx_rows"], p["dw_operands"]) + ((dt,) if p["dx_kernel"] == 1 else ()))
    want = {(2, 0, 4)}                                    # channel major
    for rows, operands in ((0, 1), (0, 3), (1, 2), (1, 3), (2, 2), (2, 3)):
        want |= {(0, rows, operands), (1, rows, operands, torch.bfloat16), (1, rows, operands, torch.float32)}
    assert got == want


@pytest.mark.parametrize("dt", (torch.bfloat16, torch.float32), ids=("bf16", "f32"))
@pytest.mark.parametrize("layout", (0, 1))
@pytest.mark.parametrize("size", LINEAR + CONV, ids=str)
def test_one_grid_is_two_launches(size, layout, dt):
    assert _plan(size, dt, layout)["one_grid"] == 1
    call = (_linear if len(size) == 4 else _conv)(size, dt, layout)
    ef.profile_enable(True)
    try:
        want = call()
    finally:
        ef.profile_enable(False)
    got = call()
    side = call(side_stream=torch.cuda.Stream())
    torch.cuda.synchronize()
    for key in KEYS:
        assert torch.equal(got[key], want[key]), key
        assert torch.equal(side[key], want[key]), key


@pytest.mark.parametrize("size", [LINEAR[0], LINEAR[4], CONV[0], CONV[2]], ids=str)
def test_one_grid_captured(size):
    assert _plan(size, torch.bfloat16, 0)["one_grid"] == 1
    call = (_linear if len(size) == 4 else _conv)(size, torch.bfloat16, 0)
    want = call()
    out = {k: torch.zeros_like(v) for k, v in want.items()}
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            call(out=out, ws=ws)
        for _ in range(3):
            for v in out.values():
                v.zero_()
            graph.replay()
            stream.synchronize()
            for key in KEYS:
                assert torch.equal(out[key], want[key]), key
            call(out=out, ws=ws)                       # the program's own work between the replays
            stream.synchronize()
