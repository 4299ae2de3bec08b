"""The optional second stream of efqat_linear_bwd_ex / efqat_conv_bwd_ex: the weight-gradient branch runs beside the
dX product and is joined before the pass that finishes dW; results are bit-identical to the one-stream call, call
after call, and the fork / join can be captured in a HIP graph.  Small layers run both products in one launch and leave the
second stream unused; the layers of `USED` use it (asked of the plan)."""
import pytest
import torch

import paper_2411_11038_amd as ef
from workloads import synth

from gpu_util import act_tensor, dev

pytestmark = pytest.mark.gpu

KEYS = ("dx", "dw", "ds_w", "ds_x", "dz_x")


def _linear_setup(seed, T, c_in, c_out, frac, layout):
    X, W, dY = synth.linear_layer(seed, T, c_in, c_out, act_dtype="bf16")
    xd, wd = act_tensor(X, "bf16"), dev(W)
    dyd = act_tensor(dY if layout == 0 else dY.T.copy(), "bf16")
    fx = ef.fakequant_fwd(xd, ef.ACT_PER_TENSOR_ASYM, 8, init_minmax=True)
    fw = ef.fakequant_fwd(wd, ef.W_PER_ROW_SYM, 4, init_minmax=True)
    k = ef.k_from_ratio(c_out, *frac)
    idx, _ = ef.channel_select(wd, k)

    def call(side, ws=None, out=None):
        return ef.linear_bwd(dyd, fx["codes"], fx["clip_bits"], xd, fx["scale"], fx["zero_point"], fw["codes"],
                             fw["clip_bits"], wd, fw["scale"], idx if k else None, dy_layout=layout, side_stream=side,
                             ws=ws, out=out)
    return call, k


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("shape,frac", [((1024, 768, 768), (1, 20)), ((300, 208, 136), (1, 4)), ((2048, 512, 1024), (1, 1)),
                                        ((520, 208, 264), (0, 1)), ((130, 70, 43), (1, 3))])
def test_linear_bwd_with_a_second_stream_is_bit_identical(shape, frac, layout):
    call, k = _linear_setup(91 + layout, *shape, frac, layout)
    ref = call(None)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    for rep in range(3):                                 # back to back: the library's events are used again at once
        got = call(side)
    torch.cuda.synchronize()
    for key in KEYS:
        if k or key in ("dx", "ds_x", "dz_x"):
            assert torch.equal(ref[key], got[key]), key


def test_conv_bwd_with_a_second_stream_is_bit_identical():
    N, H, W, c_in, c_out = 4, 10, 9, 128, 64
    X, Wt, dY = synth.conv_layer(17, N, H, W, c_in, c_out, 3, 3, 1, 1, act_dtype="bf16")
    xd, wd, dyd = act_tensor(X, "bf16"), dev(Wt), act_tensor(dY, "bf16")
    fx = ef.fakequant_fwd(xd, ef.ACT_PER_TENSOR_ASYM, 8, init_minmax=True)
    fw = ef.fakequant_fwd(wd, ef.W_PER_ROW_SYM, 4, init_minmax=True)
    idx, _ = ef.channel_select(wd, 16)
    call = lambda side: ef.conv_bwd(dyd, fx["codes"], fx["clip_bits"], xd, fx["scale"], fx["zero_point"], fw["codes"],
                                    fw["clip_bits"], wd, fw["scale"], idx, stride=1, pad=1, side_stream=side)
    ref = call(None)
    side = torch.cuda.Stream()
    got = call(side)
    got = call(side)
    torch.cuda.synchronize()
    for key in KEYS:
        assert torch.equal(ref[key], got[key]), key


def test_second_stream_fork_and_join_replay_from_a_graph():
    T, c_in, c_out = 1024, 256, 512
    call, k = _linear_setup(5, T, c_in, c_out, (1, 4), 0)
    e = lambda shape, dt: torch.empty(shape, dtype=dt, device="cuda")
    out = dict(dx=e((T, c_in), torch.bfloat16), dw=e((k, c_in), torch.float32), ds_w=e(k, torch.float32),
               ds_x=e(1, torch.float32), dz_x=e(1, torch.float32))
    ws = e(ef.lib().efqat_linear_bwd_workspace_bytes(T, c_in, c_out, k, ef.BF16, 0), torch.uint8)
    ref = {key: t.clone() for key, t in call(None).items()}
    side = torch.cuda.Stream()
    cap = torch.cuda.Stream()
    cap.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(cap):
        call(side, ws, out)                              # first use outside the capture: the events are made here
    torch.cuda.current_stream().wait_stream(cap)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call(side, ws, out)
    for rep in range(3):
        for t in out.values():
            t.zero_()
        ws.random_(0, 255)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for key in KEYS:
            assert torch.equal(ref[key], out[key]), (rep, key)


# layers that use the second stream: T, c_in, c_out, k or N, H, c_in, c_out, kernel, stride, k; layout, type of x and dY
USED = [((4096, 2048, 136, 34), 0, torch.bfloat16),      # selected columns compacted on the second stream
        ((4096, 2048, 768, 192), 0, torch.float32),
        ((4096, 2048, 136, 136), 0, torch.bfloat16),     # every channel: dY as it lies
        ((4104, 3072, 1032, 129), 1, torch.bfloat16),    # rows of a channel-major dY
        ((8192, 2048, 1024, 256), 0, torch.bfloat16),    # dX from the int8 weight codes
        ((32, 28, 256, 64, 3, 1, 16), 0, torch.bfloat16),
        ((32, 28, 256, 128, 5, 2, 128), 0, torch.float32)]


def _used(size, layout, dt):
    """call(side, ws, out), dY, workspace of a layer of USED"""
    g = torch.Generator(device="cuda")
    g.manual_seed(21)
    normal = lambda *shape: torch.randn(*shape, generator=g, device="cuda")
    code = ef.BF16 if dt == torch.bfloat16 else ef.F32
    conv = len(size) > 4
    if conv:
        N, H, c_in, c_out, ks, stride, k = size
        geometry = dict(stride=stride, pad=ks // 2)
        T_out = N * ((H + 2 * (ks // 2) - ks) // stride + 1) ** 2
        x, w = normal(N, H, H, c_in).abs().to(dt), normal(c_out, ks, ks, c_in) * 0.05
        sizes = (N, H, H, c_in, c_out, ks, ks, stride, ks // 2, k, code, layout)
        plan, need = ef.conv_bwd_plan(*sizes), ef.lib().efqat_conv_bwd_workspace_bytes(*sizes)
    else:
        T_out, c_in, c_out, k = size
        geometry = {}
        x, w = normal(T_out, c_in).to(dt), normal(c_out, c_in) * 0.05
        plan, need = ef.linear_bwd_plan(*size, code, layout), ef.lib().efqat_linear_bwd_workspace_bytes(*size, code, layout)
    assert plan["side_stream"] == 1 and plan["one_grid"] == 0, plan
    dy = normal(*((c_out, T_out) if layout else (T_out, c_out))).to(dt)
    fx = ef.fakequant_fwd(x.view(-1, c_in), ef.ACT_PER_TENSOR_ASYM, 8)
    fw = ef.fakequant_fwd(w.view(c_out, -1), ef.W_PER_ROW_SYM, 8)
    idx, _ = ef.channel_select(w.view(c_out, -1), k)
    bwd = ef.conv_bwd if conv else ef.linear_bwd
    call = lambda side, ws=None, out=None: bwd(dy, fx["codes"].view(x.shape), fx["clip_bits"], x, fx["scale"], fx["zero_point"],
                                               fw["codes"].view(w.shape), fw["clip_bits"], w, fw["scale"], idx, dy_layout=layout,
                                               side_stream=side, ws=ws, out=out, **geometry)
    return call, dy, torch.empty(need, dtype=torch.uint8, device="cuda")


# The caller's stream is late with dY and with a workspace of NaN: a fork that did not wait for it would take a dY of zeros.  The
# second stream is late: a join that was not waited for would take NaN for the product.
@pytest.mark.parametrize("late", ("caller", "side"))
@pytest.mark.parametrize("size,layout,dt", USED, ids=str)
def test_second_stream_waits_and_is_waited_for(size, layout, dt, late):
    call, dy, ws = _used(size, layout, dt)
    want = {key: t.clone() for key, t in call(None, ws).items()}
    dy0, out, side = dy.clone(), {key: torch.empty_like(t) for key, t in want.items()}, torch.cuda.Stream()
    for rep in range(2):
        dy.zero_()
        torch.cuda.synchronize()
        with torch.cuda.stream(side if late == "side" else torch.cuda.current_stream()):
            torch.cuda._sleep(2000000)                   # about a millisecond
        dy.copy_(dy0)
        ws.fill_(255)
        for t in out.values():
            t.fill_(float("nan"))
        call(side, ws, out)
        got = {key: t.clone() for key, t in out.items()}
        ws.fill_(255)                                    # the caller's next work on the workspace
        torch.cuda.synchronize()
        for key in KEYS:
            assert torch.equal(got[key], want[key]), (rep, key)


@pytest.mark.parametrize("size,layout,dt", [USED[0], USED[3], USED[5]], ids=str)
def test_used_second_stream_replays_from_a_graph(size, layout, dt):
    call, dy, ws = _used(size, layout, dt)
    want = {key: t.clone() for key, t in call(None, ws).items()}
    out, side, cap = {key: torch.empty_like(t) for key, t in want.items()}, torch.cuda.Stream(), torch.cuda.Stream()
    cap.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(cap):
        call(side, ws, out)                              # the events are made outside the capture
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call(side, ws, out)
    for rep in range(3):
        for t in out.values():
            t.fill_(float("nan"))
        ws.fill_(255)
        g.replay()
        got = {key: t.clone() for key, t in out.items()}
        torch.cuda.synchronize()
        for key in KEYS:
            assert torch.equal(got[key], want[key]), (rep, key)
        call(None, ws, out)                              # the program's own work between the replays
        torch.cuda.synchronize()
