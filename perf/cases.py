"""Timed cases of the EfQAT layer path: what one layer costs a training or evaluation loop, over the range of layers
that the workloads of this repository are made of (workloads/synth.py, bench.py) and generic neighbours of them.

A case is a dict of plain values:
  kind      "layer"     one training step of a layer: quantize X, quantize W and select channels, backward;
                        `forward`, `bias`, `optimizer` add the int8 forward product, the bias gradient and the fused
                        optimizer step
            "backward"  the restricted backward call alone, on codes the program already holds
            "forward"   evaluation: quantize X with the trained scale, int8 product
            "select"    the network-wide selections over the channels (CWPN) and the layers (LWPN) of an encoder stack
  T, c_in, c_out                   tokens and channels of a linear layer, or
  N, H, W, c_in, c_out, kernel, stride, pad   images and geometry of a convolution (N > 0)
  dtype     of X, dY, dX ("bf16" / "f32");  w_bits, a_bits;  num / den: update fraction
  layout    of dY: 0 token major, 1 channel major
  init      quantizer parameters from the data (min/max) in every step; else given ones that clip some elements
  side      hand a second stream to the backward call
"""
import math
from types import SimpleNamespace

import torch

import paper_2411_11038_amd as ef

_DEFAULTS = dict(kind="layer", T=0, N=0, H=0, W=0, c_in=0, c_out=0, kernel=1, stride=1, pad=0, dtype="bf16", w_bits=4,
                 a_bits=8, num=1, den=4, layout=0, init=True, forward=False, bias=False, optimizer=False, side=False)


def _case(name=None, **kw):
    c = dict(_DEFAULTS, **kw)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest layer anybody trains: launches and host calls are what it costs
        _case("small_linear_f32_step", T=256, c_in=256, c_out=256, dtype="f32", w_bits=8),
        # feed-forward layer of a BERT-base encoder (32 sequences of 384 tokens), everything a training step does with it
        _case("bert_ffn1_train", T=12288, c_in=768, c_out=3072, forward=True, bias=True, optimizer=True),
        # its partner, the paper's metric (the backward call alone) at a small update fraction
        _case("bert_ffn2_backward_r5", kind="backward", T=12288, c_in=3072, c_out=768, den=20, init=False),
        # attention output projection, a short contraction, gradient handed over channel major, trained 8-bit scales
        _case("bert_out_step_chan", T=12288, c_in=768, c_out=768, w_bits=8, layout=1, init=False),
        # 3x3 convolution of a ResNet-50 stage at 64 images
        _case("resnet_conv3x3_step", N=64, H=14, W=14, c_in=256, c_out=256, kernel=3, pad=1),
        # the strided convolution between two stages, single precision
        _case("resnet_conv3x3s2_backward_f32", kind="backward", N=32, H=28, W=28, c_in=128, c_out=256, kernel=3, stride=2,
              pad=1, dtype="f32", w_bits=8),
        # LLM-sized MLP, up projection: the largest step, on two streams
        _case("llm_up_step", T=8192, c_in=4096, c_out=11008, side=True),
        # LLM-sized MLP, down projection: backward from a channel-major gradient at a small fraction
        _case("llm_down_backward_chan", kind="backward", T=8192, c_in=11008, c_out=4096, layout=1, den=10),
        # a head with an odd number of classes on features of an odd width: nothing is a multiple of a vector
        _case("ragged_head_f32_step", T=2049, c_in=777, c_out=1001, dtype="f32", w_bits=8, bias=True),
        # evaluation: a long prompt through the LLM-sized up projection
        _case("llm_up_forward_prefill", kind="forward", T=2048, c_in=4096, c_out=11008, init=False),
        # evaluation: a few sequences decoding, one token each
        _case("llm_up_forward_decode", kind="forward", T=16, c_in=4096, c_out=11008, init=False),
        # choosing the unfrozen channels and layers of a BERT-base-sized stack (12 blocks, 82944 channels)
        _case("bert_stack_select", kind="select", N=12, c_in=768),
    ]


_MOST_FLOPS = 2.0 * 8192 * 4096 * 11008 * 1.25   # the largest listed case
_MOST_VALUES = 8192 * 11008                      # and its largest tensor


def draw(rng):
    def size(lo, hi):
        v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
        step = rng.choice((1, 8, 16, 64, 128))        # ragged, vector-wide and tile-friendly sizes
        return min(hi, max(lo, max(1, round(v / step)) * step))

    while True:
        kind = rng.choice(("layer", "layer", "layer", "backward", "backward", "forward", "forward", "select"))
        if kind == "select":
            return _case(kind=kind, N=size(2, 48), c_in=size(64, 2048), num=1, den=rng.choice((4, 10, 20)))
        num, den = rng.choice(((0, 1), (1, 20), (1, 10), (1, 4), (1, 4), (1, 2), (1, 1)))
        kw = dict(kind=kind, dtype=rng.choice(("bf16", "bf16", "f32")), w_bits=rng.choice((4, 8)), num=num, den=den,
                  layout=rng.choice((0, 0, 1)), init=rng.random() < 0.6)
        if kind == "forward":
            kw.update(T=size(1, 16384), c_in=size(64, 11008), c_out=size(64, 11008), num=1, den=4, layout=0, init=False)
        elif rng.random() < 0.35:
            kernel = rng.choice((1, 3, 3, 5))
            hw = rng.randint(7, 56)
            kw.update(N=size(1, 128), H=hw, W=hw, c_in=size(16, 1024), c_out=size(16, 2048), kernel=kernel,
                      stride=rng.choice((1, 1, 2)), pad=kernel // 2)
        else:
            kw.update(T=size(64, 16384), c_in=size(64, 11008), c_out=size(64, 11008))
        if kind == "layer":
            kw.update(bias=rng.random() < 0.5, optimizer=rng.random() < 0.4, side=rng.random() < 0.3,
                      forward=not kw.get("N") and rng.random() < 0.4)
        c = _case(**kw)
        t_in, t_out, taps = _sizes(c)
        # the staged matrix of a convolution has one copy of the gradient per tap
        if work(c)["flops"] <= _MOST_FLOPS and max(t_in * c["c_in"], max(t_in, t_out) * taps * c["c_out"]) <= _MOST_VALUES:
            return c


# ------------------------------------------------------------------------------------------------------------------
def _sizes(c):
    """Rows of X and of dY as matrices, and the taps of the kernel."""
    if not c["N"]:
        return c["T"], c["T"], 1
    out = lambda n: (n + 2 * c["pad"] - c["kernel"]) // c["stride"] + 1  # noqa: E731
    return c["N"] * c["H"] * c["W"], c["N"] * out(c["H"]) * out(c["W"]), c["kernel"] ** 2


def _k(c):
    return c["c_out"] * c["num"] // c["den"]


def work(c):
    if c["kind"] == "select":                        # two readings of the fp64 scores, the chosen indices
        total = 9 * c["c_in"] * c["N"]
        return dict(bytes=2 * 8.0 * total + 4.0 * (total * c["num"] // c["den"]), flops=0.0)
    t_in, t_out, taps = _sizes(c)
    e = 2 if c["dtype"] == "bf16" else 4
    k, nw = _k(c), taps * c["c_in"]
    x, y, w, q = t_in * c["c_in"], t_out * c["c_out"], nw * c["c_out"], 1 + 1 / 8
    if c["kind"] == "forward":                       # X in, codes and mask out; weight codes in, Y out
        return dict(bytes=x * (e + q) + w + y * e, flops=2.0 * t_out * nw * c["c_out"])
    b = y * e + x * (e + q) + w + x * e + k * nw * (4 + q + 4)   # dY, X with codes and mask, weight codes, dX; rows idx
    f = 2.0 * t_out * nw * (c["c_out"] + k)
    if c["kind"] == "layer":
        b += x * q + w * (4 + q)                     # codes and masks out, the master weights in
        if c["forward"]:
            b += y * e
            f += 2.0 * t_out * nw * c["c_out"]
        if c["optimizer"]:
            b += k * nw * 8.0                        # momentum in and out (the weights take the place of dW)
    return dict(bytes=float(b), flops=f)


def tolerance(c):
    if c["kind"] == "select":
        return {"rel": 1e-12}                        # means of at most some thousand scores in double precision
    if c["kind"] == "forward":
        return {"rel": 7e-3} if c["dtype"] == "bf16" else {"rel": 1e-6}   # exact integer sums, one rounding of the result
    # dY and W_q are rounded to bf16 for the matrix cores, dX to its own type: dX is 2.4e-3 (single elements up to 1.5e-2)
    # from the same product in double precision
    return {"rel": 1e-2, "max": 6e-2}


# ------------------------------------------------------------------------------------------------------------------
def prepare(c, seed):
    s = SimpleNamespace(c=c)
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    if c["kind"] == "select":
        widths = [3 * c["c_in"], c["c_in"], 4 * c["c_in"], c["c_in"]] * c["N"]
        off = [0]
        for n in widths:
            off.append(off[-1] + n)
        s.off = torch.tensor(off, dtype=torch.int64, device="cuda")
        # mean |w| of rows of N(0, 0.02^2) weights: a narrow band, another level in every layer
        level = 0.016 * torch.exp(0.25 * torch.randn(len(widths), generator=g, device="cuda", dtype=torch.float64))
        s.scores = level.repeat_interleave(torch.tensor(widths, device="cuda"))
        s.scores *= 1 + 0.03 * torch.randn(off[-1], generator=g, device="cuda", dtype=torch.float64)
        s.k_total, s.k_layers = off[-1] * c["num"] // c["den"], max(1, len(widths) * c["num"] // c["den"])
        return s

    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    t_in, t_out, taps = _sizes(c)
    c_in, c_out, conv = c["c_in"], c["c_out"], c["N"] > 0
    s.k = _k(c)
    normal = lambda *shape: torch.randn(*shape, generator=g, device="cuda")  # noqa: E731
    e = lambda *shape, dtype=torch.float32: torch.empty(shape, dtype=dtype, device="cuda")  # noqa: E731
    s.x = (normal(c["N"], c["H"], c["W"], c_in).abs() if conv else normal(t_in, c_in)).to(dt)
    s.w = normal(c_out, c["kernel"], c["kernel"], c_in) if conv else normal(c_out, c_in)
    s.w *= 0.02
    mode = (ef.ACT_PER_TENSOR_ASYM, ef.W_PER_ROW_SYM)
    nw = taps * c_in
    s.fx = dict(codes=e(*s.x.shape, dtype=torch.uint8), clip_bits=e(t_in, (c_in + 31) // 32, dtype=torch.int32),
                scale=e(1), zero_point=e(1))
    s.fw = dict(codes=e(*s.w.shape, dtype=torch.int8), clip_bits=e(c_out, (nw + 31) // 32, dtype=torch.int32),
                scale=e(c_out))
    ef.fakequant_fwd(s.x, mode[0], c["a_bits"], out=s.fx)
    ef.fakequant_fwd(s.w.view(c_out, nw), mode[1], c["w_bits"], out=dict(s.fw, codes=s.fw["codes"].view(c_out, nw)))
    if not c["init"]:                                # trained scales are tighter than the data's range
        s.fx["scale"] *= 0.8
        s.fw["scale"] *= 0.8
        ef.fakequant_fwd(s.x, mode[0], c["a_bits"], init_minmax=False, out=s.fx)
        ef.fakequant_fwd(s.w.view(c_out, nw), mode[1], c["w_bits"], init_minmax=False,
                         out=dict(s.fw, codes=s.fw["codes"].view(c_out, nw)))
    lib = ef.lib()
    ws = lambda n: e(max(int(n), 256), dtype=torch.uint8)  # noqa: E731
    s.ws_x = ws(lib.efqat_fakequant_fwd_workspace_bytes(t_in, c_in, mode[0]))
    if c["kind"] == "forward" or c["forward"]:
        s.y = e(t_out, c_out, dtype=dt)
        s.ws_fwd = ws(lib.efqat_linear_fwd_workspace_bytes(t_in, c_in, c_out))
    if c["kind"] == "forward":
        return s

    # the gradient of a mean over the rows
    s.dy = normal(c_out, t_out) if c["layout"] else normal(t_out, c_out)
    s.dy = (s.dy / t_out).to(dt)
    code = ef.BF16 if c["dtype"] == "bf16" else ef.F32
    s.fw["scores"], s.fw["idx"] = e(c_out, dtype=torch.float64), e(s.k, dtype=torch.int32)
    s.ws_w = ws(lib.efqat_weight_quant_select_workspace_bytes(c_out))
    ef.channel_select(s.w, s.k, ws=s.ws_w, out=s.fw)
    s.out = dict(dx=e(*s.x.shape, dtype=dt), dw=e(s.k, *s.w.shape[1:]), ds_w=e(s.k), ds_x=e(1), dz_x=e(1))
    if conv:
        s.ws = ws(lib.efqat_conv_bwd_workspace_bytes(c["N"], c["H"], c["W"], c_in, c_out, c["kernel"], c["kernel"],
                                                     c["stride"], c["pad"], s.k, code, c["layout"]))
        s.geometry = dict(stride=c["stride"], pad=c["pad"])
    else:
        s.ws = ws(lib.efqat_linear_bwd_workspace_bytes(t_in, c_in, c_out, s.k, code, c["layout"]))
        s.geometry = {}
    s.backward = ef.conv_bwd if conv else ef.linear_bwd
    s.side = torch.cuda.Stream() if c["side"] else None
    s.step = None
    if c["optimizer"]:
        s.step = dict(lr_w=1e-3, momentum=0.9, weight_decay=5e-4, mom_w=torch.zeros_like(s.w), lr_s=1e-6,
                      adam_m=torch.zeros(c_out, device="cuda"), adam_v=torch.zeros(c_out, device="cuda"),
                      adam_t=torch.zeros(c_out, dtype=torch.int32, device="cuda"))
    if c["bias"]:
        s.db = e(c_out)
        s.ws_b = ws(lib.efqat_bias_grad_workspace_bytes(t_out, c_out, c["layout"]))
    return s


def run(s):
    c = s.c
    if c["kind"] == "select":
        channels, per_layer = ef.network_select(s.scores, s.off, s.k_total)
        layers, unfrozen, means = ef.layer_select(s.scores, s.off, s.k_layers)
        return dict(channels=channels, per_layer=per_layer, layers=layers, unfrozen=unfrozen, means=means)
    got = {}
    if c["kind"] != "backward":
        ef.fakequant_fwd(s.x, ef.ACT_PER_TENSOR_ASYM, c["a_bits"], init_minmax=c["init"], ws=s.ws_x, out=s.fx)
        got["x"] = s.fx
    if c["kind"] == "layer":
        ef.weight_quant_select(s.w, c["w_bits"], s.k, init_minmax=c["init"], ws=s.ws_w, out=s.fw)
        got["w"] = s.fw
    if c["kind"] == "forward" or c["forward"]:
        ef.linear_fwd(s.fx["codes"], s.fx["scale"], s.fx["zero_point"], s.fw["codes"], s.fw["scale"], ws=s.ws_fwd, out=s.y)
        got["y"] = s.y
    if c["kind"] == "forward":
        return got
    if c["bias"]:
        ef.bias_grad(s.dy, dy_layout=c["layout"], ws=s.ws_b, out=s.db)
        got["db"] = s.db
    got["grads"] = s.backward(s.dy, s.fx["codes"], s.fx["clip_bits"], s.x, s.fx["scale"], s.fx["zero_point"],
                              s.fw["codes"], s.fw["clip_bits"], s.w, s.fw["scale"], s.fw["idx"] if s.k else None,
                              dy_layout=c["layout"], ws=s.ws, out=s.out, step=s.step, side_stream=s.side, **s.geometry)
    if s.step:
        got["updated"] = dict(w=s.w, **{n: s.step[n] for n in ("mom_w", "adam_m", "adam_v", "adam_t")})
    return got
