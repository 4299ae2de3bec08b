"""Top-K at the sizes where its kernels change or end a tile: one block with 1 / 4 / 8 / 16 keys per thread, the
four-launch chain beyond 16384 keys (1024 keys per block, 256 blocks at most), with distinct scores, with scores of few
values (more equal keys around the threshold than are ranked directly or kept), all equal, most of them zero, and with one
far outlier."""
import numpy as np
import pytest
import torch

import paper_2411_11038_amd as ef
from oracle import efqat_oracle as orc
from tests.gpu_util import dev
from workloads import synth

pytestmark = pytest.mark.gpu


def scores_of(kind, n):
    r = np.abs(synth.normal(777 + n, 0, (n,)))
    if kind == "distinct":
        return 0.016 * (1.0 + 0.02 * r)
    if kind == "equal":
        return np.full(n, 0.0625)
    if kind == "dead":                                 # nine of ten channels are 0: the threshold lies among them, or not
        return np.where(r < 1.6, 0.0, 0.016 * r)
    if kind == "few_values":
        return 0.5 + np.floor(r * 3.0)                 # about ten values
    s = 0.016 * (1.0 + 1e-9 * r)                       # a band far narrower than the first window next to the outlier
    s[n // 2] = 1e12
    return s


@pytest.mark.parametrize("kind", ["distinct", "few_values", "outlier", "equal", "dead"])
@pytest.mark.parametrize("n", [1, 63, 256, 257, 1024, 1025, 4096, 4097, 8193, 16384, 16385, 17 * 1024, 82944, 300001])
def test_selection_matches_the_oracle(n, kind):
    s = scores_of(kind, n)
    flat = dev(s)
    cuts = sorted({0, n // 7, n // 7, n // 2, n})      # layers of different width
    off = dev(np.array(cuts, dtype=np.int64))
    for k in sorted({1, n // 4, n // 2 + 1, n - 1, n} - {0}):
        ref = orc.top_k_channels(s, k)
        idx, per_layer = ef.network_select(flat, off, k)
        torch.cuda.synchronize()
        layer = np.searchsorted(np.array(cuts), ref, side="right") - 1
        assert np.array_equal(idx.cpu().numpy(), ref - np.array(cuts)[layer])
        assert np.array_equal(per_layer.cpu().numpy(), np.bincount(layer, minlength=len(cuts) - 1))


@pytest.mark.parametrize("n,k", [(300, 75), (16385, 5000), (20000, 0)])
def test_many_layers_are_flagged(n, k):
    s = scores_of("few_values", n)
    off = np.concatenate([[0], np.cumsum(1 + (np.arange(n) % 3))]).astype(np.int64)
    flat = np.repeat(s, np.diff(off))                  # equal scores within a layer: its mean is that score
    layers, width, _ = ef.layer_select(dev(flat), dev(off), k)
    torch.cuda.synchronize()
    ref = orc.top_k_channels(s, k)
    want = np.zeros(n, np.int64)
    want[ref] = np.diff(off)[ref]
    assert np.array_equal(layers.cpu().numpy(), ref) and np.array_equal(width.cpu().numpy(), want)


@pytest.mark.parametrize("c_out", [16384, 16385, 40000])
def test_channel_selection_with_either_scratch(c_out):
    w = synth.normal(5 + c_out, 1, (c_out, 4), std=0.02).astype(np.float32)
    k = c_out // 4
    idx, scores = ef.channel_select(dev(w), k)
    static = ef.channel_select_static(dev(w), k)
    both = ef.weight_quant_select(dev(w), 8, k)
    torch.cuda.synchronize()
    ref = orc.top_k_channels(scores.cpu().numpy(), k)
    for got in (idx, static, both["idx"]):
        assert np.array_equal(got.cpu().numpy(), ref)


def _by_bits(s, k):
    """The k largest by bit pattern as an unsigned number, equal ones by index; ascending index order."""
    return np.sort(np.lexsort((np.arange(s.size), ~s.view(np.uint64)))[:k])


# Scores with both values of the sign bit: the keys then differ in all 64 bits.  Not what channel_select makes, but the two
# calls take any doubles, and nothing may be written behind idx[k].
@pytest.mark.parametrize("kind", ["signs", "zeros", "nan"])
@pytest.mark.parametrize("n", [2, 48, 64, 65, 256, 1024, 5000, 16384, 20000])
def test_any_doubles_are_ordered_by_bit_pattern(n, kind):
    s = synth.normal(4100 + n, 0, (n,))
    if kind == "zeros":
        s = np.where(np.arange(n) % 3 == 0, -0.0, 0.0)
    elif kind == "nan":
        s = np.abs(s)
        s[n // 2:] = np.copysign(np.nan, -1.0)
        s[0] = np.inf
    off = np.arange(n + 1, dtype=np.int64)             # one score per layer: its mean is the score itself
    L, st = ef.lib(), torch.cuda.current_stream().cuda_stream
    flat, offd = dev(s), dev(off)
    for k in sorted({1, n // 3, n - 1} - {0}):
        want = _by_bits(s, k)
        for layers in (False, True):
            idx = torch.full((n + 64,), -7, dtype=torch.int32, device="cuda")
            per = torch.empty(n, dtype=torch.int32, device="cuda")
            if layers:
                ws = torch.empty(L.efqat_layer_select_workspace_bytes(n), dtype=torch.uint8, device="cuda")
                mean = torch.empty(n, dtype=torch.float64, device="cuda")
                rc = L.efqat_layer_select(flat.data_ptr(), offd.data_ptr(), n, k, mean.data_ptr(), idx.data_ptr(),
                                          per.data_ptr(), ws.data_ptr(), ws.numel(), st)
                torch.cuda.synchronize()
                want = _by_bits(mean.cpu().numpy(), k)  # -0.0 / 1 may lose its sign in the sum
            else:
                ws = torch.empty(L.efqat_network_select_workspace_bytes(n), dtype=torch.uint8, device="cuda")
                one = dev(np.array([0, n], dtype=np.int64))
                rc = L.efqat_network_select(flat.data_ptr(), one.data_ptr(), 1, n, k, idx.data_ptr(), per.data_ptr(),
                                            ws.data_ptr(), ws.numel(), st)
                torch.cuda.synchronize()
            got = idx.cpu().numpy()
            assert rc == 0 and np.array_equal(got[:k], want) and np.all(got[k:] == -7)


@pytest.mark.parametrize("kind", ["distinct", "few_values", "equal", "dead", "outlier", "signs"])
@pytest.mark.parametrize("n", [16385, 82944, 300001])
def test_a_workspace_without_room_for_the_chain_selects_the_same(n, kind):
    s = synth.normal(4100 + n, 0, (n,)) if kind == "signs" else scores_of(kind, n)
    flat, ws = dev(s), torch.empty(256, dtype=torch.uint8, device="cuda")
    cuts = dev(np.array([0, n // 7, n // 7, n // 2, n], dtype=np.int64))
    for k in (1, n // 4, n - 1, n):
        idx, per_layer = ef.network_select(flat, cuts, k, ws=ws)
        ref, ref_per = ef.network_select(flat, cuts, k)
        torch.cuda.synchronize()
        assert torch.equal(idx, ref) and torch.equal(per_layer, ref_per)


def test_scores_alone_are_workspace_enough():
    n = 20000
    small = torch.empty((n * 8 + 255) // 256 * 256, dtype=torch.uint8, device="cuda")
    w = dev(synth.normal(5, 1, (n, 4), std=0.02).astype(np.float32))
    idx, scores = ef.channel_select(w, n // 4)
    assert torch.equal(ef.channel_select(w, n // 4, ws=small)[0], idx)
    assert torch.equal(ef.weight_quant_select(w, 8, n // 4, ws=small)["idx"], idx)
    off = dev(np.arange(n + 1, dtype=np.int64))
    ref = ef.layer_select(scores, off, n // 3)
    got = ef.layer_select(scores, off, n // 3, ws=small)
    assert all(torch.equal(a, b) for a, b in zip(got, ref))
    for call in (lambda ws: ef.channel_select(w, 5, ws=ws), lambda ws: ef.layer_select(scores, off, 5, ws=ws)):
        with pytest.raises(Exception, match="workspace"):
            call(small[:-256])
