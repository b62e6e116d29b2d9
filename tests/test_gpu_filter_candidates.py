"""Filter_s where it works on lists of candidates: the Value rows, whose rough threshold comes from the extremes of groups of entries,
and the Key channels, whose rough threshold comes from a sample of the rows (of all of them up to 2048 or 4096).  The sizes are those at
which the number of candidates reaches the ends of the lists and of their register counts, and the values those for which it does not
fit (the selection then takes its other way): the set is the oracle's, entry by entry."""
import numpy as np
import pytest
import torch

from oracle import gear_oracle as go
from paper_2403_05527_amd import binding as gb
from tests import parity_util as pu

pytestmark = pytest.mark.gpu


def _values(kind, shape, seed):
    return pu.values_of_kind(kind, shape, seed).to("cuda:0")


@pytest.mark.parametrize("kind,B,H,n,ppm", [
    ("normal", 1, 1, 16390, 20000), ("normal", 1, 2, 16385, 50000), ("normal", 2, 3, 8197, 100000), ("normal", 1, 7, 16384, 60000),
    ("normal", 2, 8, 8193, 20000), ("grid", 1, 8, 16387, 50000), ("cliff", 1, 5, 16385, 20000), ("zeros", 1, 4, 16386, 20000),
    ("one sign", 2, 4, 8195, 20000), ("extremes", 1, 8, 16384, 20000), ("few vectors", 1, 6, 16389, 20000), ("normal", 1, 8, 16384, 400000),
    # one token per wave
    ("normal", 1, 1, 20, 20000), ("normal", 1, 8, 70, 50000), ("normal", 1, 9, 131, 20000), ("grid", 2, 15, 66, 20000), ("normal", 1, 17, 65, 30000),
    ("normal", 1, 32, 513, 20000), ("normal", 1, 32, 300, 50000), ("normal", 1, 32, 257, 110000), ("grid", 1, 32, 301, 20000),
    ("cliff", 1, 32, 66, 20000), ("zeros", 1, 32, 67, 20000), ("one sign", 1, 32, 68, 20000), ("extremes", 1, 40, 65, 10000),
    ("few vectors", 1, 33, 257, 20000), ("normal", 1, 40, 130, 50000), ("normal", 1, 64, 65, 20000), ("normal", 1, 64, 65, 1), ("normal", 1, 41, 65, 500000),
])
def test_sets_equal_the_oracle(kind, B, H, n, ppm):
    shape = (B, H, n, 128)
    K, V = _values(kind, shape, n + H), _values(kind, shape, n + H + 1)
    gc = gb.GearCache(gb.make_config(B, H, H, 2, 64, ppm, 20, n, 0, 2), "cuda:0")
    gc.compress(K, V, 0, 1, None)
    for which, x, want in ((0, K, go.filter_keys), (1, V, go.filter_values)):
        _check_sparse(gc, which, x, want, ppm)


def _check_sparse(gc, which, x, want, ppm):
    """The exported sparse matrix against the oracle's, the batch elements behind the first against that one where they are its copies."""
    mask, vals = gc.export_sparse(which)
    if x.stride(0) == 0:
        assert torch.equal(mask, mask[:1].expand_as(mask)) and torch.equal(vals, vals[:1].expand_as(vals)), which
        mask, vals, x = mask[:1], vals[:1], x[:1]
    mask, vals, x16 = mask.cpu().numpy(), vals.cpu().numpy(), x.cpu().numpy()
    m = want(x16, ppm)
    assert np.array_equal(mask.astype(bool), m), which
    assert np.array_equal(vals.view(np.uint16)[m], x16.view(np.uint16)[m]), which


def _copies(x, rows=65536):
    """x [1, H, n, 128] as a view of as many batch elements as it takes for more than `rows` Key rows."""
    return x.expand(rows // (x.shape[1] * x.shape[2]) + 1, -1, -1, -1)


# (the segments of 1025 to 8192 tokens are one batch element over and over: that many Key rows go by lists of candidates)
@pytest.mark.parametrize("kind,H,n,ppm,group", [
    # the sample holds every row (up to 2048, up to 4096 rows), one row of each stretch (up to 8192), eight channels per block (beyond)
    ("normal", 2, 1025, 20000, 64), ("normal", 1, 2047, 20000, 64), ("normal", 2, 2048, 50000, 64), ("normal", 2, 2049, 20000, 64),
    ("normal", 3, 2303, 10000, 64), ("normal", 1, 4096, 20000, 64), ("normal", 2, 4097, 20000, 64), ("normal", 1, 8192, 30000, 64),
    ("normal", 1, 5000, 1000, 64), ("normal", 1, 32768, 1, 64), ("normal", 1, 32768, 10000, 64), ("normal", 2, 32767, 50000, 64),
    # sixteen channels per block beyond 8192 tokens; a ratio for which the vectors stay in registers
    ("normal", 16, 8195, 20000, 64), ("cliff", 17, 8193, 20000, 0), ("normal", 1, 4096, 60000, 64), ("normal", 1, 4096, 61000, 64),
    # beyond 8192 tokens ties at a ratio for which the lists have no room: from a channel-major copy
    ("grid", 1, 9001, 150000, 64), ("cliff", 2, 16385, 200000, 0), ("constant", 1, 8193, 300000, 64),
    # thresholds that many entries share: lists too long, at one end or at both; the channel a single value, or two
] + [(kind, 1, n, 20000, group) for kind in ("grid", "coarse grid", "cliff", "zeros", "one sign", "extremes", "few vectors", "sorted", "falling", "periodic",
                                             "constant", "two values", "one end", "half", "steps", "two channels") for n, group in (
    (1501, 64), (2048, 0), (4095, 0), (4096, 64), (6001, 0), (8192, 64), (9001, 0), (20001, 64), (32768, 0))])
def test_key_sets_equal_the_oracle(kind, H, n, ppm, group):
    K = _values(kind, (1, H, n, 128), n + H + ppm)
    x = K if n > 8192 else _copies(K)
    B = x.shape[0]
    print("case", kind, B, H, n, ppm, group, flush=True)
    gc = gb.GearCache(gb.make_config(B, H, H, 2, group, ppm, 20, n, 0, 2), "cuda:0")
    gc.compress(x.contiguous(), torch.zeros_like(x).contiguous(), 0, 1, None)
    _check_sparse(gc, 0, x, go.filter_keys, ppm)
    if group == 0:
        _check_one_group(gc, 0, K, go.filter_keys, ppm, 2)


@pytest.mark.parametrize("kind", ["normal", "cliff", "falling", "two channels"])
@pytest.mark.parametrize("slabs,n,ppm,group", [
    (32, 4097, 20000, 64), (33, 4097, 20000, 64), (32, 8192, 50000, 0), (33, 8191, 20000, 0),   # a round of blocks of 1024 threads; more of 512
    (15, 8193, 20000, 64), (16, 8193, 20000, 0), (32, 8195, 20000, 64), (33, 8195, 20000, 64),   # 8 channels; 1024; 1024; 512
    (16, 16001, 20000, 64), (17, 16001, 20000, 0), (49, 16001, 20000, 64), (50, 16001, 20000, 64), (32, 32768, 10000, 0),   # 8 channels; 1024; 8; 1024
])
def test_key_sets_in_blocks_of_either_size(kind, slabs, n, ppm, group):
    K = _values(kind, (1, 1, n, 128), n + slabs)
    x = K.expand(slabs, -1, -1, -1)
    print("case", kind, slabs, n, ppm, group, flush=True)
    gc = gb.GearCache(gb.make_config(slabs, 1, 1, 2, group, ppm, 20, n, 0, 2), "cuda:0")
    gc.compress(x.contiguous(), torch.zeros_like(x).contiguous(), 0, 1, None)
    _check_sparse(gc, 0, x, go.filter_keys, ppm)
    if group == 0:
        _check_one_group(gc, 0, K, go.filter_keys, ppm, 2)


@pytest.mark.parametrize("kind", ["normal", "two channels"])
@pytest.mark.parametrize("slabs,n,ppm,group", [
    (32, 4097, 20000, 64), (33, 8191, 20000, 0), (15, 8193, 20000, 64), (16, 8193, 20000, 0), (33, 8195, 20000, 64), (17, 16001, 20000, 0),
    (49, 16001, 20000, 64), (50, 16001, 20000, 64), (32, 32768, 10000, 0), (43, 2047, 20000, 0), (91, 1025, 20000, 64),
    # 8 channels; 1024 threads up to 3.5 % in nearly full rounds; 8 channels
    (10, 8000, 40000, 64), (17, 8000, 40000, 64), (64, 9500, 30000, 64), (61, 9500, 34000, 0), (64, 9500, 36000, 64), (80, 8504, 30000, 0), (80, 8504, 50000, 0)])
def test_key_sets_of_slabs_that_differ(kind, slabs, n, ppm, group):
    """Every slab is the first one with its channels turned by another number, and so are its set, values and parameters."""
    K = _values(kind, (1, 1, n, 128), n + slabs + 1)
    turned = lambda t: torch.cat([t.roll(37 * i, dims=-1) for i in range(slabs)])
    x = turned(K)
    print("case", kind, slabs, n, ppm, group, flush=True)
    gc = gb.GearCache(gb.make_config(slabs, 1, 1, 2, group, ppm, 20, n, 0, 2), "cuda:0")
    gc.compress(x, torch.zeros_like(x), 0, 1, None)
    mask, vals = gc.export_sparse(0)
    want = torch.from_numpy(go.filter_keys(K.cpu().numpy(), ppm)).cuda()
    assert torch.equal(mask.bool(), turned(want))
    assert torch.equal(torch.where(mask.bool(), vals, 0).view(torch.int16), torch.where(turned(want), x, 0).view(torch.int16))
    codes, scale, zero = gc.export_codes(0)
    for t in (codes, scale, zero):
        assert torch.equal(t, turned(t[:1]))
    if group == 0:
        _check_one_group(gc, 0, K, go.filter_keys, ppm, 2)


@pytest.mark.parametrize("kind,H,n,ppm", [("normal", 2, 300, 20000), ("normal", 2, 5000, 20000), ("grid", 2, 5000, 20000), ("normal", 1, 9001, 10000),
                                          ("cliff", 9, 700, 20000), ("one sign", 2, 3000, 20000), ("normal", 40, 70, 20000)])
def test_one_group_per_vector(kind, H, n, ppm):
    """Per-vector grouping: the selection also finds the (scale, zero) of what it leaves."""
    shape = (1, H, n, 128)
    K, V = _values(kind, shape, n), _values(kind, shape, n + 1)
    gc = gb.GearCache(gb.make_config(1, H, H, 4, 0, ppm, 20, n, 0, 2), "cuda:0")
    gc.compress(K, V, 0, 1, None)
    for which, x, filt in ((0, K, go.filter_keys), (1, V, go.filter_values)):
        _check_one_group(gc, which, x, filt, ppm, 4)


def _check_one_group(gc, which, x, filt, ppm, bits):
    """The (scale, zero) of the first batch element's vectors, outliers counted as 0."""
    x16 = x.cpu().numpy()
    y = np.where(filt(x16, ppm), np.float16(0), x16).astype(np.float32)
    axes = 2 if which == 0 else (1, 3)
    lo, hi = y.min(axis=axes, keepdims=True), y.max(axis=axes, keepdims=True)
    scale = ((hi - lo) / np.float32(2 ** bits - 1)).astype(np.float16)
    _, got_scale, got_zero = (t[:1].cpu().numpy().astype(np.float32) for t in gc.export_codes(which))
    assert np.array_equal(got_scale, np.broadcast_to(scale, got_scale.shape).astype(np.float32)), which
    assert np.array_equal(got_zero, np.broadcast_to(lo, got_zero.shape).astype(np.float32)), which
