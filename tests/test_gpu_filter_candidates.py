"""Filter_s where it works on lists of candidates: the Value rows, whose rough threshold comes from the extremes of groups of entries,
and the Key channels, whose rough threshold comes from a sample of the rows (of all of them up to 2048 or 4096).  The sizes are those at which the number of candidates reaches the ends of the lists and of their register counts, and the
values those for which it does not fit (the selection then takes its other way): the set is the oracle's, entry by entry."""
import numpy as np
import pytest
import torch

from oracle import gear_oracle as go
from paper_2403_05527_amd import binding as gb

pytestmark = pytest.mark.gpu


def _values(kind, shape, seed):
    gen = torch.Generator().manual_seed(seed)
    x = torch.randn(shape, generator=gen)
    if kind == "grid":           # about fifty values: a threshold is shared by up to a few per cent of a vector
        x = torch.round(x * 8) / 8
    elif kind == "cliff":        # the wanted entries and many more share one value at either end
        u = torch.rand(shape, generator=gen)
        x = torch.where(u < 0.1, 3.0, torch.where(u > 0.9, -3.0, x.clamp(-2, 2)))
    elif kind == "zeros":        # most entries are zeros of both signs, the wanted ones few
        u = torch.rand(shape, generator=gen)
        x = torch.where(u < 0.99, torch.sign(torch.randn(shape, generator=gen)) * 0.0, x * 10)
    elif kind == "one sign":     # a bottom threshold at +0
        x = x.clamp_min(0.0) * torch.where(torch.rand(shape, generator=gen) < 0.5, 1.0, -0.0)
    elif kind == "extremes":     # the largest finite values and denormals
        u = torch.rand(shape, generator=gen)
        x = torch.where(u < 0.02, 65504.0, torch.where(u > 0.98, -65504.0, x * 1e-7))
    elif kind == "sorted":       # a channel's largest entries all lie together, none in most stretches of the sample
        x = x.sort(dim=2).values
    elif kind == "periodic":
        x = x + 4 * torch.sin(torch.arange(shape[2]) * (3.14159265 / 4))[:, None]
    elif kind == "few vectors":  # ties in some token rows and channels only: waves that go both ways
        t = (torch.arange(shape[2]) % 37 == 0)[:, None]
        x = torch.where(t, torch.sign(x), x)
    return x.to(torch.float16).to("cuda:0")


@pytest.mark.parametrize("kind,B,H,n,ppm", [
    ("normal", 1, 1, 16390, 20000), ("normal", 1, 2, 16385, 50000), ("normal", 2, 3, 8197, 100000), ("normal", 1, 7, 16384, 60000),
    ("normal", 2, 8, 8193, 20000), ("grid", 1, 8, 16387, 50000), ("cliff", 1, 5, 16385, 20000), ("zeros", 1, 4, 16386, 20000),
    ("one sign", 2, 4, 8195, 20000), ("extremes", 1, 8, 16384, 20000), ("few vectors", 1, 6, 16389, 20000), ("normal", 1, 8, 16384, 400000),
    # one token per wave
    ("normal", 1, 1, 20, 20000), ("normal", 1, 8, 70, 50000), ("normal", 1, 9, 131, 20000), ("grid", 2, 15, 66, 20000), ("normal", 1, 17, 65, 30000),
    ("normal", 1, 32, 513, 20000), ("normal", 1, 32, 300, 50000), ("normal", 1, 32, 257, 110000), ("grid", 1, 32, 301, 20000),
    ("cliff", 1, 32, 66, 20000), ("zeros", 1, 32, 67, 20000), ("one sign", 1, 32, 68, 20000), ("extremes", 1, 40, 65, 10000),
    ("few vectors", 1, 33, 257, 20000), ("normal", 1, 40, 130, 50000), ("normal", 1, 64, 65, 20000), ("normal", 1, 64, 65, 1), ("normal", 1, 41, 65, 500000),
    # Key channels: the sample holds every row / one row less than there are, a ragged last round of rows, long lists, no room for a list
    ("normal", 1, 2, 2047, 20000), ("normal", 1, 2, 2048, 20000), ("normal", 1, 2, 2049, 20000), ("normal", 1, 9, 2303, 10000), ("normal", 1, 2, 4096, 90000),
    ("normal", 1, 2, 4097, 90000), ("grid", 1, 3, 4099, 20000), ("cliff", 1, 2, 2100, 20000), ("zeros", 1, 2, 2600, 20000), ("one sign", 1, 2, 1500, 30000),
    ("extremes", 1, 2, 3000, 10000), ("few vectors", 1, 3, 5000, 20000), ("sorted", 1, 2, 6001, 20000), ("periodic", 1, 2, 8192, 20000),
    ("normal", 1, 1, 32768, 1), ("normal", 1, 1, 32768, 10000), ("normal", 1, 2, 32767, 50000), ("grid", 1, 1, 20001, 20000), ("sorted", 1, 1, 32768, 30000),
])
def test_sets_equal_the_oracle(kind, B, H, n, ppm):
    shape = (B, H, n, 128)
    K, V = _values(kind, shape, n + H), _values(kind, shape, n + H + 1)
    gc = gb.GearCache(gb.make_config(B, H, H, 2, 64, ppm, 20, n, 0, 2), "cuda:0")
    gc.compress(K, V, 0, 1, None)
    for which, x, want in ((0, K, go.filter_keys), (1, V, go.filter_values)):
        mask, vals = (t.cpu().numpy() for t in gc.export_sparse(which))
        x16 = x.cpu().numpy()
        m = want(x16, ppm)
        assert np.array_equal(mask.astype(bool), m), which
        assert np.array_equal(vals.view(np.uint16)[m], x16.view(np.uint16)[m]), which


@pytest.mark.parametrize("kind,H,n,ppm", [("normal", 2, 300, 20000), ("normal", 2, 5000, 20000), ("grid", 2, 5000, 20000), ("normal", 1, 9001, 10000),
                                          ("cliff", 9, 700, 20000), ("one sign", 2, 3000, 20000), ("normal", 40, 70, 20000)])
def test_one_group_per_vector(kind, H, n, ppm):
    """Per-vector grouping: the selection also finds the (scale, zero) of what it leaves."""
    shape = (1, H, n, 128)
    K, V = _values(kind, shape, n), _values(kind, shape, n + 1)
    gc = gb.GearCache(gb.make_config(1, H, H, 4, 0, ppm, 20, n, 0, 2), "cuda:0")
    gc.compress(K, V, 0, 1, None)
    for which, x, filt in ((0, K, go.filter_keys), (1, V, go.filter_values)):
        x16 = x.cpu().numpy()
        y = np.where(filt(x16, ppm), np.float16(0), x16).astype(np.float32)
        axes = 2 if which == 0 else (1, 3)
        lo, hi = y.min(axis=axes, keepdims=True), y.max(axis=axes, keepdims=True)
        scale = ((hi - lo) / np.float32(15)).astype(np.float16)
        _, got_scale, got_zero = (t.cpu().numpy().astype(np.float32) for t in gc.export_codes(which))
        assert np.array_equal(got_scale, np.broadcast_to(scale, got_scale.shape).astype(np.float32)), which
        assert np.array_equal(got_zero, np.broadcast_to(lo, got_zero.shape).astype(np.float32)), which
