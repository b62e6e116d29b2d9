"""Filter and quantization at the edges of their tiles (chunks of 512 entries, tiles of 128 tokens, strips), on values with many
ties: thresholds that many entries equal, both thresholds at one value, signed zeros, constant vectors.  Codes, scales,
outlier places and values are whole numbers and bits: equal to the oracle's."""
import pytest
import torch

import gear_workloads as gw
from tests import parity_util as pu

pytestmark = pytest.mark.gpu


def _values(kind, shape, seed):
    gen = torch.Generator().manual_seed(seed)
    x = torch.randn(shape, generator=gen)
    if kind == "steps":        # a few dozen distinct values: every threshold is tied
        x = torch.round(x * 4) / 4
    elif kind == "signs":      # three values, zeros of both signs: the two thresholds meet
        x = torch.sign(x) * (torch.rand(shape, generator=gen) < 0.01) * torch.sign(torch.randn(shape, generator=gen))
    elif kind == "constant":
        x = torch.full(shape, -0.75)
    return x.to(torch.float16).to("cuda:0")


@pytest.mark.parametrize("kind,B,H,n,bits,group,ppm", [
    ("steps", 1, 2, 65, 2, 64, 20000), ("steps", 1, 3, 257, 4, 32, 50000), ("signs", 1, 2, 511, 2, 128, 20000),
    ("steps", 2, 4, 512, 4, 64, 10000), ("constant", 1, 5, 513, 2, 0, 20000), ("signs", 1, 2, 1025, 4, 0, 50000),
    ("normal", 1, 3, 2049, 2, 32, 20000), ("steps", 1, 2, 4097, 2, 64, 20000), ("steps", 2, 2, 8193, 2, 64, 20000),
    ("signs", 1, 9, 385, 2, 64, 500000), ("steps", 1, 2, 300, 2, 64, 1),
    ("steps", 1, 9, 8201, 2, 64, 20000),     # one slab past a multiple of eight: the grids decoded by XCD
    ("steps", 1, 33, 130, 4, 64, 20000), ("steps", 1, 2, 8192, 4, 128, 20000),
    ("steps", 1, 2, 256, 4, 0, 20000), ("normal", 2, 3, 64, 2, 32, 20000),   # the last sizes before the tensors of a call go apart, and together
])
def test_filter_and_codes_equal_the_oracle(kind, B, H, n, bits, group, ppm):
    w = gw.Workload("f", B=B, H_kv=H, H_q=H, n=n, bits=bits, group=group, outlier_ppm=ppm, rank=2, rank_chunk=2, n_b=64, steps=1, seed=n)
    gc, oc = pu.make_pair(B, H, H, bits, group, ppm, 64, n, 1, 2)
    for seg, ns in enumerate((n, 64)):   # the second segment: a flushed buffer
        pu.compress_both(gc, oc, _values(kind, (B, H, ns, 128), n + seg), _values(kind, (B, H, ns, 128), n + seg + 7), 2, w.iters,
                         gw.make_init_B(w, 2, seg, "cuda:0"))
    pu.compare_components(gc, oc)


@pytest.mark.parametrize("B,H,n,group,ppm,rank,per_head", [
    (1, 1, 1, 64, 20000, 2, False), (3, 7, 64, 64, 50000, 2, False), (2, 8, 33, 0, 20000, 1, False), (5, 32, 63, 32, 20000, 4, False),
    (1, 33, 20, 64, 20000, 2, False),                                      # too many heads
    (2, 12, 21, 0, 20000, 2, True), (2, 5, 40, 0, 0, 2, False),            # (scale, zero) of the Values without their Filter
    (1, 32, 257, 64, 20000, 4, False), (2, 32, 1024, 0, 20000, 2, False), (3, 32, 513, 64, 20000, 2, False),   # 32, 64 and 96 slabs
    (64, 1, 301, 64, 20000, 2, False), (4, 9, 515, 128, 20000, 8, False), (1, 16, 1023, 64, 50000, 3, False),
])
def test_selections_of_a_short_segment(B, H, n, group, ppm, rank, per_head):
    """Keys and Values selected in one launch, or in two: the edges of the rule, and blocks whose last tokens do not exist."""
    dev = "cuda:0"
    w = gw.Workload("s", B=B, H_kv=H, H_q=H, n=n, bits=2, group=group, outlier_ppm=ppm, rank=rank, rank_chunk=2, n_b=20, steps=1, seed=n + H)
    gc, oc = pu.make_pair(B, H, H, 2, group, ppm, 20, n, 0, rank, v_per_head=per_head)
    pu.compress_both(gc, oc, gw.make_keys(w, n, 0, dev), gw.make_values(w, n, 0, dev), rank, 3, gw.make_init_B(w, rank, 0, dev))
    pu.compare_components(gc, oc)


@pytest.mark.parametrize("n", [1, 31, 32, 33, 63, 64, 65, 129, 190])
@pytest.mark.parametrize("H,bits,group,ppm,rank,per_head", [(3, 2, 64, 400000, 0, False), (4, 4, 0, 150000, 2, False), (2, 2, 32, 300000, 0, True),
                                                            (9, 2, 128, 20000, 2, False)])
def test_outliers_of_a_tile_of_few_rows(n, H, bits, group, ppm, rank, per_head):
    """The lists of a tile's Values, by rows or by channels, and up to its fullest."""
    B, dev = 2, "cuda:0"
    w = gw.Workload("f", B=B, H_kv=H, H_q=H, n=n, bits=bits, group=group, outlier_ppm=ppm, rank=rank, rank_chunk=2, n_b=20, steps=1, seed=n + H)
    gc, oc = pu.make_pair(B, H, H, bits, group, ppm, 20, n, 0, max(rank, 1), v_per_head=per_head)
    pu.compress_both(gc, oc, gw.make_keys(w, n, 0, dev), gw.make_values(w, n, 0, dev), rank, 3, gw.make_init_B(w, rank, 0, dev))
    pu.compare_components(gc, oc)
    pu.compare_decompress(gc, oc)
