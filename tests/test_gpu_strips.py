"""Compress calls large enough that a block of the quantization kernel walks several tiles of 128 tokens (a strip), at lengths that
are no multiple of a tile: what one tile leaves in LDS, the next tile's loads, the code words written one tile late, the lists of
the second tile on, rows without a low-rank term inside a strip.  The whole batch runs on the GPU; the oracle recomputes the first
and the last batch element (Keys are independent per head, Values per batch element)."""
import numpy as np
import pytest
import torch

import gear_workloads as gw
from tests import parity_util as pu

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


class Picked:
    """The views of some batch elements of a cache, for the comparisons of parity_util."""

    def __init__(self, cache, sel):
        self.cache, self.sel = cache, sel

    def export_codes(self, which):
        return [x[self.sel] for x in self.cache.export_codes(which)]

    def export_sparse(self, which):
        return [x[self.sel] for x in self.cache.export_sparse(which)]

    def export_sparse_coo(self, which):
        """The picked elements' entries of the coordinate form, their batch index renumbered."""
        c = self.cache
        per = c.cfg.H_kv * c.n_total * 128
        lin, vals = c.export_sparse_coo(which)
        parts = [(lin // per == b) for b in self.sel]
        return (torch.cat([lin[m] % per + i * per for i, m in enumerate(parts)]), torch.cat([vals[m] for m in parts]))

    def export_lowrank(self, which, seg):
        return [x[self.sel] for x in self.cache.export_lowrank(which, seg)]

    def decompress(self):
        return [x[self.sel] for x in self.cache.decompress()]


@pytest.mark.parametrize("B,H,n,bits,group,ppm,rank,iters,n_lowrank,per_head", [
    (5, 8, 3001, 2, 32, 20000, 4, 3, None, False),      # twelve strips of 256 tokens, the last of 185
    (7, 40, 1777, 4, 0, 20000, 4, 3, None, False),      # two strips, of 1024 and 753
    (7, 40, 1777, 2, 32, 50000, 2, 2, None, False),     # long overflow lists
    (20, 16, 1001, 2, 64, 20000, 4, 3, 500, True),      # one strip; the low-rank term begins inside its fourth tile
    (20, 16, 897, 4, 128, 20000, 8, 3, 1, False),       # a last tile of one row, the only one with a low-rank term
    (20, 16, 1023, 2, 128, 0, 3, 3, None, False),       # no Filter
    (9, 3, 6003, 4, 0, 20000, 2, 3, 2000, True),        # per-vector groups and the Filter per head, strips of 512 tokens
])
def test_strips_of_several_tiles(B, H, n, bits, group, ppm, rank, iters, n_lowrank, per_head):
    w = gw.Workload("strip", B=B, H_kv=H, H_q=H, n=n, bits=bits, group=group, outlier_ppm=ppm, rank=rank, rank_chunk=2, n_b=20, steps=1, seed=n)
    gc, _ = pu.make_pair(B, H, H, bits, group, ppm, 20, n, 0, rank, v_per_head=per_head)
    sel = [0, B - 1]
    oc = pu.go.OracleCache(2, H, H, 128, bits, group, ppm, per_head)
    K, V, ib = gw.make_keys(w, n, 0, DEV), gw.make_values(w, n, 0, DEV), gw.make_init_B(w, rank, 0, DEV)
    gc.compress(K, V, rank, iters, ib, n_lowrank=n_lowrank)
    kw = {} if n_lowrank is None else {"n_lowrank": n_lowrank}
    oc.compress(pu.np16(K[sel]), pu.np16(V[sel]), rank, iters, np.ascontiguousarray(pu.np16(ib)[:, sel]), **kw)
    got = Picked(gc, sel)
    pu.compare_components(got, oc)
    pu.compare_decompress(got, oc)
    pu.compare_lowrank_product(got, oc, 0)
