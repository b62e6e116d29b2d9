"""The pass that writes A on the matrix cores: steps of 16 tokens and waves of 64 with a remainder, every rank (whole and single
stores), groups that change inside a wave's tokens, rows without a low-rank term, and entries far from 1, whose residuals and
projection matrix reach the matrix cores only through their scales."""
import numpy as np
import pytest

import gear_workloads as gw
from oracle import gear_oracle as go
from tests import parity_util as pu

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n,bits,group,ppm,rank,n_lowrank,size", [
    (257, 2, 32, 20000, 1, None, 1.0),
    (272, 4, 64, 20000, 2, None, 1.0),
    (319, 2, 128, 50000, 3, None, 1.0),
    (320, 4, 0, 20000, 4, None, 1.0),
    (321, 2, 64, 0, 5, 33, 1.0),         # no Filter; the low-rank term begins inside a step
    (527, 4, 32, 20000, 6, None, 1.0),
    (511, 2, 32, 500000, 7, None, 1.0),  # half of the entries outliers
    (513, 4, 128, 20000, 8, 1, 1.0),     # one row with a low-rank term
    (400, 2, 64, 20000, 4, None, 1.0 / 1024),
    (400, 4, 32, 20000, 8, None, 1.0 / 1024),
    (400, 2, 128, 20000, 4, None, 256.0),
    (400, 4, 0, 20000, 2, None, 256.0),
])
def test_projection(n, bits, group, ppm, rank, n_lowrank, size):
    B, H = 2, 3
    w = gw.Workload("projection", B=B, H_kv=H, H_q=H, n=n, bits=bits, group=group, outlier_ppm=ppm, rank=rank, rank_chunk=2, n_b=20,
                    steps=1, seed=n + rank)
    gc, oc = pu.make_pair(B, H, H, bits, group, ppm, 20, n, 0, rank)
    K, V = gw.make_keys(w, n, 0, DEV) * size, gw.make_values(w, n, 0, DEV) * size   # (a power of two)
    ib = gw.make_init_B(w, rank, 0, DEV)
    gc.compress(K, V, rank, 3, ib, n_lowrank=n_lowrank)
    kw = {} if n_lowrank is None else {"n_lowrank": n_lowrank}
    oc.compress(pu.np16(K), pu.np16(V), rank, 3, pu.np16(ib), **kw)
    pu.compare_components(gc, oc)
    pu.compare_lowrank_product(gc, oc, 0)


@pytest.mark.parametrize("n,rank,iters", [
    (270, 8, 3), (300, 4, 2), (384, 2, 5), (512, 5, 3), (513, 8, 2), (768, 1, 3), (896, 8, 5), (897, 4, 3),   # 3 to 8 partial Gram matrices
])
def test_solver(n, rank, iters):
    """Products on the Gram matrix, for every rank the kernel is built for (2, 4, 8) and ranks between, with one, two and four of them."""
    B, H = 1, 3
    w = gw.Workload("solver", B=B, H_kv=H, H_q=H, n=n, bits=2, group=64, outlier_ppm=20000, rank=rank, rank_chunk=2, n_b=20, steps=1,
                    seed=n + rank)
    gc, oc = pu.make_pair(B, H, H, 2, 64, 20000, 20, n, 0, rank)
    K, V = gw.make_keys(w, n, 0, DEV), gw.make_values(w, n, 0, DEV)
    ib = gw.make_init_B(w, rank, 0, DEV)
    pu.compress_both(gc, oc, K, V, rank, iters, ib)
    pu.compare_lowrank_product(gc, oc, 0)


@pytest.mark.parametrize("n,bits,group,rank,size", [(272, 2, 64, 4, 1.0), (700, 4, 128, 2, 1.0), (1030, 2, 32, 8, 1.0), (601, 2, 64, 4, 1.0 / 1024), (333, 4, 0, 3, 32.0)])
def test_error_of_the_factors_is_their_rounding(n, bits, group, rank, size):
    """Against the same steps in 64 bits the stored A is off by its rounding to fp16 (2^-12 of an entry at most, 2.1e-4 of the whole).  The operands' 22 bits
    and the sums in 32 add some 2^-20 of it, which is nothing next to that in quadrature, so 1 % more is allowed.  With
    the leading parts alone (11 bits) it would be 1.4 times as much."""
    H = 2
    w = gw.Workload("error", B=1, H_kv=H, H_q=H, n=n, bits=bits, group=group, outlier_ppm=20000, rank=rank, rank_chunk=2, n_b=20, steps=1, seed=n)
    gc, oc = pu.make_pair(1, H, H, bits, group, 20000, 20, n, 0, rank)
    K, V = gw.make_keys(w, n, 0, DEV) * size, gw.make_values(w, n, 0, DEV) * size
    ib = gw.make_init_B(w, rank, 0, DEV)
    pu.compress_both(gc, oc, K, V, rank, 3, ib)
    for which, (X, seg) in enumerate(((pu.np16(K), oc.K[0]), (pu.np16(V), oc.V[0]))):
        Dh = go.dequant_keys(seg.codes, seg.scale, seg.zero, group or n) if which == 0 else go.dequant_values(seg.codes, seg.scale, seg.zero, group or 128)
        R = np.where(seg.mask, np.float16(0), X).astype(np.float64) - Dh
        A = pu.np16(gc.export_lowrank(which, 0)[0]).astype(np.float64)
        exact = np.stack([go.svd_solver(R[0, h], pu.np16(ib)[which, 0, h], 3)[0] for h in range(H)])[None]
        rounding = np.linalg.norm(exact.astype(np.float16).astype(np.float64) - exact)
        assert np.linalg.norm(A - exact) <= 1.01 * rounding, which
