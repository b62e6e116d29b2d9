"""gear_decompress at the edges of its 64-token tiles, against the reconstruction from the exported components."""
import numpy as np
import pytest
import torch

import gear_workloads as gw
from paper_2403_05527_amd import binding as gb
from tests import parity_util as pu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits,group,n,rank,ppm", [
    (2, 64, 1, 4, 20000), (4, 64, 63, 3, 20000), (2, 32, 64, 8, 20000), (4, 32, 97, 1, 50000),
    (2, 64, 131, 2, 20000), (4, 64, 250, 4, 20000), (2, 128, 133, 4, 20000), (4, 128, 126, 2, 20000),   # a last piece with rows past the end
    (2, 128, 129, 2, 20000), (4, 0, 191, 5, 20000), (2, 0, 65, 4, 20000), (2, 32, 223, 0, 20000), (4, 128, 40, 8, 0),
])
def test_decompress_is_the_sum_of_its_components(bits, group, n, rank, ppm):
    dev = "cuda:0"
    w = gw.Workload("d", B=2, H_kv=3, H_q=3, n=n, bits=bits, group=group, outlier_ppm=ppm, rank=rank, rank_chunk=2, n_b=37, steps=1, seed=n)
    c = gb.GearCache(gb.make_config(2, 3, 3, bits, group, ppm, 37, n, 1, max(rank, 2)), dev)
    c.compress(gw.make_keys(w, n, 0, dev), gw.make_values(w, n, 0, dev), rank, 3, None, seed=1)
    c.compress(gw.make_keys(w, 37, 1, dev), gw.make_values(w, 37, 1, dev), 2, 3, None, seed=2)
    for which, got in enumerate(c.decompress()):
        got = pu.np16(got)
        codes, scale, zero = [pu.np16(x).astype(np.float64) for x in c.export_codes(which)]
        S = pu.np16(c.export_sparse(which)[1]).astype(np.float64)
        g, t0, g0 = group, 0, 0
        for seg, ns in enumerate((n, 37)):
            t = np.arange(ns)
            if which == 0:
                at = g0 + (np.zeros_like(t) if g == 0 else t // g)
                sc, ze = scale[:, :, at], zero[:, :, at]
                g0 += 1 if g == 0 else -(-ns // g)
            else:
                rep = 128 // scale.shape[-1]
                sc, ze = [np.repeat(x[:, :, t0:t0 + ns], rep, axis=3) for x in (scale, zero)]
            A, Bf = [pu.np16(x).astype(np.float64) for x in c.export_lowrank(which, seg)]
            terms = [codes[:, :, t0:t0 + ns] * sc, ze, S[:, :, t0:t0 + ns]] + [A[..., r:r + 1] * np.swapaxes(Bf[..., r:r + 1], -1, -2) for r in range(A.shape[-1])]
            want, size = sum(terms), sum(np.abs(x) for x in terms)
            # half a unit of the fp16 result, and one fp32 rounding (2^-24) of the terms' size for each of the at most
            # eleven additions, taken twice for the rounding of the products
            bar = 0.5 * np.spacing(np.abs(got[:, :, t0:t0 + ns]).astype(np.float16)).astype(np.float64) * (1 + 2.0 ** -10) + 22 * 2.0 ** -24 * size
            assert (np.abs(got[:, :, t0:t0 + ns].astype(np.float64) - want) <= bar).all(), (which, seg)
            t0 += ns


@pytest.mark.parametrize("B,H,bits,group,n,rank,ppm", [
    (2, 3, 2, 64, 131, 0, 400000), (2, 3, 4, 32, 97, 4, 400000),    # four rows of a thread, lists of more entries than threads
    (2, 3, 2, 128, 190, 3, 400000), (2, 3, 4, 64, 65, 7, 150000),   # eight rows
    (16, 32, 2, 64, 9, 1, 20000), (16, 33, 2, 32, 9, 1, 20000),     # 512 tiles: four rows; 528: eight
    (24, 16, 4, 64, 70, 8, 20000), (25, 31, 2, 64, 21, 8, 20000),   # 768: four rows; 775: eight
    (32, 32, 2, 64, 64, 4, 20000), (25, 41, 4, 32, 64, 2, 100000),  # 1024 full tiles: four rows; 1025: eight
    (25, 41, 2, 32, 67, 4, 20000), (25, 41, 4, 64, 65, 0, 0),       # ... eight
    (25, 41, 4, 64, 63, 4, 20000),                                  # 1025 that are not all full: four
    (25, 41, 4, 64, 64, 4, 100001), (25, 41, 2, 64, 64, 0, 400000), # ... four with long lists
])
def test_four_and_eight_rows_of_a_thread(B, H, bits, group, n, rank, ppm):
    dev = "cuda:0"
    print("case", B, H, bits, group, n, rank, ppm, flush=True)
    gen = torch.Generator(device=dev)
    gen.manual_seed(n + rank)
    K, V = [torch.randn(B, H, n, 128, generator=gen, device=dev).to(torch.float16) for _ in range(2)]
    c = gb.GearCache(gb.make_config(B, H, H, bits, group, ppm, 20, n, 0, max(rank, 1)), dev)
    c.compress(K, V, rank, 2, None, seed=1)
    for which, got in enumerate(c.decompress()):
        codes, scale, zero = [x.double() for x in c.export_codes(which)]
        S = c.export_sparse(which)[1].double()
        if which == 0:
            at = torch.arange(n, device=dev) // group
            scale, zero = scale[:, :, at], zero[:, :, at]
        else:
            scale, zero = [x.repeat_interleave(group, dim=3) for x in (scale, zero)]
        A, Bf = [x.double() for x in c.export_lowrank(which, 0)] if rank else (None, None)
        terms = [codes * scale, zero, S] + [A[..., r:r + 1] * Bf[..., r:r + 1].transpose(-1, -2) for r in range(rank)]
        want, size = sum(terms), sum(x.abs() for x in terms)
        # the same bar as above
        half = 0.5 * torch.from_numpy(np.spacing(np.abs(pu.np16(got)).astype(np.float16)).astype(np.float64)).to(dev)
        assert bool(((got.double() - want).abs() <= half * (1 + 2.0 ** -10) + 22 * 2.0 ** -24 * size).all()), which


@pytest.mark.parametrize("B,H,bits,n", [(192, 64, 4, 65), (193, 64, 2, 65)])   # 24576 tiles: four rows; 24704: eight
def test_rows_of_a_thread_without_a_lowrank_term(B, H, bits, n):
    test_four_and_eight_rows_of_a_thread(B, H, bits, 64, n, 0, 20000)
