"""The single-launch read, and query columns shared by several blocks, at the edges of what they accept: no buffer rows, buffer rows at the edges of a wave's 32, chunks of two
pieces (one of them empty), as many waves as a block holds and one more (the split kernel), every number of query columns, causal
rows that see none of a wave's buffer rows, a rank whose rows are not one read."""
import pytest
import torch

import gear_workloads as gw
from tests import parity_util as pu

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("H,gq,bits,g,rank,n,n_b,chunks,n_bufs,q_len,slab_copies", [
    (2, 1, 2, 64, 4, 0, 64, (), (1, 32, 33, 64), 1, 1),              # nothing but buffer rows
    (2, 1, 4, 32, 3, 129, 20, (20, 1), (0, 20), 1, 1),                # a second prefill wave of one row, rank 3, no buffer wave
    (1, 2, 2, 0, 4, 128, 255, (255, 20), (0, 255), 1, 256),           # 256 slabs: chunks of two pieces, one of them empty; eight buffer waves
    (2, 4, 4, 128, 8, 300, 40, (40,), (33, 4), 1, 1),                 # four columns
    (2, 2, 2, 64, 2, 200, 64, (7,), (64, 34), 4, 1),                  # four causal rows of two heads: some see none of the second
                                                                      # buffer wave's rows
    (2, 2, 2, 64, 2, 200, 64, (7,), (64, 34), 4, 128),                # the same, eight columns in one block
    (2, 2, 4, 32, 2, 1700, 64, (7,), (64, 4), 4, 64),                 # the same in the split kernel
    (1, 1, 2, 64, 4, 2100, 64, (7,), (64, 8), 8, 2),                  # eight causal rows over blocks of fewer columns
    (8, 1, 2, 64, 4, 1900, 20, (), (20, 0), 1, 32),                   # 256 slabs: sixteen waves in the block
    (8, 1, 2, 64, 4, 1900, 20, (5,), (20, 0), 1, 32),                 # one more: the split kernel; sixteen without a buffer
])
def test_single_read(H, gq, bits, g, rank, n, n_b, chunks, n_bufs, q_len, slab_copies):
    w = gw.Workload("single", B=1, H_kv=H, H_q=H * gq, n=max(n, 1), bits=bits, group=g, outlier_ppm=30000, rank=rank,
                    rank_chunk=2, n_b=n_b, steps=1, seed=900 + n + n_b)
    print("case", w, chunks, n_bufs, q_len, flush=True)
    B = slab_copies                                                   # the same batch element over and over: one oracle element serves all
    gc, _ = pu.make_pair(B, H, H * gq, bits, g, 30000, n_b, max(n, 1), max(1, len(chunks)), rank)
    _, oc = pu.make_pair(1, H, H * gq, bits, g, 30000, n_b, max(n, 1), max(1, len(chunks)), rank)
    rep = lambda t: t.repeat(B, 1, 1, 1).contiguous()
    segs = ([(n, rank)] if n else []) + [(c, 2) for c in chunks]
    for j, (m, r) in enumerate(segs):
        K, V = gw.make_keys(w, m, j, DEV), gw.make_values(w, m, j, DEV)
        ib = gw.make_init_B(w, r, j, DEV)
        gc.compress(rep(K), rep(V), r, 3, ib.repeat(1, B, 1, 1, 1).contiguous())
        oc.compress(pu.np16(K), pu.np16(V), r, 3, pu.np16(ib))
    Kb, Vb = gw.make_keys(w, n_b, 50, DEV), gw.make_values(w, n_b, 50, DEV)
    q = torch.cat([gw.make_queries(w, j, DEV) for j in range(q_len)], dim=2)
    for n_buf in n_bufs:
        if q_len == 1:
            got = gc.decode_attn(rep(q), rep(Kb), rep(Vb), n_buf)
            oc.decode_attn(pu.np16(q), pu.np16(Kb), pu.np16(Vb), n_buf)
            want = oc.last_attn_f64
        else:
            got = gc.decode_attn_mq(rep(q), rep(Kb), rep(Vb), n_buf, True)
            want = pu.go.decode_attn_multi(oc, pu.np16(q), pu.np16(Kb), pu.np16(Vb), n_buf, True)
        assert torch.equal(got, got[:1].expand_as(got)), "equal batch elements, equal results"
        print("  n_buf", n_buf, pu.check_attention(pu.np16(got[:1]), want), flush=True)


@pytest.mark.parametrize("H,gq,n_buf,low", [(2, 1, 33, 32), (2, 4, 70, 64), (32, 1, 96, 64)])
def test_buffer_rows_of_minus_infinity_weigh_nothing(H, gq, n_buf, low):
    """Rows from `low` on score -inf: they are all that the last wave has, and the read is the one without them."""
    print("case", H, gq, n_buf, low, flush=True)
    gen = torch.Generator(device=DEV).manual_seed(n_buf)
    t = lambda *shape: torch.randn(*shape, generator=gen, device=DEV).half()
    gc, _ = pu.make_pair(1, H, H * gq, 2, 64, 20000, 128, 300, 1, 4)
    gc.compress(t(1, H, 300, 128), t(1, H, 300, 128), 4, 3, None)
    K, V, q = t(1, H, 128, 128), t(1, H, 128, 128), t(1, H * gq, 1, 128)
    q[..., 0] = -1.0
    want = gc.decode_attn(q, K, V, low)
    K[:, :, low:, 0] = float("inf")
    got = gc.decode_attn(q, K, V, n_buf)
    assert torch.equal(got, want)
