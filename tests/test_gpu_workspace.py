"""The workspace: every solver's arrays share one region, so whatever is left in it must not reach a result, and nothing is
written behind it.  Each call runs on a workspace of exactly the size gear_cache_bytes asks for, filled with zeros and with ones,
with a guard behind it."""
import pytest
import torch

import gear_workloads as gw
from paper_2403_05527_amd import binding as gb

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
GUARD = 1 << 16


def outputs(cfg, segs, rank, iters, n_lowrank, fill):
    w = gw.Workload("ws", B=cfg.B, H_kv=cfg.H_kv, H_q=cfg.H_q, n=cfg.n_prefill_max, bits=cfg.bits, group=cfg.group, outlier_ppm=cfg.outlier_ppm,
                    rank=rank, rank_chunk=rank, n_b=cfg.n_buf_cap, steps=1, seed=3)
    c = gb.GearCache(cfg, DEV)
    block = torch.empty(c.workspace_bytes + GUARD, dtype=torch.uint8, device=DEV)
    c.workspace = block[:c.workspace_bytes]

    def call(f, *a, **k):
        block[:c.workspace_bytes] = fill
        block[c.workspace_bytes:] = 0xA5
        got = f(*a, **k)
        assert bool((block[c.workspace_bytes:] == 0xA5).all()), "written behind the workspace"
        return got

    for j, n in enumerate(segs):
        call(c.compress, gw.make_keys(w, n, j % 3, DEV), gw.make_values(w, n, j % 3, DEV), rank, iters, None, seed=j,
             n_lowrank=None if n_lowrank is None else min(n, n_lowrank))
    res = []
    for which in (0, 1):
        res += list(c.export_codes(which)) + list(c.export_sparse(which)) + list(call(c.export_sparse_coo, which))
        for seg in range(min(len(segs), 2)):
            res += list(c.export_lowrank(which, seg))
    res += list(c.decompress())
    Kb, Vb = gw.make_keys(w, cfg.n_buf_cap, 5, DEV), gw.make_values(w, cfg.n_buf_cap, 5, DEV)
    gq = cfg.H_q // cfg.H_kv
    rows = 8 // gq
    q = torch.randn(cfg.B, cfg.H_q, rows, 128, generator=torch.Generator().manual_seed(1)).to(torch.float16).to(DEV)
    single = torch.cat([call(c.decode_attn, q[:, :, i:i + 1].contiguous(), Kb, Vb, 1) for i in range(rows)], dim=2)
    res.append(single)
    if cfg.rank_max > 0 and cfg.n_prefill_max > 256:   # as many query rows as a call takes always fit
        many = call(c.decode_attn_mq, q, Kb, Vb, 1, False)
        # two fp16 roundings, and sums of the same terms in another order
        assert torch.allclose(many.float(), single.float(), rtol=2e-3, atol=2e-3)
        res.append(many)
    return res


@pytest.mark.parametrize("B,H_kv,gq,bits,group,ppm,n_b,segs,chunks_max,rank,iters,n_lowrank,per_head", [
    (1, 2, 1, 2, 64, 20000, 20, [300, 20, 7], 2, 4, 3, None, False),           # Gram matrices, then flushed buffers
    (2, 3, 2, 4, 32, 20000, 64, [64, 64], 1, 3, 2, None, False),               # both tensors of at most 64 tokens
    (1, 3, 1, 2, 64, 20000, 255, [65, 255, 100], 2, 8, 3, None, False),        # 65..256 tokens: tensor by tensor
    (1, 2, 4, 4, 0, 20000, 20, [700, 20], 1, 2, 1, None, True),                # a single round
    (1, 2, 1, 2, 64, 20000, 20, [500, 20], 1, 0, 1, None, False),              # no low-rank term
    (1, 2, 1, 2, 128, 10000, 20, [8200, 20], 1, 4, 3, None, False),            # more than 8192 tokens
    (1, 2, 1, 2, 128, 150000, 20, [8200, 20], 1, 4, 3, None, False),           # with a channel-major copy of the keys
    (1, 1, 1, 2, 0, 0, 20, [8200, 20], 1, 2, 1, None, False),                  # the same without outliers, and a single round
    (1, 2, 1, 2, 64, 20000, 20, [9001], 0, 0, 3, None, True),
    (1, 3, 1, 2, 32, 20000, 20, [1100, 20], 1, 4, 3, 333, True),               # the low-rank term on the last rows
    (1, 1, 1, 2, 64, 20000, 20, [257] + [20] * 256, 256, 1, 2, None, False),   # more segments than the solvers' room holds records of
    (1, 1, 1, 2, 64, 20000, 255, [20] + [255] * 256, 256, 0, 1, None, False),  # ... or counts of the coordinate form
])
def test_nothing_is_read_from_it_or_written_behind_it(B, H_kv, gq, bits, group, ppm, n_b, segs, chunks_max, rank, iters, n_lowrank, per_head):
    cfg = gb.make_config(B, H_kv, H_kv * gq, bits, group, ppm, n_b, segs[0], chunks_max, rank,
                         flags=gb.GEAR_FLAG_V_FILTER_PER_HEAD if per_head else 0)
    a = outputs(cfg, segs, rank, iters, n_lowrank, 0)
    b = outputs(cfg, segs, rank, iters, n_lowrank, 0xFF)
    assert len(a) == len(b)
    for x, y in zip(a, b):
        assert x.shape == y.shape and torch.equal(x.contiguous().view(torch.uint8), y.contiguous().view(torch.uint8))
