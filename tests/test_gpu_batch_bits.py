"""A request's results do not depend on what else is in the launch (GPU): the same bits by itself, in a batch
and with loose bounds, on both sides of every rule that chooses a kernel or a tile by the size of the launch.
"""
import numpy as np
import pytest
import torch

import workloads as W
from sxgpu import GpuLayer, desc_of, log

pytestmark = pytest.mark.gpu

try:
    import paper_2606_01751_amd as sx
except Exception:  # pragma: no cover
    sx = None


def _work(hq, hkv, d, lengths, dtype, seed=0):
    specs = []
    for i, t in enumerate(lengths):
        a = max(1, t // 5)
        specs.append([(a, False, 0, None)] + ([(t - 2 * a, True, 40 + i, None)] if t > 2 * a else []) +
                     ([(min(a, t - a), False, 0, None)] if t > a else []))
    return W.custom_workload(specs, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, dtype=dtype, rope_base=1e4, seed=seed)


def _attention_bits(w, route):
    """Full and sparse attention (and, float32, two-pass scores) of the first request of w alone, with bounds as
    loose as the whole batch, and in the batch.  route(rows, keys, requests): the rule's answer, which has to
    differ between the first call and the last."""
    lengths = [r.n_tokens for r in w.requests]
    n, T, most = len(lengths), lengths[0], max(lengths)
    g = GpuLayer(w, W.layer_tensors(w, 0))
    g.run_sparse(0.2)
    rows = g.plan.budget(0.2)[1]
    alone = sx.Plan(desc_of(w), w.requests[:1], w.n_dst_blocks, w.n_src_blocks)
    few = alone.budget(0.2)[1]
    q, k, v = (g.t[x] for x in "qkv")
    cu = torch.tensor(w.token_offsets, dtype=torch.int32, device="cuda")
    full, sparse = [], []
    for cnt, bound in ((1, T), (1, most), (n, most)):
        out, lse = torch.zeros_like(q), torch.zeros(q.shape[:2], dtype=torch.float32, device="cuda")
        sx.full_attn(desc_of(w), q, k, v, cu, cnt, bound, out, lse)
        full.append((out[:T], lse[:T]))
    for p, bound in ((alone, few), (alone, T), (g.plan, rows)):
        out = torch.zeros_like(q)
        sx.sparse_attn(p, q, g.rows, g.n_rows, bound, g.k_cache, g.v_cache, out)
        sparse.append(out[:T])
    torch.cuda.synchronize()
    assert route(T, T, 1) != route(most, most, n), "full attention: both calls take one route"
    assert route(few, T, 1) != route(rows, most, n), "sparse attention: both calls take one route"
    for x, y in full[1:]:
        assert torch.equal(x, full[0][0]) and torch.equal(y, full[0][1])
    for x in sparse[1:]:
        assert torch.equal(x, sparse[0])
    assert torch.isfinite(full[0][0].float()).all() and sparse[0].any()
    if w.dtype == "f32":
        one = torch.zeros(w.total_tokens, dtype=torch.float32, device="cuda")
        sx.sparseq_score(alone, q, g.k_cache, one)
        g.score()
        torch.cuda.synchronize()
        assert torch.equal(one[:T], g.scores[:T])
    alone.close()


# 256 tiles of 32 columns are where the tiles of a launch get 32 instead of 16 of them; the last tile of the
# first request is partial at either width
@pytest.mark.parametrize("hq,hkv,d,lengths", [(8, 2, 64, (333, 400, 256, 500)), (28, 4, 128, (90, 300, 301)),
                                              (8, 8, 128, (201,) + (260,) * 16), (33, 1, 64, (70, 301))],
                         ids=lambda x: str(x).replace(" ", "")[:24])
def test_float32_tile_width(hq, hkv, d, lengths):
    log(f"[batch bits] f32 {hq}/{hkv}/{d} {lengths}")
    g = hq // hkv
    _attention_bits(_work(hq, hkv, d, lengths, "f32"), lambda rows, keys, n: (rows * g + 31) // 32 * hkv * n >= 256)


def _tile(rows, n, requests):
    """The product tile (features x rows) of the library's rule."""
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    best = None
    for bn, bm, cost in ((256, 256, 1.5), (256, 128, 0.95), (128, 128, 0.60), (128, 64, 0.46), (64, 64, 0.35)):
        c = -(-(-(-rows // bm) * requests * (n // bn)) // cu) * cost
        if best is None or c < 0.98 * best[0]:
            best = (c, (bn, bm))
    return best[1]


# rows of the request (of eight times as many tokens) and of the batch's others, features, k: every tile among
# the calls of all cases, more than one in each
@pytest.mark.parametrize("rows,others,n,k", [(60, (900, 800, 700), 4096, 192), (200, (120,) * 9, 6144, 320),
                                             (255, (40,) * 3, 512, 704), (129, (100, 300), 28672, 128)],
                         ids=lambda x: str(x).replace(" ", "")[:16])
def test_products(rows, others, n, k):
    log(f"[batch bits] product of {rows} rows with {others}, {k} -> {n}")
    tokens, counts = (8 * rows,) + others, (rows,) + others
    w = W.custom_workload([[(t, False, 0, None)] for t in tokens], n_q_heads=8, n_kv_heads=2, head_dim=128, dtype="bf16", rope_base=1e4)
    gen = torch.Generator().manual_seed(n + rows)
    x = torch.randn((w.total_tokens, k), generator=gen).bfloat16().cuda()
    wt = (torch.randn((n, k), generator=gen) / k ** 0.5).bfloat16().cuda()
    res = torch.randn((w.total_tokens, n), generator=gen).bfloat16().cuda()
    row = torch.cat([torch.arange(t, dtype=torch.int32) for t in tokens]).cuda()
    cnt = torch.tensor(counts, dtype=torch.int32, device="cuda")
    got, tiles = [], set()
    for many, bound in ((1, rows), (1, 8 * rows), (len(counts), max(counts)), (len(counts), max(tokens))):
        plan = sx.Plan(desc_of(w), w.requests[:many], w.n_dst_blocks, w.n_src_blocks)
        y = torch.zeros((w.total_tokens, n), dtype=torch.bfloat16, device="cuda")
        sx.gemm_rows(plan, row, cnt, bound, x, wt, y, residual=res)
        torch.cuda.synchronize()
        got.append(y[:rows])
        tiles.add(_tile(bound, n, many))
        plan.close()
    assert len(tiles) > 1, tiles
    for y in got[1:]:
        assert torch.equal(y, got[0])
    ref = x[:rows].float() @ wt.float().t() + res[:rows].float()
    assert (got[0].float() - ref).abs().max() <= 2.0 ** -7 * ref.abs().max()
