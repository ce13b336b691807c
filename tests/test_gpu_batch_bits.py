"""A request's results do not depend on what else is in the launch (GPU): the same bits by itself, in a batch
and with loose bounds, on both sides of every rule that chooses a kernel or a tile by the size of the launch.
"""
import numpy as np
import pytest
import torch

import workloads as W
from sxgpu import GpuLayer, attention_route, desc_of, log

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


# the request alone in 32-column workgroups of eight or four waves, the batch in the 256-column grid, and at the end
# in those of four and two waves: group sizes that do and do not divide 256 and 32, both head dims, partial last
# rounds (256, 128 and 64 keys) and key tiles
@pytest.mark.parametrize("hq,hkv,d,lengths", [
    (32, 8, 128, (600,) + (500, 550, 3, 640) * 2), (28, 4, 128, (701,) + (650,) * 6), (8, 2, 128, (385,) + (800,) * 20),
    (64, 16, 64, (700,) + (650, 690) * 3), (33, 1, 64, (129,) + (650,) * 12), (8, 8, 64, (63,) + (1000,) * 25),
    (64, 1, 128, (31,) + (300,) * 9), (16, 4, 64, (97,) + (120,) * 40), (6, 2, 64, (200,) + (64, 130) * 60),
    (8, 2, 128, (300,) + (290, 257) * 4)], ids=lambda x: str(x).replace(" ", "")[:24])
def test_bfloat16_attention(hq, hkv, d, lengths):
    log(f"[batch bits] bf16 {hq}/{hkv}/{d} {lengths}")
    _attention_bits(_work(hq, hkv, d, lengths, "bf16"), lambda rows, keys, n: attention_route(rows, keys, n, hq, hkv, d))


@pytest.mark.parametrize("hq,hkv,d,T,below", [(32, 8, 128, 1537, 1536), (16, 16, 64, 6000, 3072)], ids=["d128", "d64"])
def test_bfloat16_attention_at_the_rule(hq, hkv, d, T, below):
    """The last bound that goes to 32-column workgroups and the next, for full attention (with a request of T rows
    in the second call only) and for sparse attention."""
    log(f"[batch bits] at the rule {hq}/{hkv}/{d}")
    assert attention_route(below, T, 1, hq, hkv, d) and not attention_route(below + 1, T, 1, hq, hkv, d)
    n = below + 1 - 40
    w = W.custom_workload([[(T, False, 0, None)]], n_q_heads=hq, n_kv_heads=hkv, head_dim=d, dtype="bf16", rope_base=1e4, seed=d)
    g = GpuLayer(w, W.layer_tensors(w, 0))
    sx.kv_scatter(g.plan, g.t["k"], g.t["v"], g.k_cache, g.v_cache)
    g.set_rows([np.arange(T - n, T)])
    out = []
    for bound in (below, below + 1):
        o = torch.zeros_like(g.out)
        sx.sparse_attn(g.plan, g.t["q"], g.rows, g.n_rows, bound, g.k_cache, g.v_cache, o)
        out.append(o)
    torch.cuda.synchronize()
    assert torch.equal(out[0], out[1]) and out[0][:n].any(-1).all()
    # full attention takes its longest request as the number of keys too
    last = max(t for t in range(1, T) if attention_route(t, t, 1, hq, hkv, d))
    assert not attention_route(last + 1, last + 1, 1, hq, hkv, d)
    out = []
    for t in (last, last + 1):
        cu = torch.tensor([0, t], dtype=torch.int32, device="cuda")
        o = torch.zeros_like(g.out)
        sx.full_attn(desc_of(w), g.t["q"], g.t["k"], g.t["v"], cu, 1, t, o)
        out.append(o)
    torch.cuda.synchronize()
    rpw = 256 // (hq // hkv)
    same = last // rpw * rpw      # the rows of the row tiles that both calls fill
    assert torch.equal(out[0][:same], out[1][:same]) and out[1][:last + 1].any(-1).all()


# requests per launch: workgroups of eight, four and (d = 64) two waves, and the 256-column grid
@pytest.mark.parametrize("hq,hkv,d,counts", [(8, 2, 128, {1: 8, 3: 4, 24: 0}), (14, 2, 128, {1: 8, 2: 4, 24: 0}),
                                             (16, 4, 64, {1: 8, 2: 4, 4: 2, 24: 0})], ids=["g4", "g7", "d64"])
def test_bfloat16_attention_of_growing_scores(hq, hkv, d, counts):
    """Scores that outgrow the running maximum again and again (by more than 2^64 in the probability): in the first
    and the second half of any key tile of a round, in several of one, from a first tile of -inf on; and
    infinite scores and values."""
    log(f"[batch bits] growing scores {hq}/{hkv}/{d}")
    T = 640
    gen = torch.Generator().manual_seed(d)
    base = [torch.randn((T, h, d), generator=gen) for h in (hq, hkv, hkv)]
    desc = sx.make_desc(hq, hkv, d, "bf16", 1e4)
    for n, waves in counts.items():
        assert attention_route(T, T, n, hq, hkv, d) == waves
    # steps: (key, score in units of log2 e from there on), by a dimension that only this uses
    for steps, odd in (([(70, 90.0)], None), ([(100, 90.0), (161, 200.0)], None), ([(200, 100.0), (260, 190.0), (330, 400.0)], None),
                       ([(0, -900.0), (64, -500.0), (128, -300.0), (192, -100.0), (300, 0.0)], None), ([(600, 80.0)], None),
                       ([(0, -float("inf")), (64, 0.0)], None), ([(0, -float("inf")), (150, 0.0), (400, 100.0)], None),
                       ([(0, 0.0)], ("k", 500, float("inf"))), ([(0, 0.0)], ("v", 77, float("nan"))), ([(0, 0.0)], ("v", 639, float("inf")))):
        q, k, v = (x.clone() for x in base)
        q[..., 0] = 1.0
        k[..., 0] = 0.0
        for key, z in steps:
            k[key:, :, 0] = z * d ** 0.5
        if odd:
            (k if odd[0] == "k" else v)[odd[1], 0, 1] = odd[2]
        one = [x.bfloat16().cuda() for x in (q, k, v)]
        first = None
        for n in counts:
            t = [x.repeat(n, 1, 1) for x in one]
            cu = torch.arange(0, T * n + 1, T, dtype=torch.int32, device="cuda")
            out, lse = torch.zeros_like(t[0]), torch.zeros(t[0].shape[:2], dtype=torch.float32, device="cuda")
            sx.full_attn(desc, *t, cu, n, T, out, lse)
            torch.cuda.synchronize()
            first = first or (out, lse)
            for r in (0, n - 1):
                for x, y in ((out, first[0]), (lse, first[1])):
                    x = x[r * T:(r + 1) * T]
                    assert torch.equal(x.isnan(), y.isnan()) and torch.equal(x.nan_to_num(7.0), y.nan_to_num(7.0)), (n, steps, odd)
        a = first[0]
        if odd is None and steps[0][1] > -1e30:
            z = torch.einsum("ihd,jhd->hij", one[0].double().cpu(), one[1].double().cpu().repeat_interleave(hq // hkv, 1)) * d ** -0.5
            z.masked_fill_(torch.ones(T, T, dtype=torch.bool).triu(1), -float("inf"))
            ref = torch.einsum("hij,jhd->ihd", z.softmax(-1), one[2].double().cpu().repeat_interleave(hq // hkv, 1))
            assert (a.double().cpu() - ref).abs().max() <= 4e-2, steps


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
