"""Persistent attention grids: results do not depend on how the row tiles are shared out.

Sparse attention takes its row tiles from work queues held in the plan, full attention from
queue slots held by the library, and every launch must leave its counters at zero for the next.
These tests replay captured graphs (sparse attention keeps its plan counters under capture; full
attention switches to one workgroup per row tile), interleave eager calls of other sizes between
the replays, and run full attention on two streams at once, comparing every result with the first
eager one bit for bit (each row tile is computed by one workgroup with the same arithmetic,
whichever workgroup takes it).
"""
from __future__ import annotations

import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

try:
    import paper_2606_01751_amd as sx
    from sxgpu import GpuLayer, attention_route, desc_of, dev, log
except Exception:  # pragma: no cover - collected without the library
    sx = None


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    sx.lib()


@pytest.fixture(params=[(32, 8, 128), (64, 16, 64)], ids=["d128", "d64"])
def w(request):
    """Three requests (1700, 513 and 2600 tokens), bf16, large enough that every launch below, the first request's
    own among them, goes to the 256-column grid."""
    hq, hkv, d = request.param
    rng = np.random.default_rng(11)
    specs = [W.random_request_specs(rng, T, max_seg=90) for T in (1700, 513, 2600)]
    return W.custom_workload(specs, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, dtype="bf16", rope_base=1e4,
                             rope_style="neox", seed=11, plant_per_segment=3, name="persist")


def _on_the_grid(w, rows, requests, keys=None):
    assert attention_route(rows, keys or rows, requests, w.n_q_heads, w.n_kv_heads, w.head_dim) == 0


def test_full_attention_graph_replays_and_two_streams(w):
    log("[persistent] full attention: eager, 3 graph replays, two streams")
    t = W.layer_tensors(w, 0)
    q, k, v = dev(t["q"], w), dev(t["k"], w), dev(t["v"], w)
    cu = torch.tensor(w.token_offsets, dtype=torch.int32, device="cuda")
    n_req, max_t = len(w.requests), max(r.n_tokens for r in w.requests)
    # the first request alone: a launch of another size between the replays
    cu1 = torch.tensor(w.token_offsets[:2], dtype=torch.int32, device="cuda")
    t1 = w.requests[0].n_tokens
    _on_the_grid(w, max_t, n_req)
    _on_the_grid(w, t1, 1)

    def run(out, stream=None):
        sx.full_attn(desc_of(w), q, k, v, cu, n_req, max_t, out, stream=stream)

    want = torch.zeros_like(q)
    run(want)
    torch.cuda.synchronize()
    assert torch.isfinite(want.float()).all()
    out_g = torch.zeros_like(q)
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        run(out_g)
    other, first = torch.zeros_like(q), torch.zeros_like(q)
    for i in range(3):
        out_g.zero_()
        other.zero_()
        first.zero_()
        run(other)
        sx.full_attn(desc_of(w), q, k, v, cu1, 1, t1, first)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out_g, want), f"replay {i}"
        assert torch.equal(other, want), f"eager call before replay {i}"
        assert torch.equal(first[:t1], want[:t1]), f"one-request call before replay {i}"
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    o1, o2 = torch.zeros_like(q), torch.zeros_like(q)
    torch.cuda.synchronize()
    with torch.cuda.stream(s1):
        run(o1)
    with torch.cuda.stream(s2):
        run(o2)
    torch.cuda.synchronize()
    assert torch.equal(o1, want) and torch.equal(o2, want)


def test_sparse_attention_graph_replays_and_fewer_rows(w):
    log("[persistent] sparse attention: eager, 3 graph replays, calls with fewer rows between them")
    g = GpuLayer(w, W.layer_tensors(w, 0))
    ratio = 0.3
    g.realign()
    g.scatter_nonreused()
    g.score()
    g.select(ratio)
    g.scatter_rows(ratio)
    m = g.plan.budget(ratio)[1]
    _on_the_grid(w, m, len(w.requests), max(r.n_tokens for r in w.requests))

    def run(out, n_rows, stream=None):
        sx.sparse_attn(g.plan, g.t["q"], g.rows, n_rows, m, g.k_cache, g.v_cache, out, stream=stream)

    want = torch.zeros_like(g.out)
    run(want, g.n_rows)
    torch.cuda.synchronize()
    n = g.n_rows.cpu().numpy()
    offs = w.token_offsets
    assert n.min() > 2
    half = torch.from_numpy((n // 2).astype(np.int32)).to("cuda")
    out_g = torch.zeros_like(g.out)
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        run(out_g, g.n_rows)
    fewer = torch.zeros_like(g.out)
    for i in range(3):
        out_g.zero_()
        fewer.zero_()
        run(fewer, half)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out_g, want), f"replay {i}"
        for r in range(len(w.requests)):
            a, b = offs[r], offs[r] + int(n[r] // 2)
            assert torch.equal(fewer[a:b], want[a:b]), f"request {r} with half its rows before replay {i}"
            assert not fewer[b:offs[r] + int(n[r])].any(), f"request {r}: rows past the bound written"


def test_sparse_attention_planned_tile_order(w):
    """sx_rows_mask plans the order in which sx_sparse_attn takes its row tiles for the same row list;
    the result must not change, also when n_rows changes at the same address after the plan was
    made (the attention then sees a different tile count and keeps the queue's own order)."""
    log("[persistent] sparse attention with the planned tile order of sx_rows_mask")
    g = GpuLayer(w, W.layer_tensors(w, 0))
    ratio = 0.3
    g.realign()
    g.scatter_nonreused()
    g.score()
    g.select(ratio)
    g.scatter_rows(ratio)
    m = g.plan.budget(ratio)[1]
    _on_the_grid(w, m, len(w.requests), max(r.n_tokens for r in w.requests))
    want = torch.zeros_like(g.out)
    sx.sparse_attn(g.plan, g.t["q"], g.rows, g.n_rows, m, g.k_cache, g.v_cache, want)
    mask = torch.zeros(w.total_tokens, dtype=torch.uint8, device="cuda")
    sx.rows_mask(g.plan, g.rows, g.n_rows, m, mask)
    for i in range(2):
        out = torch.zeros_like(g.out)
        sx.sparse_attn(g.plan, g.t["q"], g.rows, g.n_rows, m, g.k_cache, g.v_cache, out)
        torch.cuda.synchronize()
        assert torch.equal(out, want), f"planned order, call {i}"
    n = g.n_rows.cpu().numpy()
    g.n_rows.copy_(torch.from_numpy((n // 2).astype(np.int32)))
    out = torch.zeros_like(g.out)
    sx.sparse_attn(g.plan, g.t["q"], g.rows, g.n_rows, m, g.k_cache, g.v_cache, out)
    torch.cuda.synchronize()
    offs = w.token_offsets
    for r in range(len(w.requests)):
        a, b = offs[r], offs[r] + int(n[r] // 2)
        assert torch.equal(out[a:b], want[a:b]), f"request {r} with half its rows after the plan"
        assert not out[b:offs[r] + int(n[r])].any()


def test_many_launches_cycle_every_queue_slot(w):
    """70 full-attention launches (more than the 64 library queue slots, so every slot is reused)
    of three sizes in turn, and 30 sparse-attention launches on one plan with three row counts in
    turn: every result is bit-identical to the first one of its size, so each launch left its
    counters at zero."""
    log("[persistent] 70 full-attention and 30 sparse-attention launches in turn")
    t = W.layer_tensors(w, 0)
    q, k, v = dev(t["q"], w), dev(t["k"], w), dev(t["v"], w)
    offs = w.token_offsets
    n_req = len(w.requests)
    # full attention over the first 1, 2 and 3 requests
    sizes = [(torch.tensor(offs[:i + 2], dtype=torch.int32, device="cuda"), i + 1,
              max(r.n_tokens for r in w.requests[:i + 1])) for i in range(n_req)]
    want = []
    for cu, nr, mx in sizes:
        _on_the_grid(w, mx, nr)
        o = torch.zeros_like(q)
        sx.full_attn(desc_of(w), q, k, v, cu, nr, mx, o)
        want.append(o)
    torch.cuda.synchronize()
    outs = []
    for i in range(70):
        cu, nr, mx = sizes[i % n_req]
        o = torch.zeros_like(q)
        sx.full_attn(desc_of(w), q, k, v, cu, nr, mx, o)
        outs.append(o)
    torch.cuda.synchronize()
    for i, o in enumerate(outs):
        assert torch.equal(o, want[i % n_req]), f"full-attention launch {i}"
    g = GpuLayer(w, t)
    ratio = 0.3
    g.realign()
    g.scatter_nonreused()
    g.score()
    g.select(ratio)
    g.scatter_rows(ratio)
    m = g.plan.budget(ratio)[1]
    _on_the_grid(w, m, len(w.requests), max(r.n_tokens for r in w.requests))
    n = g.n_rows.cpu().numpy()
    counts = [torch.from_numpy(np.maximum(n // d, 1).astype(np.int32)).to("cuda") for d in (1, 2, 3)]
    ref = []
    for c in counts:
        o = torch.zeros_like(g.out)
        sx.sparse_attn(g.plan, g.t["q"], g.rows, c, m, g.k_cache, g.v_cache, o)
        ref.append(o)
    torch.cuda.synchronize()
    outs = []
    for i in range(30):
        o = torch.zeros_like(g.out)
        sx.sparse_attn(g.plan, g.t["q"], g.rows, counts[i % 3], m, g.k_cache, g.v_cache, o)
        outs.append(o)
    torch.cuda.synchronize()
    for i, o in enumerate(outs):
        assert torch.equal(o, ref[i % 3]), f"sparse-attention launch {i}"


# key-value heads (32 workgroups per head at 8, 64 at 4, no plan for more: 2)
@pytest.mark.parametrize("hq,hkv", [(32, 8), (28, 4), (16, 2)])
def test_every_planned_order_takes_every_tile_once(hq, hkv):
    """The order that sx_rows_mask plans for row counts that leave fewer tiles than workgroups, as many, a few more
    and several times as many, all of one cost and of very different ones; and for a count that changed
    after planning.  Against the same calls on a plan without an order, bit for bit: a tile taken twice or
    left out would show in the rows that it has to write."""
    log(f"[persistent] planned orders {hq}/{hkv}")
    lengths = (6000, 300, 5000)
    w = W.custom_workload([[(T, False, 0, None)] for T in lengths], n_q_heads=hq, n_kv_heads=hkv, head_dim=64, dtype="bf16",
                          rope_base=1e4, seed=2)
    g = GpuLayer(w, W.layer_tensors(w, 0))
    sx.kv_scatter(g.plan, g.t["k"], g.t["v"], g.k_cache, g.v_cache)
    other = sx.Plan(desc_of(w), w.requests, w.n_dst_blocks, w.n_src_blocks)
    bound, rpw = max(lengths), 256 // (hq // hkv)
    _on_the_grid(w, bound, len(lengths))
    per_head = torch.cuda.get_device_properties(0).multi_processor_count // hkv
    rng = np.random.default_rng(3)

    def some(n, T):      # n rows, the last ones or spread
        return np.sort(rng.choice(T, size=n, replace=False))

    tiles = lambda n: min(n * rpw, lengths[0])
    sets = [
        [some(1, 6000), some(0, 300), some(1, 5000)],                                   # two tiles
        [some(tiles(per_head - 1), 6000), some(1, 300), some(0, 5000)],                 # one per workgroup
        [some(tiles(per_head), 6000), some(1, 300), some(1, 5000)],                     # a few more
        [np.arange(6000), np.arange(300), np.arange(5000)],                             # several, falling costs
        [np.arange(6000 - 5 * rpw, 6000), some(0, 300), np.arange(5000 - 5 * rpw, 5000)],   # two costs, tied
        [np.arange(5), np.arange(5), np.arange(5)],                                     # all alike
        [some(0, 6000), some(0, 300), some(0, 5000)],                                   # nothing
    ]
    mask = torch.zeros(w.total_tokens, dtype=torch.uint8, device="cuda")
    for i, rows in enumerate(sets):
        g.set_rows(rows)
        sx.rows_mask(g.plan, g.rows, g.n_rows, bound, mask)
        for fewer in (0, 1, 300):
            g.n_rows.copy_(torch.tensor([max(0, len(r) - fewer) for r in rows], dtype=torch.int32))
            out = []
            for plan in (g.plan, other):
                o = torch.zeros_like(g.out)
                sx.sparse_attn(plan, g.t["q"], g.rows, g.n_rows, bound, g.k_cache, g.v_cache, o)
                out.append(o)
            torch.cuda.synchronize()
            assert torch.equal(out[0], out[1]), (i, fewer)
            for off, r in zip(w.token_offsets, rows):
                n = max(0, len(r) - fewer)
                assert out[0][off:off + n].any(-1).all() and not out[0][off + n:off + len(r)].any(), (i, fewer)
    other.close()
