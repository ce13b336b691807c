"""bfloat16 attention on both sides of the rule that sends launches of few query rows to 32-column
workgroups (GPU): against the oracle, and the 256-column grids' replays and repeats bit for bit.

Tolerance: probabilities and outputs are bf16 (2^-8 of values below 4), as in the parity tests: 2e-2.
"""
import numpy as np
import pytest
import torch

import oracle as O
import workloads as W
from sxgpu import GpuLayer, attention_route, desc_of, dev, host, log, lse_route

pytestmark = pytest.mark.gpu

try:
    import paper_2606_01751_amd as sx
except Exception:  # pragma: no cover
    sx = None


def _work(hq, hkv, d, lengths, seed=0):
    specs = []
    for i, t in enumerate(lengths):
        a = max(1, t // 5)
        specs.append([(a, False, 0, None)] + ([(t - 2 * a, True, 40 + i, None)] if t > 2 * a else []) +
                     ([(min(a, t - a), False, 0, None)] if t > a else []))
    return W.custom_workload(specs, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, dtype="bf16", rope_base=1e4, seed=seed)


# (q heads, kv heads, d, request lengths): 1 to 33 columns, group sizes that do not divide 32, one key to several
# rounds; then launches of the 256-column grid in all three passes (full, sparse, log-sum-exp), the
# longest request's log-sum-exps in pieces of keys, with requests of few rows beside them
SHORT = [(8, 2, 64, (1, 4, 5, 8, 9)), (7, 1, 128, (37, 1)), (8, 8, 64, (15, 16, 17, 31, 33)), (28, 4, 128, (70, 129)),
         (33, 1, 64, (63, 2)), (64, 1, 128, (31,)), (8, 2, 128, (127, 128, 385, 640))]
LONG = [(32, 8, 128, (2100, 600, 500, 3)), (64, 16, 64, (2100, 650, 640)), (28, 4, 64, (2100, 1900, 700, 900))]


@pytest.mark.parametrize("hq,hkv,d,lengths", SHORT + LONG, ids=lambda x: str(x).replace(" ", ""))
def test_attention_routes(hq, hkv, d, lengths):
    log(f"[attn routes] {hq}/{hkv}/{d} {lengths}")
    w = _work(hq, hkv, d, lengths)
    t = W.layer_tensors(w, 0)
    q, k, v = (dev(t[n], w) for n in "qkv")
    cu = torch.tensor(w.token_offsets, dtype=torch.int32, device="cuda")
    out, lse = torch.zeros_like(q), torch.zeros((w.total_tokens, hq), dtype=torch.float32, device="cuda")
    sx.full_attn(desc_of(w), q, k, v, cu, len(lengths), max(lengths), out, lse)
    g = GpuLayer(w, t)
    g.realign()
    g.scatter_nonreused()
    g.score()
    g.select(0.2)
    g.scatter_rows(0.2)
    g.attend(0.2)
    torch.cuda.synchronize()
    n, most, bound = len(lengths), max(lengths), g.plan.budget(0.2)[1]
    probes = max(len(O.probe_positions(r.n_tokens, r.segments)) for r in w.requests)
    routes = attention_route(most, most, n, hq, hkv, d), attention_route(bound, most, n, hq, hkv, d), lse_route(probes, most, n, hq, hkv, d)
    if (hq, hkv, d, lengths) in LONG:
        assert routes[:2] == (0, 0) and routes[2][0] == 0 and routes[2][1] > 1
    else:
        assert all(routes[:2]) and routes[2] == (4, 1)
    got, glse, sparse, scores = host(out), host(lse), host(g.out), host(g.scores)
    rows, n_rows, kc, vc = g.rows.cpu().numpy(), g.n_rows.cpu().numpy(), host(g.k_cache), host(g.v_cache)
    scale = O.softmax_scale(d)
    rng = np.random.default_rng(1)
    for r, (req, off) in enumerate(zip(w.requests, w.token_offsets)):
        T = req.n_tokens
        qr, kr, vr = (t[n][off:off + T] for n in "qkv")
        some = np.unique(np.concatenate([[0, T - 1], rng.integers(0, T, 40)]))
        assert np.abs(got[off:off + T][some] - O.attention_rows(qr, kr, vr, some, scale)).max() <= 2e-2
        for i in some[:8]:
            z = np.einsum("hd,jhd->hj", qr[i].astype(np.float64), np.repeat(kr[:i + 1].astype(np.float64), hq // hkv, 1)) * scale
            want = z.max(1) + np.log(np.exp(z - z.max(1, keepdims=True)).sum(1))
            assert np.abs(glse[off + i] - want).max() <= 1e-3 * max(1.0, np.abs(want).max())
        keys, vals = O.gather_tokens(req, w, kc), O.gather_tokens(req, w, vc)
        R = rows[off:off + n_rows[r]].astype(np.int64)
        pick = np.unique(np.concatenate([[0, len(R) - 1], rng.integers(0, len(R), 40)]))
        ref = O.attention_rows(qr, keys, vals, R[pick], scale)
        assert np.abs(sparse[off + pick] - ref).max() <= 2e-2
        # every probe row gives each head probability 1
        probes = O.probe_positions(T, req.segments)
        assert abs(scores[off:off + T].sum() - hq * len(probes)) <= 1e-3 * hq * len(probes)


@pytest.mark.parametrize("hq,hkv,d,lengths", [SHORT[3], SHORT[-1], LONG[0], LONG[1]], ids=lambda x: str(x).replace(" ", ""))
def test_replays_and_repeats_are_identical(hq, hkv, d, lengths):
    """Graph replays with eager calls between them, all equal to the first eager result; a row list cut by
    max_rows leaves the further rows alone."""
    log(f"[attn routes] replay {hq}/{hkv}/{d} {lengths}")
    w = _work(hq, hkv, d, lengths, seed=3)
    g = GpuLayer(w, W.layer_tensors(w, 0))
    g.run_sparse(0.2)
    most = g.plan.budget(0.2)[1]
    q, k, v = (g.t[n] for n in "qkv")
    cu = torch.tensor(w.token_offsets, dtype=torch.int32, device="cuda")
    full, out = torch.zeros_like(q), torch.zeros_like(q)

    def both(o, f):
        sx.sparse_attn(g.plan, q, g.rows, g.n_rows, most, g.k_cache, g.v_cache, o)
        sx.full_attn(desc_of(w), q, k, v, cu, len(lengths), max(lengths), f)

    both(out, full)
    torch.cuda.synchronize()
    assert torch.equal(out, g.out)
    first = (out.clone(), full.clone())
    o2, f2 = torch.zeros_like(q), torch.zeros_like(q)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        both(o2, f2)
    side.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        both(o2, f2)
    for _ in range(3):
        o2.zero_()
        f2.zero_()
        graph.replay()
        both(out, full)
        torch.cuda.synchronize()
        assert torch.equal(o2, first[0]) and torch.equal(f2, first[1])
        assert torch.equal(out, first[0]) and torch.equal(full, first[1])
    cut = min(5, most)
    part = torch.full_like(q, 7.0)
    sx.sparse_attn(g.plan, q, g.rows, g.n_rows, cut, g.k_cache, g.v_cache, part)
    torch.cuda.synchronize()
    n_rows = g.n_rows.cpu().numpy()
    for r, off in enumerate(w.token_offsets[:-1]):
        n = min(cut, n_rows[r])
        assert (part[off + n:w.token_offsets[r + 1]] == 7.0).all()
        assert (part[off:off + n].float() - first[0][off:off + n].float()).abs().max() <= 2e-2


def test_more_requests_than_a_grid_dimension_holds():
    """70000 one-token requests: few enough items for the 32-column workgroups, too many requests for their grid.
    One key has probability 1, so an output is its value."""
    log("[attn routes] 70000 requests")
    n, d = 70000, 64
    gen = torch.Generator(device="cuda").manual_seed(4)
    q, v = (torch.randn((n, h, d), generator=gen, device="cuda").bfloat16() for h in (2, 1))
    cu = torch.arange(n + 1, dtype=torch.int32, device="cuda")
    out = torch.zeros_like(q)
    sx.full_attn(sx.make_desc(2, 1, d, "bf16", 1e4), q, v, v, cu, n, 1, out)
    torch.cuda.synchronize()
    assert torch.equal(out, v.expand_as(out))
