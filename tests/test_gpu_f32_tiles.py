"""float32 attention and column sums at the edges of their 16- and 32-column tiles (GPU).

Against float64 on the CPU.  Tolerances: a score is a sum of d float32 products, off by at most
d 2^-24 sum |q k| scale, 2e-5 for N(0, 1) inputs at d = 128; an output is a mean of values below 5
weighted by probabilities that far off, and a score sums probabilities: 1e-4 of its value.
"""
import numpy as np
import pytest
import torch

import oracle as O
import workloads as W
from sxgpu import GpuLayer, desc_of, host, log

pytestmark = pytest.mark.gpu

try:
    import paper_2606_01751_amd as sx
except Exception:  # pragma: no cover
    sx = None


def _full(desc, q, k, v, lengths):
    dev = [torch.from_numpy(x).cuda() for x in (q, k, v)]
    cu = torch.tensor([0] + list(np.cumsum(lengths)), dtype=torch.int32, device="cuda")
    out = torch.zeros_like(dev[0])
    lse = torch.zeros(q.shape[:2], dtype=torch.float32, device="cuda")
    sx.full_attn(desc, *dev, cu, len(lengths), max(lengths), out, lse)
    torch.cuda.synchronize()
    return host(out), host(lse)


# (q heads, kv heads, d, request lengths): columns of a request = length x heads per KV head, so 1 to 33
# columns, whole and partial tiles, group sizes that do not divide a tile; the last two lie on the two
# sides of the rule that chooses 32-column tiles (256 tiles)
SHAPES = [
    (8, 2, 64, (1, 4, 5, 8, 9)), (7, 1, 128, (37, 1)), (8, 8, 64, (15, 16, 17, 31, 33)), (28, 4, 64, (70,)),
    (16, 1, 128, (130,)), (32, 8, 64, (255,)), (32, 8, 128, (257, 64)),
]


@pytest.mark.parametrize("hq,hkv,d,lengths", SHAPES, ids=[f"{a}-{b}-{c}-{'.'.join(map(str, t))}" for a, b, c, t in SHAPES])
def test_full_attention_tiles(hq, hkv, d, lengths):
    log(f"[f32 tiles] full {hq}/{hkv}/{d} {lengths}")
    rng = np.random.default_rng(len(lengths) * d + hq)
    T = sum(lengths)
    q, k, v = (rng.standard_normal((T, h, d)).astype(np.float32) for h in (hq, hkv, hkv))
    out, lse = _full(sx.make_desc(hq, hkv, d, "f32", 1e4), q, k, v, lengths)
    off, g = 0, hq // hkv
    for n in lengths:
        for h in range(hq):
            z = q[off:off + n, h].astype(np.float64) @ k[off:off + n, h // g].astype(np.float64).T / np.sqrt(d)
            z[np.triu_indices(n, 1)] = -np.inf
            top = z.max(1, keepdims=True)
            p = np.exp(z - top)
            ref = p @ v[off:off + n, h // g].astype(np.float64) / p.sum(1, keepdims=True)
            assert np.abs(out[off:off + n, h] - ref).max() <= 1e-4
            assert np.abs(lse[off:off + n, h] - (top[:, 0] + np.log(p.sum(1)))).max() <= 1e-4
        off += n


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("hq,hkv", [(8, 2), (32, 8)], ids=["narrow", "wide"])
def test_masked_keys_may_hold_any_value(hq, hkv, d):
    """V rows with infinities and NaN reach the rows that see them and no other."""
    log(f"[f32 tiles] non-finite V {hq}/{hkv}/{d}")
    T, bad = 300, {45: np.inf, 46: -np.inf, 200: np.nan}
    rng = np.random.default_rng(9)
    q, k, v = (rng.standard_normal((T, h, d)).astype(np.float32) for h in (hq, hkv, hkv))
    desc = sx.make_desc(hq, hkv, d, "f32", 1e4)
    clean, _ = _full(desc, q, k, v, (T,))
    for j, x in bad.items():
        v[j, 0, 3] = x
    out, _ = _full(desc, q, k, v, (T,))
    g = hq // hkv
    assert np.array_equal(out[:45], clean[:45])
    assert np.isposinf(out[45, :g, 3]).all()
    assert np.isnan(out[46:, :g, 3]).all()
    rest = [x for x in range(d) if x != 3]
    assert np.array_equal(out[:, :g, rest], clean[:, :g, rest])
    assert np.array_equal(out[:, g:], clean[:, g:])


@pytest.mark.parametrize("hq,hkv,d", [(14, 2, 64), (8, 8, 128), (33, 1, 64)], ids=["g7", "g1", "g33"])
def test_scores_tiles(hq, hkv, d):
    log(f"[f32 tiles] scores {hq}/{hkv}/{d}")
    specs = [[(33, False, 0, None), (100, True, 7, None), (1, False, 0, None), (66, True, 0, None)], [(31, True, 4, None)],
             [(5, False, 0, None)]]
    w = W.custom_workload(specs, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, dtype="f32", rope_base=1e4, seed=d)
    t = W.layer_tensors(w, 0)
    g = GpuLayer(w, t)
    g.realign()
    g.scatter_nonreused()
    g.score()
    torch.cuda.synchronize()
    got, kc = host(g.scores), host(g.k_cache)
    for r, (req, off) in enumerate(zip(w.requests, w.token_offsets)):
        keys = O.gather_tokens(req, w, kc)
        ref = O.sparseq_scores(t["q"][off:off + req.n_tokens], keys, O.probe_positions(req.n_tokens, req.segments),
                               O.softmax_scale(d))
        have = got[off:off + req.n_tokens]
        assert np.all(np.abs(have - ref) <= 1e-4 * np.abs(ref) + 1e-7), r


def test_one_pass_scores_far_from_one():
    """Probabilities below the normal range count with what float32 holds of them, and those above it are
    infinite, never NaN.  Tolerance: 1e-4 of the value as above, and half a unit (2^-149) per subnormal probability."""
    log("[f32 tiles] one-pass scores far from one")
    specs = [[(33, False, 0, None), (100, True, 7, None), (66, False, 0, None)]]
    w = W.custom_workload(specs, n_q_heads=8, n_kv_heads=2, head_dim=64, dtype="f32", rope_base=1e4, seed=5)
    t = W.layer_tensors(w, 0)
    g = GpuLayer(w, t)
    g.realign()
    g.scatter_nonreused()
    req, scale = w.requests[0], O.softmax_scale(64)
    keys = O.gather_tokens(req, w, host(g.k_cache)).astype(np.float64)
    z = np.einsum("ihd,jhd->hij", t["q"].astype(np.float64), np.repeat(keys, 4, 1)) * scale
    z[:, np.triu(np.ones(z.shape[1:], bool), 1)] = -np.inf
    lse = np.logaddexp.reduce(z, 2)
    probes = O.probe_positions(req.n_tokens, req.segments)
    for shift in (0.0, 90.0, 95.0, -200.0):
        caller = (lse + shift).T.astype(np.float32)
        sx.sparseq_score(g.plan, g.t["q"], g.k_cache, g.scores, lse_in=torch.from_numpy(np.ascontiguousarray(caller)).cuda())
        got = host(g.scores).astype(np.float64)
        p = np.exp(z[:, probes] - caller.T.astype(np.float64)[:, probes, None])
        ref = p.sum((0, 1))
        if shift < 0:
            assert np.isposinf(got).all()
        else:
            assert (np.abs(got - ref) <= 1e-4 * ref + p.shape[0] * p.shape[1] * 2.0 ** -150).all(), shift


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("hq,hkv", [(1, 1), (32, 32)], ids=["narrow", "wide"])
def test_attention_of_subnormal_probabilities(hq, hkv, d):
    """A key whose probability is far below the normal range counts when its value is large.  Tolerance: half a
    unit (2^-150) of a probability of e^-90, 2^-129, is 2^-21 of it; the score's rounding (90 x 2^-23) twice that
    and more: 1e-4."""
    log(f"[f32 tiles] subnormal probabilities {hq}/{hkv}/{d}")
    T = 8 if hq == 1 else 300
    q, k, v = (np.zeros((T, h, d), np.float32) for h in (hq, hkv, hkv))
    q[:, :, 0] = np.sqrt(d)
    k[0, :, 0] = -90.0
    v[0] = 1e35
    out, _ = _full(sx.make_desc(hq, hkv, d, "f32", 1e4), q, k, v, (T,))
    ref = 1e35 * np.exp(-90.0) / np.arange(1, T)
    assert (np.abs(out[1:] / ref[:, None, None] - 1) <= 1e-4).all()
