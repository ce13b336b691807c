"""RMSNorm and RoPE of listed rows at the edges of their workgroups (GPU).

Against the oracle in float64.  RMSNorm: formed in float64, rounded to float32 and from there to bf16, so off by
half a bf16 unit of the value's binade and half a float32 unit (2^-24 of it); a sum in float32 would be off by more
wherever a value lies near a boundary.  RoPE: two products of magnitude |x| with cos / sin rounded to float32,
rounded to bf16.
"""
import numpy as np
import pytest
import torch

import oracle as O
import workloads as W
from sxgpu import desc_of, host, log

pytestmark = pytest.mark.gpu

try:
    import paper_2606_01751_amd as sx
except Exception:  # pragma: no cover
    sx = None


def _plan(lengths, d, style="neox"):
    w = W.custom_workload([[(t, False, 0, 11)] for t in lengths], n_q_heads=6, n_kv_heads=2, head_dim=d, dtype="bf16",
                          rope_base=1e4, rope_style=style)
    return w, sx.Plan(desc_of(w), w.requests, w.n_dst_blocks, w.n_src_blocks)


def _rows(w, counts):
    """The last counts[r] tokens of each request as its row list."""
    rows = torch.zeros(w.total_tokens, dtype=torch.int32)
    tok, slot = [], []
    for req, off, n in zip(w.requests, w.token_offsets, counts):
        r = np.arange(req.n_tokens - n, req.n_tokens)
        rows[off:off + n] = torch.from_numpy(r.astype(np.int32))
        tok += (off + r).tolist()
        slot += range(off, off + n)
    return rows.cuda(), torch.tensor(counts, dtype=torch.int32, device="cuda"), np.array(tok, int), np.array(slot, int)


# one piece per thread (2048), two (4096), one element past each, several pieces read twice, the smallest row
@pytest.mark.parametrize("h", [8, 2040, 2048, 2056, 4096, 4104, 10248])
def test_rmsnorm_row_lengths(h):
    log(f"[layer rows] rmsnorm {h}")
    w, plan = _plan((5, 9), 64)
    rows, n_rows, tok, slot = _rows(w, [1, 7])
    gen = torch.Generator().manual_seed(h)
    x = torch.randn((14, h), generator=gen).bfloat16()
    gamma = (1 + 0.1 * torch.randn(h, generator=gen)).bfloat16()
    y = torch.full((14, h), 7.0, dtype=torch.bfloat16, device="cuda")
    sx.rmsnorm_rows(plan, rows, n_rows, 7, x.cuda(), gamma.cuda(), 1e-5, y, x_by_token=True)
    torch.cuda.synchronize()
    ref = O.rmsnorm(x[tok].double().numpy(), gamma.double().numpy(), 1e-5)
    got = host(y).astype(np.float64)
    half = 2.0 ** (np.floor(np.log2(np.abs(ref) + 1e-300)) - 8)      # half a unit of bf16
    assert (np.abs(got[slot] - ref) <= half + 1.001 * 2.0 ** -24 * np.abs(ref)).all()
    assert (got[np.setdiff1d(np.arange(14), slot)] == 7.0).all()
    plan.close()


# 4 (d = 128) or 8 (d = 64) tokens per workgroup: one token, one short, whole, one more
@pytest.mark.parametrize("style", ["neox", "gptj"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("counts", [[1, 0], [3, 4], [7, 5], [8, 9]], ids=str)
def test_rope_row_counts(counts, d, style):
    log(f"[layer rows] rope {counts} {d} {style}")
    w, plan = _plan((9, 12), d, style)
    rows, n_rows, tok, _ = _rows(w, counts)
    gen = torch.Generator().manual_seed(d)
    q, k = (torch.randn((21, n, d), generator=gen).bfloat16() for n in (6, 2))
    dq, dk = q.cuda(), k.cuda()
    sx.rope_rows(plan, rows, n_rows, max(counts), dq, dk)
    torch.cuda.synchronize()
    pos = np.concatenate([np.arange(r.n_tokens) + 11 for r in w.requests])
    for x, y in ((q, dq), (k, dk)):
        ref = x.double().numpy().copy()
        ref[tok] = O.rope_at_positions(x[tok].float().numpy(), pos[tok], 1e4, style)
        size = np.abs(x.double().numpy()).max()
        assert (np.abs(host(y) - ref) <= 2.0 ** -8 * np.abs(ref) + 4 * 2.0 ** -24 * size).all()
        rest = np.setdiff1d(np.arange(21), tok)
        assert np.array_equal(host(y)[rest], x[rest].float().numpy())
    plan.close()
