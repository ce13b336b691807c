"""Layer-body products on every tile shape, at the edges of rows, k pieces and k groups (GPU).

Against float64 on the CPU.  Tolerance: the result is a float32 sum of K bf16 products, off by at most
K 2^-24 sum |x w| (with the residual), rounded once to bf16 (8 significant bits: half a unit in the last
place is at most 2^-8 of the value).
"""
import numpy as np
import pytest
import torch

import workloads as W
from sxgpu import desc_of, log

pytestmark = pytest.mark.gpu

try:
    import paper_2606_01751_amd as sx
except Exception:  # pragma: no cover
    sx = None

# (rows per request, features, k): the five shapes (256 x 256, 256 x 128, 128 x 128, 128 x 64, 64 x 64
# features x rows) with whole tiles, one row more and one less, and k from one 64-wide piece up to
# counts that leave the stage buffers or a k group partly filled
CASES = [
    ((385,), 28672, 64), ((400,), 28672, 320),
    ((128,), 28672, 64), ((129,), 28672, 256), ((255,), 28672, 192),
    ((384,), 6144, 64), ((383,), 6144, 128), ((300,), 6144, 320), ((257,), 6144, 448),
    ((384,), 4096, 64), ((321,), 4096, 128), ((384,), 4096, 192), ((350,), 4096, 576),
    ((1,), 256, 64), ((64,), 4096, 192), ((65,), 4096, 256), ((255,), 4096, 320), ((7, 63, 130), 512, 704),
]


@pytest.mark.parametrize("lengths,n,k", CASES, ids=["x".join(map(str, c[0])) + f"-{c[1]}-{c[2]}" for c in CASES])
def test_gemm_rows_shapes(lengths, n, k):
    log(f"[gemm tiles] rows {lengths} n {n} k {k}")
    w = W.custom_workload([[(t + 5, False, 0, None)] for t in lengths], n_q_heads=8, n_kv_heads=2, head_dim=128, dtype="bf16",
                          rope_base=1e4)
    plan = sx.Plan(desc_of(w), w.requests, w.n_dst_blocks, w.n_src_blocks)
    total = w.total_tokens
    gen = torch.Generator().manual_seed(n + k + sum(lengths))
    x = torch.randn((total, k), generator=gen).bfloat16()
    wt = (torch.randn((n, k), generator=gen) / k ** 0.5).bfloat16()
    res = torch.randn((total, n), generator=gen).bfloat16()
    rows, n_rows, tok, slot = torch.zeros(total, dtype=torch.int32), [], [], []
    for off, t in zip(w.token_offsets, lengths):     # rows 0 .. and a gap of five tokens inside
        r = torch.cat([torch.arange(t // 2), torch.arange(t // 2 + 5, t + 5)])
        rows[off:off + t] = r
        n_rows.append(t)
        tok += (off + r).tolist()
        slot += range(off, off + t)
    dev = [v.cuda() for v in (rows, torch.tensor(n_rows, dtype=torch.int32), x, wt, res)]
    y = torch.full((total, n), 7.0, dtype=torch.bfloat16, device="cuda")
    sx.gemm_rows(plan, dev[0], dev[1], max(lengths), dev[2], dev[3], y, residual=dev[4], x_by_token=True, y_by_token=False)
    torch.cuda.synchronize()
    got = y.cpu()
    a, b = x[tok].double(), wt.double()
    ref = a @ b.T + res[slot].double()
    bound = (k * 2.0 ** -24) * (a.abs() @ b.abs().T + res[slot].double().abs()) + 2.0 ** -8 * ref.abs() * 1.01 + 1e-30
    assert ((got[slot].double() - ref).abs() <= bound).all()
    rest = np.setdiff1d(np.arange(total), slot)
    assert (got[rest] == 7.0).all()
    # stacked parts, token addressed
    parts = [torch.zeros((total, n // 2), dtype=torch.bfloat16, device="cuda") for _ in range(2)] if n % 512 == 0 else \
        [torch.zeros((total, n), dtype=torch.bfloat16, device="cuda")]
    sx.gemm_rows_split(plan, dev[0], dev[1], max(lengths), dev[2], dev[3], parts, x_by_token=True, y_by_token=True)
    torch.cuda.synchronize()
    both = torch.cat([p.cpu() for p in parts], 1)[tok].double()
    ref = a @ b.T
    bound = (k * 2.0 ** -24) * (a.abs() @ b.abs().T) + 2.0 ** -8 * ref.abs() * 1.01 + 1e-30
    assert ((both - ref).abs() <= bound).all()
    plan.close()
