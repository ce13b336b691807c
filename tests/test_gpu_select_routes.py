"""Selection, and row masks on both sides of their one-launch limit (GPU), exact against the oracle.

A row list of up to 16384 rows is masked in one launch, by workgroups of 8192 tokens, bfloat16 plans with the tile
order in the same; a longer one in a clearing and a marking launch, and the order in a third.
"""
import types

import numpy as np
import pytest
import torch

import oracle as O
from sxgpu import log

pytestmark = pytest.mark.gpu

try:
    import paper_2606_01751_amd as sx
except Exception:  # pragma: no cover
    sx = None


def _request(pieces, dst0, src0):
    segs, t, used = [], 0, 0
    for n, cached in pieces:
        segs.append(types.SimpleNamespace(seq_start=t, length=n, cached=int(cached), old_pos=0, new_pos=t,
                                          src_block_start=used if cached else -1))
        used += -(-n // 16) if cached else 0
        t += n
    nb = -(-t // 16)
    return types.SimpleNamespace(n_tokens=t, segments=segs, block_table=np.arange(dst0, dst0 + nb, dtype=np.int32),
                                 src_block_ids=np.arange(src0, src0 + used, dtype=np.int32)), nb, used


def _plan(requests, dtype="bf16", all_positions=False):
    reqs, a, b = [], 0, 0
    for p in requests:
        r, nb, used = _request(p, a, b)
        reqs.append(r)
        a, b = a + nb, b + used
    desc = sx.make_desc(8, 2, 64, dtype, 1e4, topk_all_positions=all_positions)
    return reqs, sx.Plan(desc, reqs, a, max(b, 1))


SCORES = {
    "lognormal": lambda rng, n: rng.lognormal(0, 1, n),
    "ties": lambda rng, n: rng.integers(0, 4, n).astype(np.float32),
    "equal": lambda rng, n: np.full(n, 0.25),
    "signed": lambda rng, n: rng.normal(0, 1, n) * 10.0 ** rng.integers(-30, 30, n),
    "near": lambda rng, n: (np.float32(1.5).view(np.uint32) + rng.integers(0, 300, n).astype(np.uint32)).view(np.float32),
}
# request lengths at the edges of a thread's 8 tokens, a 2048-token chunk, the one-workgroup selection's rounds of
# 8192 tokens and its limit of two, and a mask workgroup's 8192 tokens
LENGTHS = [(1, 7, 8, 9), (2047, 2049), (8192, 777), (8191, 8193, 16384), (16385, 9), (32768,), (32767, 5), (32769, 100)]


@pytest.mark.parametrize("kind", SCORES)
@pytest.mark.parametrize("lengths", LENGTHS, ids=lambda x: "-".join(map(str, x)))
def test_selection_is_exact(lengths, kind):
    log(f"[select routes] {lengths} {kind}")
    rng = np.random.default_rng(sum(lengths) + len(kind))
    pieces = []
    for n in lengths:
        a = max(1, n // 9)
        pieces.append([(n, True)] if n < 8 else [(a, False), (n - 2 * a, True), (a, n % 2 == 0)])
    for all_pos in (False, True):
        reqs, plan = _plan(pieces, all_positions=all_pos)
        total = sum(lengths)
        offs = np.concatenate([[0], np.cumsum(lengths)])
        host_s = SCORES[kind](rng, total).astype(np.float32)
        scores = torch.from_numpy(host_s).cuda()
        for ratio in (0.0, 0.05, 0.37, 1.0):
            rows = torch.full((total,), -5, dtype=torch.int32, device="cuda")
            n_rows = torch.zeros(len(lengths), dtype=torch.int32, device="cuda")
            mask = torch.full((total + 3,), 9, dtype=torch.uint8, device="cuda")
            sx.topk_select(plan, scores, ratio, rows, n_rows)
            sx.rows_mask(plan, rows, n_rows, plan.budget(ratio)[1], mask[:total])
            torch.cuda.synchronize()
            got, cnt, m = rows.cpu().numpy(), n_rows.cpu().numpy(), mask.cpu().numpy()
            want = np.zeros(total, np.uint8)
            for r, (req, off) in enumerate(zip(reqs, offs)):
                n = req.n_tokens
                cand = O.reuse_positions(n, req.segments) if not all_pos else np.arange(n)
                key = O.topk_keys(host_s[off:off + n].astype(np.float64), cand, O.budget(len(cand), ratio))
                base = np.concatenate([O.nonreuse_positions(n, req.segments), O.overflow_positions(n, req.segments, 16),
                                       O.tail_fallback(n, req.segments)])
                R = np.unique(np.concatenate([key, base]).astype(np.int64))
                assert cnt[r] == len(R), (r, ratio, all_pos)
                assert np.array_equal(got[off:off + len(R)], R), (r, ratio, all_pos)
                assert (got[off + len(R):off + n] == -5).all()
                want[off + R] = 1
            assert np.array_equal(m[:total], want) and (m[total:] == 9).all()
        plan.close()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n", [16384, 16385])
def test_row_masks(n, dtype):
    """Lists at the one-launch limit, cut by max_rows, with values outside the request ignored."""
    log(f"[select routes] mask {n} {dtype}")
    total = 70001
    reqs, plan = _plan([[(total, False)], [(33, False)]], dtype)
    lists = [np.arange(total - n, total, dtype=np.int32), np.array([-3, 0, 5, 32, 33, 40], np.int32)]
    rows = torch.zeros(total + 33, dtype=torch.int32)
    rows[:n] = torch.from_numpy(lists[0])
    rows[total:total + 6] = torch.from_numpy(lists[1])
    n_rows = torch.tensor([n, 6], dtype=torch.int32, device="cuda")
    mask = torch.full((total + 33,), 9, dtype=torch.uint8, device="cuda")
    dev = rows.cuda()
    for most in (n, 3, 0):
        sx.rows_mask(plan, dev, n_rows, most, mask)
        torch.cuda.synchronize()
        want = np.zeros(total + 33, np.uint8)
        want[lists[0][:most]] = 1
        keep = lists[1][:most]
        want[total + keep[(keep >= 0) & (keep < 33)]] = 1
        assert np.array_equal(mask.cpu().numpy(), want), most
    plan.close()
