"""Scores with one product per logit: tiles per wave and their remainders, blocks of 32 rows and theirs, the parts of several
workgroups merged in the selection or by a launch of their own, and rows that are done again relative to their largest logit."""
import ctypes
import os

import pytest
import torch

from paper_2509_17396_amd import binding as ep
from paper_2509_17396_amd import build
from tests import parity_util as pu
from tests.test_gpu_score_few_heads import inputs, reference

pytestmark = pytest.mark.gpu
DEV = "cuda"
BF16, F32 = torch.bfloat16, torch.float32


def splits(dtype, d, heads, rows, patch, n, causal, room):
    so = os.path.join(os.path.dirname(build.LIB), "selftest", "liblaunch_rules.so")
    if not os.path.exists(so):
        build.build_selftests()
    return ctypes.CDLL(so).row_splits(ep.DTYPE_F32 if dtype == F32 else ep.DTYPE_BF16, d, heads, rows, patch, n, causal, 0,
                                      ctypes.c_longlong(room))


# dtype, head_dim, batch, KV heads, group, patch, keys, whether causal, whether the workspace has room for parts.  Keys: one tile, tiles
# of a wave from 2 to 8 with one key more or less, odd numbers of tiles through several blocks of rows (the two buffers change places).
# Heads: no multiple of 8.  Without room one workgroup takes all blocks.
CASES = [(BF16, 128, 1, 1, 1, 1, 1, 0, 1), (BF16, 128, 1, 3, 1, 32, 33, 0, 1), (BF16, 128, 2, 3, 1, 33, 512, 0, 1),
         (BF16, 128, 1, 5, 3, 20, 513, 0, 1), (BF16, 128, 1, 4, 4, 64, 480, 1, 1), (BF16, 128, 9, 5, 1, 50, 767, 1, 1),
         (BF16, 128, 40, 5, 2, 32, 1025, 0, 1), (BF16, 128, 8, 5, 2, 50, 1535, 0, 1), (BF16, 128, 33, 4, 3, 33, 1999, 1, 1),
         (BF16, 128, 16, 2, 4, 64, 2048, 0, 1), (BF16, 128, 16, 8, 2, 30, 1300, 0, 0), (BF16, 128, 16, 8, 2, 32, 1600, 0, 0),
         (BF16, 64, 1, 2, 7, 32, 255, 0, 1), (BF16, 64, 2, 3, 4, 16, 641, 1, 1), (BF16, 64, 3, 7, 2, 40, 1281, 0, 1),
         (BF16, 64, 5, 4, 7, 9, 1793, 0, 1), (BF16, 64, 16, 8, 2, 32, 700, 0, 0), (BF16, 64, 16, 8, 2, 32, 2048, 0, 0),
         (BF16, 96, 4, 8, 1, 64, 2024, 0, 1), (BF16, 72, 2, 3, 1, 20, 300, 0, 1), (BF16, 80, 2, 2, 8, 20, 511, 1, 1),
         (BF16, 88, 16, 8, 2, 32, 1100, 0, 0), (F32, 64, 1, 2, 4, 32, 384, 0, 1), (F32, 64, 16, 2, 7, 33, 900, 1, 1),
         (F32, 64, 32, 4, 2, 32, 1400, 0, 0), (F32, 64, 13, 10, 1, 31, 2047, 0, 1)]


@pytest.mark.parametrize("reduce", [ep.REDUCE_MAX, ep.REDUCE_SUM], ids=["max", "sum"])
@pytest.mark.parametrize("case", CASES, ids=["-".join(map(str, ("f32" if c[0] == F32 else "bf16",) + c[1:])) for c in CASES])
def test_scores_and_steps(case, reduce):
    """Scores against float64: logits below 16 in base 2, whose 32 partial sums are rounded to 2^-21 at most, 1e-5 of a weight.  The steps
    with and without the caller's score buffer select from the same sums of parts, and move the same rows."""
    dtype, d, nb, heads, group, p, n, causal, room = case
    print(f"[gpu test] score rows {case} reduce={reduce}", flush=True)
    q, k = inputs(nb, heads, group, p, n + causal * p, d, dtype)
    v = torch.randn_like(k.float()).to(dtype)
    m = max(1, n * 3 // 5)
    prm = ep.make_params(q, k, n_cached=min(m, n), n_block=n - min(m, n), budget=m, reduce=reduce, causal_patch=causal)
    blocks = (group * p + 31) // 32
    ws = torch.zeros(ep.epicache_workspace_size(prm) + room * blocks * nb * heads * n * 4, dtype=torch.uint8, device=DEV)
    assert splits(dtype, d, nb * heads, group * p, p, n, causal, 1 << 40 if room else 0) == (blocks if room else 1)
    scores = torch.full((nb, heads, n), -1.0, device=DEV)
    ep.epicache_score(prm, q, k, scores, ws)
    for b, h in {(0, 0), (nb - 1, heads - 1), (nb // 2, heads // 2)}:
        want = reference(q, k, b, h, n, reduce, causal)[0]
        pu.assert_scores_close(scores[b, h].cpu().numpy(), want.cpu().numpy(), 1e-5, f"{case} b={b} h={h}")
    if n == m:
        return
    results = []
    for with_scores in (True, False):
        k2, v2 = k.clone(), v.clone()
        keep = torch.full((nb, heads, m), -1, dtype=torch.int32, device=DEV)
        again = torch.full_like(scores, -1.0) if with_scores else None
        ep.epicache_evict_step(prm, q, k2, v2, ws, scores=again, keep_idx=keep)
        if with_scores:
            assert torch.equal(again, scores)
        assert torch.equal(keep, torch.sort(torch.sort(scores, dim=-1, descending=True, stable=True)[1][..., :m], dim=-1)[0].int())
        index = keep.long()[..., None].expand(-1, -1, -1, d)
        assert torch.equal(k2[:, :, :m], torch.gather(k, 2, index)) and torch.equal(v2[:, :, :m], torch.gather(v, 2, index))
        results.append(keep)
    assert torch.equal(*results)


@pytest.mark.parametrize("reduce", [ep.REDUCE_MAX, ep.REDUCE_SUM], ids=["max", "sum"])
@pytest.mark.parametrize("dtype,d,n", [(BF16, 128, 500), (BF16, 64, 1100), (BF16, 96, 300), (F32, 64, 700)])
def test_rows_far_from_one(dtype, d, n, reduce):
    """Rows whose weights relative to 1 overflow, vanish or keep a few keys only, in one block with ordinary ones and in blocks of
    their own; keys that no row sees, or one row only."""
    print(f"[gpu test] score rows, far from one {dtype} d={d} N={n} reduce={reduce}", flush=True)
    q, k = inputs(2, 40, 2, 32, n, d, dtype)
    k[..., 0] = 8.0
    q[0, :, 3, 0] = 60.0    # all logits of these rows far above 0 ...
    q[0, :, 20:24, 0] = -60.0   # ... or below
    q[1, ::2] *= 40.0           # and all rows of a block far apart
    k[0, 0, 5] = 0.0
    k[0, 0, 5, 0] = float("-inf")
    q[0, :2, :, 0] = q[0, :2, :, 0].abs() + 0.1
    prm = ep.make_params(q, k, n_cached=n // 2, n_block=n - n // 2, budget=n // 2, reduce=reduce)
    ws = torch.zeros(ep.epicache_workspace_size(prm) + 80 * 2 * n * 4, dtype=torch.uint8, device=DEV)
    assert splits(dtype, d, 80, 64, 32, n, 0, 1 << 40) == 2
    scores = torch.empty(2, 40, n, device=DEV)
    ep.epicache_score(prm, q, k, scores, ws)
    for b, h in ((0, 0), (0, 39), (1, 0), (1, 1), (1, 38)):
        rows = q[b, 2 * h:2 * h + 2].reshape(64, d).double()
        keys = k[b, h].double()
        gone = torch.isinf(keys).any(dim=1)
        z = rows @ torch.where(gone[:, None], 0.0, keys).T.contiguous() / d ** 0.5
        w = torch.softmax(z.masked_fill(gone[None], -float("inf")), dim=1)
        want = w.max(dim=0).values if reduce == ep.REDUCE_MAX else w.sum(dim=0)
        # The far rows' logits are below 128 in base 2, and below 1024 in the second item: 32 partial sums (fp32, the longest chain)
        # that are rounded to half of 2^-17, and of 2^-14, make 8.5e-5 and 6.8e-4 of a weight.
        pu.assert_scores_close(scores[b, h].cpu().numpy(), want.cpu().numpy(), 1e-4 if b == 0 else 1e-3, f"b={b} h={h}")
