"""Scores of few heads: workgroups of a head on all XCDs, and query rows shared out to groups of waves, at the edges of key blocks
and row tiles, against float64."""
import ctypes
import os

import pytest
import torch

from paper_2509_17396_amd import binding as ep
from paper_2509_17396_amd import build
from tests import parity_util as pu

pytestmark = pytest.mark.gpu
DEV = "cuda"


def form(dtype, heads, rows, n, d):
    """Whether workgroups go to all XCDs, and the groups of waves in the key-stationary pass 2 (0: it streams the keys)."""
    so = os.path.join(os.path.dirname(build.LIB), "selftest", "liblaunch_rules.so")
    if not os.path.exists(so):
        build.build_selftests()
    groups = ctypes.c_int(0)
    spread = ctypes.CDLL(so).score_form(ep.DTYPE_F32 if dtype == torch.float32 else ep.DTYPE_BF16, heads, rows, n, d,
                                        ctypes.byref(groups))
    return spread, groups.value


def inputs(nb, heads, group, p, n, d, dtype=torch.bfloat16):
    g = torch.Generator(device=DEV).manual_seed(n + p)
    q = (1.5 * torch.randn(nb, heads * group, p, d, device=DEV, generator=g)).to(dtype)
    return q, torch.randn(nb, heads, n, d, device=DEV, generator=g).to(dtype)


def reference(q, k, b, h, n, reduce, causal=0):
    """Scores of head (b, h) over its first n keys, and the normalisers of its rows; causal: the patch's keys follow those."""
    group, p, d = q.shape[1] // k.shape[1], q.shape[2], q.shape[3]
    rows = q[b, h * group:(h + 1) * group].reshape(-1, d).double()
    z = rows @ k[b, h, :n + causal * p].double().T.contiguous() / d ** 0.5
    if causal:
        late = torch.arange(p, device=DEV)[None] > torch.arange(p, device=DEV)[:, None]
        z[:, n:] = z[:, n:].masked_fill(late.repeat(group, 1), -float("inf"))
    w = torch.softmax(z, dim=1)[:, :n]
    return w.max(dim=0).values if reduce == ep.REDUCE_MAX else w.sum(dim=0), torch.logsumexp(z, dim=1).reshape(group, p).float()


# batch, KV heads, group, patch, keys, head_dim: rows above 256 in 4, 2 or 1 groups, tiles that are no multiple of them, patches that do
# and do not fill tiles; heads that are no multiple of 8, on one XCD and on all.  Behind each whether on all, and the groups.
SHAPES = [((1, 1, 1, 257, 1, 128), (0, 4)), ((1, 1, 5, 64, 63, 128), (0, 4)), ((1, 2, 5, 64, 65, 64), (0, 4)), ((1, 1, 7, 64, 700, 128), (0, 4)),
          ((1, 4, 7, 256, 769, 128), (0, 4)), ((1, 2, 3, 100, 1999, 64), (0, 4)), ((1, 2, 3, 100, 2000, 64), (1, 4)),
          ((1, 1, 3, 128, 8192, 128), (1, 4)), ((1, 1, 3, 128, 8193, 128), (1, 4)), ((1, 1, 3, 128, 16384, 128), (1, 4)), ((1, 1, 3, 128, 16385, 128), (1, 2)), ((1, 1, 3, 100, 33000, 128), (1, 1)),
          ((1, 3, 4, 128, 5000, 128), (1, 4)), ((3, 4, 4, 129, 2500, 64), (1, 2)), ((1, 8, 7, 64, 1025, 128), (0, 4)),
          ((1, 8, 4, 75, 4000, 128), (0, 2)), ((1, 8, 4, 128, 8500, 64), (0, 1)), ((1, 12, 3, 64, 4001, 128), (1, 0)),
          ((2, 5, 2, 20, 25000, 64), (1, 0)), ((1, 6, 1, 200, 300, 128), (0, 0)), ((3, 4, 8, 40, 2111, 96), (1, 1)),
          ((1, 3, 3, 64, 2100, 256), (1, 1))]


@pytest.mark.parametrize("reduce", [ep.REDUCE_MAX, ep.REDUCE_SUM], ids=["max", "sum"])
@pytest.mark.parametrize("shape,taken", SHAPES, ids=["-".join(map(str, s)) for s, _ in SHAPES])
def test_scores_of_few_heads(shape, taken, reduce):
    nb, heads, group, p, n, d = shape
    print(f"[gpu test] scores of few heads {shape} reduce={reduce}", flush=True)
    assert form(torch.bfloat16, nb * heads, group * p, n, d) == taken
    q, k = inputs(*shape)
    prm = ep.make_params(q, k, n_cached=n, n_block=0, budget=1, reduce=reduce)
    scores = torch.full((nb, heads, n), float("nan"), device=DEV)
    ws = torch.full((ep.epicache_workspace_size(prm),), 0xff, dtype=torch.uint8, device=DEV)
    ep.epicache_score(prm, q, k, scores, ws)
    lse = torch.empty(nb, heads * group, p, device=DEV)
    want = torch.empty(nb, heads, n, dtype=torch.float64, device=DEV)
    for b in range(nb):
        for h in range(heads):
            want[b, h], lse[b, h * group:(h + 1) * group] = reference(q, k, b, h, n, reduce)
    pu.assert_scores_close(scores.cpu().numpy(), want.cpu().numpy(), 1e-4, f"{shape}")
    again = torch.full_like(scores, float("nan"))
    ep.epicache_score(prm, q, k, again, ws)
    assert torch.equal(again, scores)
    ep.epicache_score_lse(prm, q, k, lse, again, ws)  # pass 2 alone
    pu.assert_scores_close(again.cpu().numpy(), want.cpu().numpy(), 1e-4, f"{shape} lse")


# the same on all XCDs for rows of other layouts and for pass 1 with the patch's own keys: group, patch, keys, head_dim, dtype, groups
SPREAD = [(4, 100, 2500, 128, torch.bfloat16, 4), (4, 100, 2500, 96, torch.bfloat16, 1), (4, 100, 2500, 64, torch.float32, 1),
          (3, 50, 2300, 128, torch.float32, 1)]


@pytest.mark.parametrize("reduce", [ep.REDUCE_MAX, ep.REDUCE_SUM], ids=["max", "sum"])
@pytest.mark.parametrize("causal", [0, 1], ids=["context_only", "causal_patch"])
@pytest.mark.parametrize("shape", SPREAD, ids=["-".join(map(str, s)) for s in SPREAD])
def test_scores_on_all_xcds(shape, causal, reduce):
    group, p, n, d, dtype, groups = shape
    heads = 3
    print(f"[gpu test] scores on all XCDs {shape} causal={causal} reduce={reduce}", flush=True)
    assert form(dtype, heads, group * p, n, d) == (1, groups)
    q, k = inputs(1, heads, group, p, n + causal * p, d, dtype)
    prm = ep.make_params(q, k, n_cached=n, n_block=0, budget=1, reduce=reduce, causal_patch=causal)
    scores = torch.full((1, heads, n), float("nan"), device=DEV)
    ws = torch.full((ep.epicache_workspace_size(prm),), 0xff, dtype=torch.uint8, device=DEV)
    ep.epicache_score(prm, q, k, scores, ws)
    want = torch.stack([reference(q, k, 0, h, n, reduce, causal)[0] for h in range(heads)])[None]
    pu.assert_scores_close(scores.cpu().numpy(), want.cpu().numpy(), 1e-4, f"{shape} causal={causal}")


@pytest.mark.parametrize("reduce", [ep.REDUCE_MAX, ep.REDUCE_SUM], ids=["max", "sum"])
@pytest.mark.parametrize("with_lse", [False, True], ids=["two_passes", "pass_2"])
@pytest.mark.parametrize("heads,group,p", [(3, 4, 100), (6, 3, 128), (12, 3, 64)], ids=["rows_400", "rows_384", "stream"])
def test_ragged_scores_on_all_xcds(heads, group, p, with_lse, reduce):
    """Heads without keys, with one, a tile and one, and all of them: splits and key blocks that hold nothing of a head."""
    nb, n, d = 1, 4001, 128
    print(f"[gpu test] ragged scores on all XCDs heads={heads} rows={group * p} lse={with_lse} reduce={reduce}", flush=True)
    assert form(torch.bfloat16, heads, group * p, n, d) == (1, 0 if group * p <= 256 else 4 if heads == 3 else 2)
    q, k = inputs(nb, heads, group, p, n, d)
    lengths = ([n, 0, 65] + [1, 2047, 3000, 64, 0, 2048, 777, n - 1, 128])[:heads]
    n_ctx = torch.tensor([lengths], dtype=torch.int32, device=DEV)
    prm = ep.make_params(q, k, n_cached=n, n_block=0, budget=1, reduce=reduce)
    scores = torch.full((nb, heads, n), -7.0, device=DEV)
    ws = torch.full((ep.epicache_workspace_size(prm),), 0xff, dtype=torch.uint8, device=DEV)
    lse, want = torch.zeros(nb, heads * group, p, device=DEV), {}
    for h in range(heads):
        if lengths[h]:
            want[h], lse[0, h * group:(h + 1) * group] = reference(q, k, 0, h, lengths[h], reduce)
    ep.epicache_score_ragged(prm, q, k, n_ctx, scores, ws, row_lse=lse if with_lse else None)
    for h in range(heads):
        assert bool((scores[0, h, lengths[h]:] == -7.0).all())
        if lengths[h]:
            pu.assert_scores_close(scores[0, h, :lengths[h]].cpu().numpy(), want[h].cpu().numpy(), 1e-4, f"head {h}")
