"""Scores of few heads: workgroups of a head on all XCDs, and query rows shared out to groups of waves, at the edges of key blocks
and row tiles, against float64."""
import pytest
import torch

from paper_2509_17396_amd import binding as ep
from tests import parity_util as pu

pytestmark = pytest.mark.gpu
DEV = "cuda"

# batch, KV heads, group, patch, keys, head_dim: rows above 256 in 4, 2 or 1 groups, tiles that are no multiple of them, patches that do
# and do not fill tiles; heads that are no multiple of 8, on one XCD and on all
SHAPES = [(1, 1, 1, 257, 1, 128), (1, 1, 5, 64, 63, 128), (1, 2, 5, 64, 65, 64), (1, 1, 7, 64, 700, 128), (1, 4, 7, 256, 769, 128),
          (1, 2, 3, 100, 1999, 64), (1, 2, 3, 100, 2000, 64), (1, 1, 3, 128, 8192, 128), (1, 1, 3, 128, 8193, 128), (1, 3, 4, 128, 5000, 128),
          (3, 4, 4, 129, 2500, 64), (1, 8, 7, 64, 1025, 128), (1, 12, 3, 64, 4001, 128), (2, 5, 2, 20, 25000, 64), (1, 6, 1, 200, 300, 128),
          (3, 4, 8, 40, 2111, 96), (1, 3, 3, 64, 2100, 256)]


@pytest.mark.parametrize("reduce", [ep.REDUCE_MAX, ep.REDUCE_SUM], ids=["max", "sum"])
@pytest.mark.parametrize("shape", SHAPES, ids=["-".join(map(str, s)) for s in SHAPES])
def test_scores_of_few_heads(shape, reduce):
    nb, heads, group, p, n, d = shape
    print(f"[gpu test] scores of few heads {shape} reduce={reduce}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(n + p)
    q = (1.5 * torch.randn(nb, heads * group, p, d, device=DEV, generator=g)).bfloat16()
    k = torch.randn(nb, heads, n, d, device=DEV, generator=g).bfloat16()
    prm = ep.make_params(q, k, n_cached=n, n_block=0, budget=1, reduce=reduce)
    scores = torch.full((nb, heads, n), float("nan"), device=DEV)
    ws = torch.full((ep.epicache_workspace_size(prm),), 0xff, dtype=torch.uint8, device=DEV)
    ep.epicache_score(prm, q, k, scores, ws)
    lse = torch.empty(nb, heads * group, p, device=DEV)
    want = torch.empty(nb, heads, n, dtype=torch.float64, device=DEV)
    for b in range(nb):
        for h in range(heads):
            z = q[b, h * group:(h + 1) * group].reshape(-1, d).double() @ k[b, h].double().T.contiguous() / d ** 0.5
            lse[b, h * group:(h + 1) * group] = torch.logsumexp(z, dim=1).reshape(group, p).float()
            w = torch.softmax(z, dim=1)
            want[b, h] = w.max(dim=0).values if reduce == ep.REDUCE_MAX else w.sum(dim=0)
    pu.assert_scores_close(scores.cpu().numpy(), want.cpu().numpy(), 1e-4, f"{shape}")
    again = torch.full_like(scores, float("nan"))
    ep.epicache_score(prm, q, k, again, ws)
    assert torch.equal(again, scores)
    ep.epicache_score_lse(prm, q, k, lse, again, ws)  # pass 2 alone
    pu.assert_scores_close(again.cpu().numpy(), want.cpu().numpy(), 1e-4, f"{shape} lse")
