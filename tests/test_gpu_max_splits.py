"""Key splits of the streaming reduction with reduce = max: no bit of a score depends on them.  Every item of a batch, scored
on supplied normalisers, against the same item alone, whose few heads are cut into other splits, at the sizes where a form's
workgroups reach one, two or three a CU and one or several rounds; with reduce = max and the library's own normalisers the
scores are also held to the definition in fp64."""
import pytest
import torch

from paper_2509_17396_amd import binding as ep

pytestmark = pytest.mark.gpu
DEV = "cuda"

SIZES = [  # items, KV heads, rows per head as (group, patch), d, N, dtype
    (1, 1, (1, 1), 64, 1, torch.bfloat16), (32, 8, (1, 32), 64, 1100, torch.bfloat16), (130, 8, (1, 20), 128, 130, torch.bfloat16),
    (8, 8, (1, 64), 32, 2111, torch.bfloat16), (64, 8, (2, 32), 64, 641, torch.bfloat16), (65, 8, (1, 64), 128, 321, torch.bfloat16),
    (3, 32, (1, 96), 96, 1000, torch.bfloat16), (24, 32, (1, 128), 64, 200, torch.bfloat16), (28, 32, (2, 64), 128, 257, torch.bfloat16),
    (8, 8, (3, 64), 64, 2100, torch.bfloat16), (66, 8, (3, 64), 128, 2050, torch.bfloat16), (12, 8, (4, 50), 64, 1000, torch.bfloat16),
    (12, 8, (4, 64), 128, 1000, torch.bfloat16), (4, 8, (2, 64), 256, 700, torch.bfloat16), (80, 8, (1, 64), 200, 129, torch.bfloat16),
    (16, 8, (2, 64), 64, 500, torch.float32), (40, 8, (1, 30), 128, 190, torch.float32)]


@pytest.mark.parametrize("nb,hkv,rows,d,n,dtype", SIZES)
def test_scores_of_an_item_do_not_depend_on_the_batch(nb, hkv, rows, d, n, dtype):
    print(f"[gpu test] max_splits {nb}x{hkv} rows={rows} d={d} N={n} {dtype}", flush=True)
    g, p = rows
    gen = torch.Generator(device=DEV).manual_seed(n + d)
    q = torch.randn(nb, hkv * g, p, d, device=DEV, generator=gen).to(dtype)
    k = torch.randn(nb, hkv, n, d, device=DEV, generator=gen).to(dtype)
    lse = torch.rand(nb, hkv * g, p, device=DEV, generator=gen) + 5.0

    def scored(b0, b1, with_lse):
        prm = ep.make_params(q[b0:b1], k[b0:b1], n_cached=0, n_block=n, budget=max(1, n // 2), reduce=ep.REDUCE_MAX)
        s = torch.full((b1 - b0, hkv, n), -1.0, device=DEV)
        ws = ep.alloc_workspace(prm)
        if with_lse:
            ep.epicache_score_lse(prm, q[b0:b1], k[b0:b1], lse[b0:b1].contiguous(), s, ws)
        else:
            ep.epicache_score(prm, q[b0:b1], k[b0:b1], s, ws)
        return s

    whole = scored(0, nb, True)
    for b in sorted({0, nb // 2, nb - 1}):
        assert torch.equal(whole[b:b + 1].view(torch.int32), scored(b, b + 1, True).view(torch.int32))
    own = scored(0, nb, False)
    b = nb - 1
    z = torch.matmul(q[b].double().view(hkv, g * p, d), k[b].double().transpose(1, 2).contiguous()) * d ** -0.5
    want = torch.softmax(z, dim=-1).amax(dim=1)
    # fp32 logits of about sqrt(d) * 2^-24 error each, weights relative to it; bf16 inputs are exact in both
    assert torch.allclose(own[b].double(), want, rtol=1e-5, atol=1e-30)
