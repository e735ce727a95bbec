"""epicache_evict_step_static near the size of its array: whatever fits with one key split is taken, however many splits
the step would like, and nothing larger is."""
import ctypes
import random

import pytest
import torch

from paper_2509_17396_amd import binding as ep

FITS_WITH_FEWER_SPLITS = [  # items, KV heads, query heads per KV head, patch, head_dim, N, M
    (224, 8, 7, 64, 64, 4173, 2791), (282, 8, 7, 64, 8, 2762, 2123), (137, 8, 7, 128, 8, 5442, 5072),
    (238, 2, 7, 128, 8, 13445, 12908)]


def params(nb, hkv, g, p, d, n, m, dtype=ep.DTYPE_BF16):
    hq = hkv * g
    return ep.Params(ctypes.sizeof(ep.Params), nb, hq, hkv, d, m, n - m, m, p, dtype, ep.REDUCE_SUM, 0.0, 0, 0,
                     hq * p * d, p * d, d, hkv * n * d, n * d, d)


def smallest_workspace(nb, hkv, g, p, n, m, scores, keep):
    """With one key split: a (reference, sum) pair and a normaliser per scoring row, scores, kept indices, normalisers."""
    def up(x):
        return (x + 255) // 256 * 256
    rows = (g * p + 63) // 64 * 64
    size = up(nb * hkv * rows * 12)
    if not (scores and keep):
        size += up(nb * hkv * n * 4)
    if not keep:
        size += up(nb * hkv * min(m, n) * 4) + up(nb * hkv * g * p * 4)
    return size


def refused(prm, scores, keep):
    """Only where there is no device to launch on: the call gets as far as looking for one."""
    a = ctypes.c_void_p(4096)
    st = ep.load().epicache_evict_step_static(ctypes.byref(prm), a, a, ctypes.c_void_p(8192), a if scores else None,
                                              a if keep else None, None)
    assert st in (ep.ERR_WORKSPACE_TOO_SMALL, ep.ERR_DEVICE)
    return st == ep.ERR_WORKSPACE_TOO_SMALL


@pytest.mark.skipif(torch.cuda.is_available(), reason="the pointers are not real")
def test_what_fits_with_one_split_is_taken_and_nothing_else():
    for geometry in FITS_WITH_FEWER_SPLITS:
        assert ep.epicache_workspace_size(params(*geometry)) > ep.STATIC_SCRATCH_BYTES
        assert not refused(params(*geometry), False, False), geometry
    rng = random.Random(5)
    for _ in range(4000):
        nb, hkv, g, p = rng.randint(1, 400), rng.choice([1, 2, 4, 8]), rng.choice([1, 3, 4, 7]), rng.choice([16, 50, 64, 128])
        d, n = rng.choice([8, 64, 96, 128]), int(2 ** rng.uniform(6, 16))
        m, dtype = rng.randint(1, n), rng.choice([ep.DTYPE_F32, ep.DTYPE_BF16])
        for scores, keep in ((False, False), (False, True), (True, False), (True, True)):
            too_large = smallest_workspace(nb, hkv, g, p, n, m, scores, keep) > ep.STATIC_SCRATCH_BYTES
            assert refused(params(nb, hkv, g, p, d, n, m, dtype), scores, keep) == too_large, (nb, hkv, g, p, d, n, m)


@pytest.mark.gpu
def test_step_with_fewer_splits_keeps_the_same_rows():
    nb, hkv, g, p, d, n, m = FITS_WITH_FEWER_SPLITS[1]
    print(f"[gpu test] static scratch, fewer key splits: {FITS_WITH_FEWER_SPLITS[1]}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(1)
    q = torch.randn(nb, hkv * g, p, d, device="cuda", generator=gen).bfloat16()
    k = torch.randn(nb, hkv, n, d, device="cuda", generator=gen).bfloat16()
    v = torch.randn(nb, hkv, n, d, device="cuda", generator=gen).bfloat16()
    prm = ep.make_params(q, k, n_cached=m, n_block=n - m, budget=m, reduce=ep.REDUCE_SUM)
    scores = torch.empty(nb, hkv, n, device="cuda")
    ep.epicache_score(prm, q, k, scores, ep.alloc_workspace(prm))
    k0, v0 = k.clone(), v.clone()
    keep = torch.full((nb, hkv, m), -1, dtype=torch.int32, device="cuda")
    ep.epicache_evict_step_static(prm, q, k, v, None, keep)
    idx = keep.long()
    assert (idx[..., 1:] > idx[..., :-1]).all() and idx.min() >= 0 and idx.max() < n
    # sums of up to N fp32 exponentials in another order: relative differences of some 1e-6 at most
    line = scores.topk(m, dim=-1).values[..., -1:]
    kept = torch.zeros_like(scores, dtype=torch.bool).scatter_(-1, idx, True)
    assert (scores >= line * (1 - 1e-5))[kept].all() and (scores <= line * (1 + 1e-5))[~kept].all()
    rows = idx.unsqueeze(-1).expand(-1, -1, -1, d)
    assert torch.equal(k[:, :, :m].view(torch.int16), k0.view(torch.int16).gather(2, rows))
    assert torch.equal(v[:, :, :m].view(torch.int16), v0.view(torch.int16).gather(2, rows))
