"""Rows moved in ranges that wait for each other: epicache_compact with room for their claims, and the launcher with clear ones,
against plain indexing, bit for bit, at the edges of ranges and rounds, and whole steps whose rows are too many for the
selection's own launch."""
import ctypes
import os

import pytest
import torch

from paper_2509_17396_amd import binding as ep
from paper_2509_17396_amd import build

pytestmark = pytest.mark.gpu
DEV = "cuda"


def bits(t):
    return t.view(torch.int32 if t.dtype == torch.float32 else torch.int16)


def cache(nb, heads, n, d, dtype, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    k, v = (torch.randn(nb, heads, n, d, device=DEV, generator=g).to(dtype) for _ in range(2))
    return g, k, v


def selftest(name):
    so = os.path.join(os.path.dirname(build.LIB), "selftest", f"lib{name}.so")
    if not os.path.exists(so):
        build.build_selftests()
    return ctypes.CDLL(so)


def kept_rows(kind, nb, heads, n, m, g):
    if kind == "drawn":
        return torch.rand(nb, heads, n, device=DEV, generator=g).topk(m, dim=-1).indices.sort(dim=-1).values.int().contiguous()
    if kind in ("in_place", "last_moves"):  # none does: ranges that read nothing and wait for nothing, but the last one
        keep = torch.arange(m, device=DEV)
        if kind == "last_moves":
            keep[-1] = n - 1
        return keep.expand(nb, heads, m).int().contiguous()
    # every row moves, by the most and by the least there is
    return torch.arange(n - m if kind == "tail" else 1, n, device=DEV)[:m].expand(nb, heads, m).int().contiguous()


def gathered(k0, v0, keep, m):
    rows = keep.long().unsqueeze(-1).expand(-1, -1, -1, k0.shape[-1])
    return [torch.cat([bits(x).gather(2, rows), bits(x)[:, :, m:]], dim=2) for x in (k0, v0)]


# batch, heads, rows, kept, head_dim, dtype: sizes for which the call clears claims and takes ranges
SHAPES = [(1, 3, 20000, 11000, 128, torch.bfloat16), (1, 2, 33000, 32768, 128, torch.bfloat16), (1, 1, 4200, 4097, 128, torch.bfloat16),
          (2, 4, 9001, 7777, 96, torch.bfloat16), (1, 5, 8000, 7999, 256, torch.bfloat16), (1, 2, 30000, 25000, 8, torch.bfloat16),
          (1, 3, 17000, 9000, 40, torch.bfloat16), (1, 2, 9000, 4096, 256, torch.float32), (1, 7, 5000, 3073, 64, torch.float32),
          (1, 40, 3000, 1537, 128, torch.bfloat16), (52, 8, 1400, 1281, 128, torch.bfloat16), (80, 8, 600, 500, 128, torch.bfloat16)]
# sizes for which it does not, though the workspace has the room
PLAIN = [(1, 1, 2000, 1537, 128, torch.bfloat16), (1, 2, 9000, 4000, 256, torch.float32), (1, 7, 5000, 2049, 64, torch.float32),
         (56, 4, 1100, 1025, 128, torch.bfloat16), (64, 8, 700, 600, 128, torch.bfloat16)]


@pytest.mark.parametrize("kind", ["drawn", "tail", "all_but_the_first"])
@pytest.mark.parametrize("shape", SHAPES + PLAIN, ids=["-".join(map(str, s)) for s in SHAPES + PLAIN])
def test_compact_in_ranges_is_a_gather(shape, kind):
    nb, heads, n, m, d, dtype = shape
    print(f"[gpu test] compact in ranges {shape} {kind}", flush=True)
    rules = selftest("launch_rules")
    row = d * dtype.itemsize
    ranges = rules.compact_parts(nb * heads, m, row) > 0 and rules.compact_parts_pay_for_claims(nb * heads, m, row)
    assert bool(ranges) == (shape in SHAPES)
    g, k0, v0 = cache(nb, heads, n, d, dtype, n + d)
    keep = kept_rows(kind, nb, heads, n, m, g)
    prm = ep.make_params(k0[:, :, :16], k0, n_cached=m, n_block=n - m, budget=m)
    want = gathered(k0, v0, keep, m)
    per_head = 256 * nb * heads
    inside = torch.full((per_head + keep.numel() * 4,), 0xff, dtype=torch.uint8, device=DEV)
    inside[:keep.numel() * 4] = keep.view(torch.uint8).flatten()
    for ws, idx in ((torch.full((per_head,), 0xff, dtype=torch.uint8, device=DEV), keep),   # claims start as anything
                    (torch.full((per_head - 1,), 0xff, dtype=torch.uint8, device=DEV), keep),  # no room
                    (None, keep),
                    (inside, inside)):                                                       # the indices lie there
        k, v = k0.clone(), v0.clone()
        ep.epicache_compact(prm, idx, k, v, ws)
        torch.cuda.synchronize()
        assert torch.equal(bits(k), want[0]) and torch.equal(bits(v), want[1])
    assert torch.equal(inside[:keep.numel() * 4].view(torch.int32), keep.flatten())


# sizes that a step moves in ranges and epicache_compact does not; how many: one (which needs no claims), as few as hold the rows, more
STEP_SHAPES = [((1, 230, 400, 300, 128, torch.bfloat16), 1), ((64, 8, 700, 512, 128, torch.bfloat16), 1),
               ((64, 8, 700, 513, 128, torch.bfloat16), 2), ((1, 1, 2000, 1537, 128, torch.bfloat16), 32),
               ((1, 2, 3000, 1000, 256, torch.float32), 32), ((1, 7, 5000, 2049, 64, torch.float32), 18),
               ((3, 10, 2300, 1600, 96, torch.bfloat16), 4), ((1, 20, 300, 257, 128, torch.bfloat16), 6),
               ((1, 4, 900, 769, 32, torch.bfloat16), 31), ((5, 6, 310, 300, 80, torch.bfloat16), 4)]


@pytest.mark.parametrize("kind", ["drawn", "tail", "all_but_the_first", "in_place", "last_moves"])
@pytest.mark.parametrize("shape,ranges", STEP_SHAPES, ids=["-".join(map(str, s)) for s, _ in STEP_SHAPES])
def test_ranges_of_a_step_are_a_gather(shape, ranges, kind):
    nb, heads, n, m, d, dtype = shape
    print(f"[gpu test] ranges of a step {shape} {kind}", flush=True)
    lib, pitch = selftest("select_compact_patience"), ctypes.c_int(0)
    per_head = lib.claims_per_head(ctypes.byref(pitch))
    lib.compact_with_claims.argtypes = [ctypes.c_int] * 6 + [ctypes.c_void_p] * 5
    g, k0, v0 = cache(nb, heads, n, d, dtype, n + d)
    keep = kept_rows(kind, nb, heads, n, m, g)
    want = gathered(k0, v0, keep, m)
    claims = torch.zeros(nb * heads, per_head, dtype=torch.int32, device=DEV)
    k, v = k0.clone(), v0.clone()
    got = lib.compact_with_claims(nb, heads, d, dtype.itemsize, n, m, keep.data_ptr(), claims.data_ptr(), k.data_ptr(), v.data_ptr(),
                                  torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert got == ranges
    assert torch.equal(bits(k), want[0]) and torch.equal(bits(v), want[1])


def test_compact_writes_no_more_of_its_workspace_than_it_says():
    """The first 256 bytes per head, and nothing where that is more than there is or the kept indices lie there."""
    nb, heads, n, m, d = 1, 6, 12000, 8000, 128
    print("[gpu test] compact leaves the rest of its workspace", flush=True)
    g, k0, v0 = cache(nb, heads, n, d, torch.bfloat16, 3)
    keep = torch.rand(nb, heads, n, device=DEV, generator=g).topk(m, dim=-1).indices.sort(dim=-1).values.int().contiguous()
    prm = ep.make_params(k0[:, :, :16], k0, n_cached=m, n_block=n - m, budget=m)
    used = 256 * nb * heads
    before = torch.randint(0, 256, (used + 4096,), dtype=torch.uint8, device=DEV, generator=g)
    ws = before.clone()
    ep.epicache_compact(prm, keep, k0.clone(), v0.clone(), ws)
    torch.cuda.synchronize()
    assert torch.equal(ws[used:], before[used:])
    assert not torch.equal(ws[:used], before[:used])  # the ranges' claims: this is the form that needs them
    ws = before.clone()
    ep.epicache_compact(prm, keep, k0.clone(), v0.clone(), ws[:used - 1])
    torch.cuda.synchronize()
    assert torch.equal(ws, before)


@pytest.mark.parametrize("n,m,path", [(18000, 11000, "step"), (18000, 11000, "static"), (16500, 9000, "snapkv"), (17000, 16999, "lse")])
def test_steps_with_too_many_rows_for_one_launch(n, m, path):
    nb, heads, p, d = 1, 2, 32, 128
    print(f"[gpu test] step, rows in ranges n={n} m={m} {path}", flush=True)
    g, k0, v0 = cache(nb, heads, n, d, torch.bfloat16, n)
    q = torch.randn(nb, heads * 2, p, d, device=DEV, generator=g).bfloat16()
    prm = ep.make_params(q, k0, n_cached=m, n_block=n - m, budget=m, reduce=ep.REDUCE_SUM)
    for _ in range(2):  # the second call finds what the first has left in the workspace
        k, v = k0.clone(), v0.clone()
        keep = torch.full((nb, heads, m), -1, dtype=torch.int32, device=DEV)
        if path == "static":
            ep.epicache_evict_step_static(prm, q, k, v, None, keep)
        elif path == "snapkv":
            ws = torch.full((ep.epicache_snapkv_workspace_size(prm),), 0xff, dtype=torch.uint8, device=DEV)
            ep.epicache_evict_step_snapkv(prm, q, k, v, ws, keep_idx=keep)
        else:
            ws = torch.full((ep.epicache_workspace_size(prm),), 0xff, dtype=torch.uint8, device=DEV)
            if path == "lse":
                ep.epicache_evict_step_lse(prm, q, k, v, torch.zeros(nb, heads * 2, p, device=DEV), ws, keep_idx=keep)
            else:
                ep.epicache_evict_step(prm, q, k, v, ws, keep_idx=keep)
        torch.cuda.synchronize()
        idx = keep.long()
        assert (idx[..., 1:] > idx[..., :-1]).all() and idx.min() >= 0 and idx.max() < n
        rows = idx.unsqueeze(-1).expand(-1, -1, -1, d)
        for x, x0 in ((k, k0), (v, v0)):
            assert torch.equal(bits(x)[:, :, :m], bits(x0).gather(2, rows)) and torch.equal(bits(x)[:, :, m:], bits(x0)[:, :, m:])


@pytest.mark.parametrize("chunks", [0, 1, 3], ids=["one_stream", "one_chunk", "last_of_three"])
@pytest.mark.parametrize("select", [ep.SELECT_PER_HEAD, ep.SELECT_POOLED], ids=["per_head", "pooled"])
def test_ragged_rows_in_ranges(select, chunks):
    """Heads of uneven lengths, one of them empty: ranges that are cut for the longest, and some that have no rows."""
    nb, heads, p, d, n, m = 3, 2, 32, 128, 9000, 5000
    print(f"[gpu test] ragged rows in ranges select={select} chunks={chunks}", flush=True)
    g, k0, v0 = cache(nb, heads, n, d, torch.bfloat16, 7)
    q = torch.randn(nb, heads * 2, p, d, device=DEV, generator=g).bfloat16()
    n_ctx = torch.tensor([[9000, 3000], [8999, 1], [7001, 0]], dtype=torch.int32, device=DEV)
    budgets = torch.tensor([5000, 4097, 300], dtype=torch.int32, device=DEV)
    prm = ep.make_params(q, k0, n_cached=m, n_block=n - m, budget=m, reduce=ep.REDUCE_SUM)
    if chunks:
        size, cap, _ = ep.epicache_ragged_overlapped_workspace_size(prm, select, chunks)
        aux = torch.cuda.Stream()
    else:
        size, cap = ep.epicache_ragged_workspace_size(prm, select)
    ws = torch.full((size,), 0xff, dtype=torch.uint8, device=DEV)
    for _ in range(2):
        k, v = k0.clone(), v0.clone()
        keep = torch.full((nb, heads, cap), -1, dtype=torch.int32, device=DEV)
        kept = torch.zeros(nb, heads, dtype=torch.int32, device=DEV)
        if chunks:
            ep.epicache_evict_step_ragged_overlapped(prm, select, q, k, v, n_ctx, budgets, kept, ws, aux, chunks, keep_idx=keep)
        else:
            ep.epicache_evict_step_ragged(prm, select, q, k, v, n_ctx, budgets, kept, ws, keep_idx=keep)
        torch.cuda.synchronize()
        for b in range(nb):
            total = kept[b].sum().item()
            want = budgets[b].item() * heads if select == ep.SELECT_POOLED else 0
            assert select != ep.SELECT_POOLED or total == min(want, n_ctx[b].sum().item())
            for h in range(heads):
                c = kept[b, h].item()
                idx = keep[b, h, :c].long()
                assert select == ep.SELECT_POOLED or c == min(budgets[b].item(), n_ctx[b, h].item())
                assert c == 0 or ((idx[1:] > idx[:-1]).all() and idx[0] >= 0 and idx[-1] < n_ctx[b, h])
                for x, x0 in ((k, k0), (v, v0)):
                    assert torch.equal(bits(x)[b, h, :c], bits(x0)[b, h, idx]) and torch.equal(bits(x)[b, h, c:], bits(x0)[b, h, c:])


def test_ragged_ranges_of_many_heads():
    """More ranges than the chip holds at once: heads that keep nothing, less than one range, just one, and several of them."""
    nb, heads, p, d, n, m = 40, 8, 32, 128, 2200, 450
    print("[gpu test] ragged ranges of many heads", flush=True)
    g, k0, v0 = cache(nb, heads, n, d, torch.bfloat16, 19)
    q = torch.randn(nb, heads, p, d, device=DEV, generator=g).bfloat16()
    n_ctx = torch.randint(1, n + 1, (nb, heads), dtype=torch.int32, device=DEV, generator=g)
    n_ctx[0], n_ctx[1, 1:], n_ctx[2, :7] = 0, 0, 3
    n_ctx[3], n_ctx[4] = torch.tensor([n, 512, 0, 0, 0, 0, 513, 0], device=DEV), n
    budgets = torch.full((nb,), m, dtype=torch.int32, device=DEV)
    prm = ep.make_params(q, k0, n_cached=m, n_block=n - m, budget=m, reduce=ep.REDUCE_SUM)
    size, cap = ep.epicache_ragged_workspace_size(prm, ep.SELECT_POOLED)
    rows = ctypes.c_int(0)
    assert selftest("launch_rules").compact_ranges(nb * heads, m, cap, d * 2, ctypes.byref(rows)) == 5 and rows.value == 512
    ws = torch.full((size,), 0xff, dtype=torch.uint8, device=DEV)
    for _ in range(2):
        k, v = k0.clone(), v0.clone()
        keep = torch.full((nb, heads, cap), -1, dtype=torch.int32, device=DEV)
        kept = torch.zeros(nb, heads, dtype=torch.int32, device=DEV)
        ep.epicache_evict_step_ragged(prm, ep.SELECT_POOLED, q, k, v, n_ctx, budgets, kept, ws, keep_idx=keep)
        torch.cuda.synchronize()
        counts = kept.tolist()
        assert {0, 3} <= {c for x in counts for c in x} and max(c for x in counts for c in x) > 1024
        for b in range(nb):
            assert sum(counts[b]) == min(m * heads, int(n_ctx[b].sum()))
            for h in range(heads):
                c = counts[b][h]
                idx = keep[b, h, :c].long()
                for x, x0 in ((k, k0), (v, v0)):
                    assert torch.equal(bits(x)[b, h, :c], bits(x0)[b, h, idx]) and torch.equal(bits(x)[b, h, c:], bits(x0)[b, h, c:])


@pytest.mark.parametrize("heads,n,m,d", [(5, 9000, 4000, 128), (7, 14000, 13000, 128), (9, 2000, 1000, 128), (13, 6000, 5000, 64), (3, 4097, 4000, 256)])
def test_ranges_of_few_heads_on_all_xcds(heads, n, m, d):
    print(f"[gpu test] selection and ranges, heads={heads} n={n} m={m} d={d}", flush=True)
    g, k0, v0 = cache(1, heads, n, d, torch.bfloat16, n)
    q = torch.randn(1, heads, 32, d, device=DEV, generator=g).bfloat16()
    prm = ep.make_params(q, k0, n_cached=m, n_block=n - m, budget=m, reduce=ep.REDUCE_MAX)
    ws = torch.full((ep.epicache_workspace_size(prm),), 0xff, dtype=torch.uint8, device=DEV)
    scores = torch.empty(1, heads, n, device=DEV)
    want = torch.empty(1, heads, m, dtype=torch.int32, device=DEV)
    ep.epicache_score(prm, q, k0, scores, ws)
    ep.epicache_topk(prm, scores, want, ws)
    for _ in range(2):
        k, v = k0.clone(), v0.clone()
        keep = torch.full((1, heads, m), -1, dtype=torch.int32, device=DEV)
        ep.epicache_evict_step(prm, q, k, v, ws, keep_idx=keep)
        torch.cuda.synchronize()
        assert torch.equal(keep, want)
        rows = keep.long().unsqueeze(-1).expand(-1, -1, -1, d)
        for x, x0 in ((k, k0), (v, v0)):
            assert torch.equal(bits(x)[:, :, :m], bits(x0).gather(2, rows)) and torch.equal(bits(x)[:, :, m:], bits(x0)[:, :, m:])


@pytest.mark.parametrize("group,with_lse", [(2, False), (2, True), (13, False), (13, True)], ids=["stream", "stream_lse", "rows_416", "rows_416_lse"])
def test_scoring_clears_the_claims_of_every_head(group, with_lse):
    """Heads without a key among them: their claims start as what an earlier call left there, small whole numbers."""
    nb, heads, p, d, n, m = 3, 2, 32, 128, 9000, 5000
    print(f"[gpu test] claims of heads without keys, group={group} lse={with_lse}", flush=True)
    g, k, v = cache(nb, heads, n, d, torch.bfloat16, 11)
    q = torch.randn(nb, heads * group, p, d, device=DEV, generator=g).bfloat16()
    n_ctx = torch.tensor([[9000, 0], [0, 8000], [7001, 0]], dtype=torch.int32, device=DEV)
    budgets = torch.full((nb,), m, dtype=torch.int32, device=DEV)
    prm = ep.make_params(q, k, n_cached=m, n_block=n - m, budget=m, reduce=ep.REDUCE_SUM)
    size, cap = ep.epicache_ragged_workspace_size(prm, ep.SELECT_PER_HEAD)
    kept = torch.zeros(nb, heads, dtype=torch.int32, device=DEV)
    lse = torch.zeros(nb, heads * group, p, device=DEV) if with_lse else None
    ws = torch.full((size // 4,), 7, dtype=torch.int32, device=DEV)
    ep.epicache_evict_step_ragged(prm, ep.SELECT_PER_HEAD, q, k, v, n_ctx, budgets, kept, ws.view(torch.uint8),
                                  keep_idx=torch.empty(nb, heads, cap, dtype=torch.int32, device=DEV), row_lse=lse)
    torch.cuda.synchronize()
    assert kept.tolist() == [[m, 0], [0, m], [m, 0]]
    words = ws.cpu()
    pitch, per_head = 16, 64  # words: ranges taken and ranges loaded of K, the same of V, a line of 64 bytes each; of a head
    full = [0, 3, 4]          # heads with rows: every one took and reported the same number of ranges, more than one
    places = []
    for at in range(0, words.numel() - nb * heads * per_head, per_head):
        c = [[int(words[at + h * per_head + i * pitch]) & 0xffffffff for i in range(4)] for h in range(nb * heads)]
        if 1 < c[0][0] <= 32 and all(x == [c[0][0], (1 << c[0][0]) - 1] * 2 for x in (c[h] for h in full)):
            places.append(c)
    assert places, "the claims were not found"
    for h in (1, 2, 5):  # nobody has rows to report: cleared, and taken at most as often as there are ranges
        taken_k, loaded_k, taken_v, loaded_v = places[0][h]  # (a place further on is the same one, seen from a later head)
        assert taken_k in (0, places[0][0][0]) and taken_v == taken_k
        assert loaded_k in (0, places[0][0][1]) and loaded_v == loaded_k
