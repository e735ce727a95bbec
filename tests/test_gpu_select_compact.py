"""Selection and compaction in one launch against the two calls for them: the same kept rows and the same bits of K and V,
at the sizes where its form or its number of parts changes, with rows of all lengths and layouts, with and without kept
indices, and on two streams at once."""
import pytest
import torch

from paper_2509_17396_amd import binding as ep

pytestmark = pytest.mark.gpu
DEV = "cuda"


def make(nb, hkv, g, p, d, n, m, dtype, seed, spare=0, rows=None):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    rows = (rows or n) + spare
    q = torch.randn(nb, hkv * g, p, d, device=DEV, generator=gen).to(dtype)
    k = torch.randn(nb, hkv, rows, d, device=DEV, generator=gen).to(dtype)
    v = torch.randn(nb, hkv, rows, d, device=DEV, generator=gen).to(dtype)
    prm = ep.make_params(q, k, n_cached=min(m, n), n_block=n - min(m, n), budget=m, reduce=ep.REDUCE_SUM)
    return q, k, v, prm


def bits(t):
    return t.view(torch.int32 if t.dtype == torch.float32 else torch.int16)


def by_the_two_calls(prm, q, k, v, m, lse=None):
    scores = torch.empty(k.shape[0], k.shape[1], prm.n_cached + prm.n_block, device=DEV)
    keep = torch.empty(k.shape[0], k.shape[1], m, dtype=torch.int32, device=DEV)
    ws = ep.alloc_workspace(prm)
    if lse is None:
        ep.epicache_score(prm, q, k, scores, ws)
    else:
        ep.epicache_score_lse(prm, q, k, lse, scores, ws)
    ep.epicache_topk(prm, scores, keep, ws)
    k, v = k.clone(), v.clone()
    ep.epicache_compact(prm, keep, k, v, ws)
    return keep, k, v


SIZES = [  # items, KV heads, d, N, M, dtype, spare rows
    (1, 1, 128, 2, 1, torch.bfloat16, 0), (1, 3, 8, 300, 299, torch.bfloat16, 5), (2, 1, 64, 384, 256, torch.float32, 0),
    (1, 2, 128, 2048, 1100, torch.bfloat16, 0), (2, 2, 128, 2049, 2048, torch.bfloat16, 64), (1, 2, 256, 4096, 70, torch.bfloat16, 3),
    (3, 8, 128, 4097, 3000, torch.bfloat16, 0), (2, 16, 96, 2024, 1024, torch.bfloat16, 0), (1, 4, 80, 8192, 4111, torch.bfloat16, 0),
    (1, 3, 200, 8193, 5000, torch.bfloat16, 1), (1, 1, 128, 16384, 8000, torch.float32, 0), (1, 2, 24, 16384, 16383, torch.bfloat16, 0),
    (1, 2, 128, 16385, 8000, torch.bfloat16, 0), (1, 1, 128, 16384, 16383, torch.bfloat16, 0),
    # 256 KB of rows per workgroup, up to and beyond 64 MB of them in all
    (4, 16, 128, 2000, 1900, torch.bfloat16, 0), (4, 8, 128, 4001, 3900, torch.bfloat16, 0),
    (4, 8, 128, 8000, 4096, torch.bfloat16, 0), (4, 8, 128, 8000, 4097, torch.bfloat16, 0),
    (2, 8, 128, 16000, 8192, torch.bfloat16, 0), (3, 7, 256, 2500, 1900, torch.bfloat16, 0)]


@pytest.mark.parametrize("with_keep", [True, False])
@pytest.mark.parametrize("nb,hkv,d,n,m,dtype,spare", SIZES)
def test_step_moves_the_rows_that_the_two_calls_move(nb, hkv, d, n, m, dtype, spare, with_keep):
    print(f"[gpu test] select_compact {nb}x{hkv} d={d} N={n} M={m} {dtype} keep={with_keep}", flush=True)
    q, k, v, prm = make(nb, hkv, 2, 20, d, n, m, dtype, n + d, spare)
    want_keep, want_k, want_v = by_the_two_calls(prm, q, k, v, m)
    keep = torch.full((nb, hkv, m), -1, dtype=torch.int32, device=DEV) if with_keep else None
    ep.epicache_evict_step(prm, q, k, v, ep.alloc_workspace(prm), keep_idx=keep)
    assert not with_keep or torch.equal(keep, want_keep)
    assert torch.equal(bits(k), bits(want_k)) and torch.equal(bits(v), bits(want_v))


def parts_of(prm):
    """Where the scores and the kept indices start in the workspace of a step, and where it ends."""
    def up(x):
        return (x + 255) // 256 * 256
    heads, n = prm.n_batch * prm.n_kv_heads, prm.n_cached + prm.n_block
    size = ep.epicache_workspace_size(prm)
    off_keep = size - up(heads * min(prm.budget, n) * 4) - up(prm.n_batch * prm.n_q_heads * prm.patch_len * 4)
    return off_keep - up(heads * n * 4), off_keep, size


@pytest.mark.parametrize("m", [96, 97, 128])
def test_with_and_without_the_part_for_kept_indices(m):
    q, k0, v0, prm = make(1, 2, 2, 20, 128, 3000, m, torch.bfloat16, 5)
    want_keep, want_k, want_v = by_the_two_calls(prm, q, k0, v0, m)
    _, off_keep, total = parts_of(prm)
    for size in (total, off_keep):
        k, v, keep = k0.clone(), v0.clone(), torch.full((1, 2, m), -1, dtype=torch.int32, device=DEV)
        ep.epicache_evict_step(prm, q, k, v, torch.empty(size, dtype=torch.uint8, device=DEV), keep_idx=keep)
        assert torch.equal(keep, want_keep) and torch.equal(bits(k), bits(want_k)) and torch.equal(bits(v), bits(want_v))


# one pass over the rows, in tiles of 32 and of 256; row tiles whose splits are combined between the passes or not, in
# both of the layouts of a row's normaliser
BEHIND = [(1, 2, 1, 20, 128, 3000, 200, torch.bfloat16), (2, 4, 4, 64, 128, 1024, 512, torch.bfloat16),
          (2, 32, 4, 80, 64, 2304, 200, torch.bfloat16), (2, 32, 4, 80, 96, 2304, 200, torch.bfloat16),
          (1, 2, 4, 80, 128, 2000, 300, torch.bfloat16), (1, 2, 4, 80, 80, 2000, 300, torch.bfloat16),
          (1, 3, 2, 30, 64, 700, 300, torch.float32), (1, 2, 2, 150, 64, 700, 300, torch.float32)]


@pytest.mark.parametrize("way", ["plain", "lse", "one_chunk"])
@pytest.mark.parametrize("nb,hkv,g,p,d,n,m,dtype", BEHIND)
def test_what_a_step_does_not_need_of_the_workspace_is_left_alone(nb, hkv, g, p, d, n, m, dtype, way):
    """The caller's kept indices may lie where the workspace would have them, anything else behind them."""
    print(f"[gpu test] select_compact behind the workspace {nb}x{hkv} rows={g * p} d={d} N={n} M={m} {dtype} {way}", flush=True)
    q, k0, v0, prm = make(nb, hkv, g, p, d, n, m, dtype, n + d)
    lse = torch.rand(nb, hkv * g, p, device=DEV, generator=torch.Generator(device=DEV).manual_seed(1)) + 6.0
    want_keep, want_k, want_v = by_the_two_calls(prm, q, k0, v0, m, lse if way == "lse" else None)
    off_scores, off_keep, total = parts_of(prm)

    def step(ws, k, v, scores, keep):
        if way == "plain":
            ep.epicache_evict_step(prm, q, k, v, ws, scores, keep)
        elif way == "lse":
            ep.epicache_evict_step_lse(prm, q, k, v, lse, ws, scores, keep)
        else:
            ep.epicache_evict_step_overlapped(prm, q, k, v, ws, torch.cuda.Stream(), 1, scores, keep)
        torch.cuda.synchronize()

    k, v, ws = k0.clone(), v0.clone(), torch.full((total,), 0x5a, dtype=torch.uint8, device=DEV)
    keep = torch.full((nb, hkv, m), -1, dtype=torch.int32, device=DEV)
    step(ws, k, v, torch.empty(nb, hkv, n, device=DEV), keep)
    assert bool((ws[off_scores:] == 0x5a).all())
    assert torch.equal(keep, want_keep) and torch.equal(bits(k), bits(want_k)) and torch.equal(bits(v), bits(want_v))
    k, v = k0.clone(), v0.clone()
    keep = ws[off_keep:off_keep + nb * hkv * m * 4].view(torch.int32).view(nb, hkv, m)
    step(ws, k, v, None, keep)
    assert bool((ws[off_keep + nb * hkv * m * 4:] == 0x5a).all())
    assert torch.equal(keep, want_keep) and torch.equal(bits(k), bits(want_k)) and torch.equal(bits(v), bits(want_v))


@pytest.mark.parametrize("n,m,w", [(1000, 700, 64), (4337, 3000, 64), (9000, 4100, 17)])
def test_window_rows_behind_the_selected_ones(n, m, w):
    print(f"[gpu test] select_compact with a window N={n} M={m} w={w}", flush=True)
    q, k, v, prm = make(2, 2, 2, w, 128, n, m, torch.bfloat16, n)
    k0, v0 = k.clone(), v.clone()
    scores = torch.empty(2, 2, n - w, device=DEV)
    keep = torch.full((2, 2, m), -1, dtype=torch.int32, device=DEV)
    ws = torch.empty(ep.epicache_snapkv_workspace_size(prm), dtype=torch.uint8, device=DEV)
    ep.epicache_evict_step_snapkv(prm, q, k, v, ws, scores, keep)
    for b in range(2):
        for h in range(2):
            best = torch.sort(scores[b, h].cpu(), descending=True, stable=True).indices[:m - w].sort().values
            want = torch.cat([best, torch.arange(n - w, n)])
            assert torch.equal(keep[b, h].cpu().long(), want)
            assert torch.equal(bits(k)[b, h, :m], bits(k0)[b, h][want.to(DEV)])
            assert torch.equal(bits(v)[b, h, :m], bits(v0)[b, h][want.to(DEV)])


def test_steps_on_two_streams_at_once():
    """Each launch fills the chip by itself, so that parts of both wait for CUs while others wait for parts."""
    print("[gpu test] select_compact on two streams", flush=True)
    a, b = make(4, 8, 2, 16, 128, 8192, 4096, torch.bfloat16, 1), make(4, 8, 2, 16, 128, 8100, 4000, torch.bfloat16, 2)
    want = [by_the_two_calls(prm, q, k, v, m)[1:] for (q, k, v, prm), m in ((a, 4096), (b, 4000))]
    caches = [[(q, k.clone(), v.clone(), prm, ep.alloc_workspace(prm)) for _ in range(6)] for q, k, v, prm in (a, b)]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    for i in range(6):
        for s, c in zip(streams, caches):
            with torch.cuda.stream(s):
                q, k, v, prm, ws = c[i]
                ep.epicache_evict_step(prm, q, k, v, ws)
    torch.cuda.synchronize()
    for c, (wk, wv) in zip(caches, want):
        for _, k, v, _, _ in c:
            assert torch.equal(bits(k), bits(wk)) and torch.equal(bits(v), bits(wv))


def hard_keys(kind, gen, k):
    """Keys whose scores tie across the threshold, or are not finite."""
    nb, hkv, n, d = k.shape
    if kind == "repeated":    # every key up to nine times, in runs and far apart
        k.copy_(k[:, :, torch.randint(0, max(1, n // 9), (n,), device=DEV, generator=gen)])
        k[:, :, n // 3:n // 2] = k[:, :, n // 3:n // 3 + 1]
    elif kind == "one_value":
        k.copy_(k[:, :, :1].expand(-1, -1, n, -1).clone())
    elif kind == "infinite":  # weights of 0 and NaN, all of the last head's NaN
        k[:, :, n // 5] = float("-inf")
        k[:, 0, n // 7:n // 6] = -1e30
        k[:, -1, 1] = float("nan")
    return k


def strided(t, rows_between, gen):
    """The same rows at a token stride of 1 + rows_between of them, with noise in between."""
    nb, h, n, d = t.shape
    wide = torch.randn(nb, h, n, 1 + rows_between, d, device=DEV, generator=gen).to(t.dtype)
    wide[:, :, :, 0] = t
    return wide, wide[:, :, :, 0]


@pytest.mark.parametrize("way", ["plain", "one_chunk", "attn", "attn_causal"])
@pytest.mark.parametrize("kind", ["smooth", "repeated", "one_value", "infinite"])
@pytest.mark.parametrize("nb,hkv,d,n,m,dtype,between", [
    (1, 2, 64, 600, 250, torch.float32, 0), (2, 3, 128, 2100, 1500, torch.bfloat16, 1), (1, 8, 64, 4200, 2000, torch.bfloat16, 3),
    (1, 2, 96, 9001, 4500, torch.bfloat16, 0)])
def test_every_route_on_hard_keys_and_in_wide_layouts(nb, hkv, d, n, m, dtype, between, kind, way):
    """Against epicache_topk on the step's own scores and epicache_compact on its indices; rows between the cache's stay."""
    print(f"[gpu test] select_compact {way} {kind} {nb}x{hkv} d={d} N={n} M={m} {dtype} between={between}", flush=True)
    gen, p, causal = torch.Generator(device=DEV).manual_seed(n + d), 24, way == "attn_causal"
    rows = n + (p if causal else 0)
    q = torch.randn(nb, hkv * 2, p, d, device=DEV, generator=gen).to(dtype)
    k0 = hard_keys(kind, gen, torch.randn(nb, hkv, rows, d, device=DEV, generator=gen).to(dtype))
    v0 = torch.randn(nb, hkv, rows, d, device=DEV, generator=gen).to(dtype)
    (wide_k, k), (wide_v, v) = strided(k0, between, gen), strided(v0, between, gen)
    want_wide_k, want_wide_v = wide_k.clone(), wide_v.clone()
    want_k, want_v = want_wide_k[:, :, :, 0], want_wide_v[:, :, :, 0]
    # sums over the queries are added up in an order that follows the key's place; equal keys have equal maxima
    reduce = ep.REDUCE_MAX if kind in ("repeated", "one_value") else ep.REDUCE_SUM
    prm = ep.make_params(q, k, n_cached=m, n_block=n - m, budget=m, reduce=reduce, causal_patch=int(causal))
    ws, scores = ep.alloc_workspace(prm), torch.empty(nb, hkv, n, device=DEV)
    keep = torch.full((nb, hkv, m), -1, dtype=torch.int32, device=DEV)
    if way == "plain":
        ep.epicache_evict_step(prm, q, k, v, ws, scores, keep)
    elif way == "one_chunk":
        ep.epicache_evict_step_overlapped(prm, q, k, v, ws, torch.cuda.Stream(), 1, scores, keep)
    else:
        ep.epicache_evict_step_attn(prm, q, k, v, torch.empty(nb, hkv * 2, p, d, device=DEV, dtype=dtype), ws, scores, keep)
    torch.cuda.synchronize()
    want_keep = torch.empty_like(keep)
    ep.epicache_topk(prm, scores, want_keep, ws)
    ep.epicache_compact(prm, want_keep, want_k, want_v, ws)
    assert torch.equal(keep, want_keep)
    assert torch.equal(bits(wide_k), bits(want_wide_k)) and torch.equal(bits(wide_v), bits(want_wide_v))
    if kind == "one_value":   # equal scores: the first rows stay
        assert torch.equal(keep, torch.arange(m, dtype=torch.int32, device=DEV).expand(nb, hkv, m))
