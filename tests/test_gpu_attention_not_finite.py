"""Patch attention over caches that hold infinities and NaNs: a value that a query does not see (a later patch token's,
or the padding of a key row in the kernels' layouts) has no part in its output, and one that it sees reaches its own
column and no other.  Against a float64 reference that only ever touches the rows a query sees."""
import numpy as np
import pytest
import torch

from paper_2509_17396_amd import synth
from tests.test_gpu_patch_attention import gpu_patch_attention, out_tolerance

pytestmark = pytest.mark.gpu

# query heads, KV heads, batch, patch, context rows: one to eight row blocks and key groups per workgroup, and the edges
# of key tiles
SHAPES = [(2, 1, 1, 5, 100), (8, 2, 2, 40, 170), (16, 4, 16, 33, 96), (24, 8, 48, 70, 63)]


def reference(q, k, v, n, causal):
    """o[b, h, t, :] and the normalisers, query by query over the keys it sees."""
    nb, hq, p, d = q.shape
    g = hq // k.shape[1]
    out, lse = np.zeros(q.shape), np.zeros(q.shape[:3])
    for b in range(nb):
        for h in range(hq):
            kk, vv = k[b, h // g], v[b, h // g]
            for t in range(p):
                seen = n + t + 1 if causal else n
                z = (q[b, h, t] * kk[:seen]).sum(1) / np.sqrt(d)
                w = np.exp(z - z.max())
                lse[b, h, t] = z.max() + np.log(w.sum())
                w /= w.sum()
                w[z == -np.inf] = 0
                # a key that is masked out by a logit of -inf has no finite values replaced below
                out[b, h, t] = (w[:, None] * vv[:seen]).sum(0)
    return out, lse


@pytest.mark.parametrize("causal", [1, 0], ids=["causal_patch", "context_only"])
@pytest.mark.parametrize("shape", SHAPES, ids=["RW1", "R160", "R132", "R210"])
@pytest.mark.parametrize("d", [8, 40, 64, 96, 112, 128])
def test_only_what_a_query_sees_counts(d, shape, causal):
    hq, hkv, nb, p, n = shape
    nb = min(nb, 4) if d in (8, 112) else nb
    print(f"[gpu test] attention, values not finite: d={d} shape={shape} causal={causal}", flush=True)
    g = torch.Generator().manual_seed(d + n)
    q = torch.randn(nb, hq, p, d, generator=g).bfloat16()
    k = torch.randn(nb, hkv, n + p, d, generator=g).bfloat16()
    v = torch.randn(nb, hkv, n + p, d, generator=g).bfloat16()
    inf = float("inf")
    last = nb - 1
    v[0, 0, n + p - 1, 1] = inf            # the last patch token: of interest to itself alone
    v[0, 0, n + p // 2, d - 1] = -inf
    v[last, -1, n + 1, 0] = float("nan")
    v[last, -1, n // 3, 2], v[last, -1, n // 2, 2] = inf, -inf   # context rows, seen by all: NaN in column 2
    v[0, 0, n - 1, 3] = inf
    k[0, 0, n + p - 1, 0] = float("nan")   # a key that only the last token sees
    # logits of -inf for a whole row of keys: the last element of the key row against positive queries
    q[last, :, :, d - 1] = q[last, :, :, d - 1].abs() + 0.5
    k[last, 0, n // 4, d - 1] = -inf
    with np.errstate(invalid="ignore"):
        want, want_lse = reference(*(synth.to_f64_numpy(x) for x in (q, k, v)), n, causal)
    out, lse, _ = gpu_patch_attention(q, k, v, n, causal)
    ok = np.isfinite(want)
    assert ok.any() and not ok.all()
    np.testing.assert_array_equal(np.isnan(out), np.isnan(want))
    np.testing.assert_array_equal(out[~ok], want[~ok])
    finite_v = synth.to_f64_numpy(v)
    finite_v = finite_v[np.isfinite(finite_v)]
    assert (np.abs(out[ok] - want[ok]) <= out_tolerance(want, finite_v, q.dtype)[ok]).all()
    ok = np.isfinite(want_lse)
    np.testing.assert_array_equal(np.isnan(lse), ~ok)
    assert np.abs(lse - want_lse)[ok].max() <= 2e-5 * (1 + np.abs(want_lse[ok]).max())


@pytest.mark.parametrize("dtype,d", [("f32", 40), ("f32", 128), ("bf16", 160), ("bf16", 64), ("bf16", 128)])
def test_a_run_of_logits_of_minus_infinity_in_front(dtype, d):
    print(f"[gpu test] attention, a run of -inf logits {dtype} d={d}", flush=True)
    g = torch.Generator().manual_seed(d)
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    n, p = 600, 9
    q = torch.randn(1, 4, p, d, generator=g)
    q[..., 0] = q[..., 0].abs() + 0.5
    q = q.to(t)
    k, v = torch.randn(1, 2, n + p, d, generator=g).to(t), torch.randn(1, 2, n + p, d, generator=g).to(t)
    k[0, 0, :300, 0] = -float("inf")
    with np.errstate(invalid="ignore"):
        want, want_lse = reference(*(synth.to_f64_numpy(x) for x in (q, k, v)), n, 1)
    assert np.isfinite(want).all()
    out, lse, _ = gpu_patch_attention(q, k, v, n, 1)
    assert (np.abs(out - want) <= out_tolerance(want, synth.to_f64_numpy(v), q.dtype)).all()
    assert np.abs(lse - want_lse).max() <= 2e-5 * (1 + np.abs(want_lse).max())
