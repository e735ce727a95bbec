"""Scores of rows that do not fill the kernels' row layouts, with infinities among their values: a logit of -inf takes its
key out of the row, as it does at any row length, and whatever stands behind the row in its layout counts as zero."""
import numpy as np
import pytest
import torch

from paper_2509_17396_amd import synth
from tests import parity_util as pu
from tests.test_gpu_parity import gpu_score

pytestmark = pytest.mark.gpu


def reference(q, k, reduce):
    """float64, logits of -inf included"""
    nb, hq, p, d = q.shape
    hkv = k.shape[1]
    rows = q.reshape(nb, hkv, hq // hkv * p, d)
    z = np.empty(rows.shape[:3] + (k.shape[2],))
    for i in range(k.shape[2]):   # no sum over keys and elements at once: an infinity times 0 of another key is none
        z[..., i] = (rows * k[:, :, None, i]).sum(-1) / np.sqrt(d)
    w = np.exp(z - z.max(-1, keepdims=True))
    w /= w.sum(-1, keepdims=True)
    return w.max(2) if reduce == 0 else w.sum(2)


@pytest.mark.parametrize("reduce", [0, 1], ids=["max", "sum"])
@pytest.mark.parametrize("dtype,d", [("bf16", 8), ("bf16", 24), ("bf16", 40), ("bf16", 64), ("bf16", 72), ("bf16", 88),
                                     ("bf16", 112), ("bf16", 128), ("bf16", 136), ("bf16", 200), ("bf16", 256),
                                     ("f32", 8), ("f32", 24), ("f32", 48), ("f32", 72), ("f32", 120), ("f32", 128), ("f32", 160)])
@pytest.mark.parametrize("hq,hkv,p,n", [(2, 2, 7, 65), (4, 2, 33, 450), (6, 2, 60, 333), (4, 1, 75, 700)],
                         ids=["R7", "R66", "R180", "R300"])
def test_a_logit_of_minus_infinity_takes_its_key_out(dtype, d, hq, hkv, p, n, reduce):
    print(f"[gpu test] scores, -inf logits {dtype} d={d} Hq={hq} Hkv={hkv} p={p} N={n} reduce={reduce}", flush=True)
    g = torch.Generator().manual_seed(d + n)
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    q = torch.randn(2, hq, p, d, generator=g)
    q[..., d - 1] = q[..., d - 1].abs() + 0.5   # in the row's last chunk, against positive queries
    q, k = q.to(t), torch.randn(2, hkv, n, d, generator=g).to(t)
    k[0, 0, n // 3, d - 1] = k[1, -1, n - 1, d - 1] = k[0, -1, 0, d - 1] = -float("inf")
    want = reference(*pu.oracle_inputs(q, k), reduce)
    assert np.isfinite(want).all() and (want == 0).sum() == 3
    got = gpu_score(q.cuda(), k.cuda(), n, n // 2, reduce)
    pu.assert_scores_close(got, want, 1e-5 if dtype == "f32" else 1e-4, f"d={d}")
    assert (got[want == 0] == 0).all()


@pytest.mark.parametrize("reduce", [0, 1], ids=["max", "sum"])
@pytest.mark.parametrize("dtype,d", [("bf16", 40), ("bf16", 64), ("bf16", 128), ("bf16", 256), ("f32", 64), ("f32", 160)])
def test_a_run_of_such_keys_in_front_of_the_others(dtype, d, reduce):
    print(f"[gpu test] scores, a run of -inf logits {dtype} d={d} reduce={reduce}", flush=True)
    g = torch.Generator().manual_seed(d)
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    q = torch.randn(2, 4, 33, d, generator=g)
    q[..., 0] = q[..., 0].abs() + 0.5
    q, k = q.to(t), torch.randn(2, 2, 700, d, generator=g).to(t)
    k[0, 0, :300, 0] = -float("inf")
    want = reference(*pu.oracle_inputs(q, k), reduce)
    got = gpu_score(q.cuda(), k.cuda(), 700, 350, reduce)
    pu.assert_scores_close(got, want, 1e-5 if dtype == "f32" else 1e-4, f"d={d}")
    assert (got[0, 0, :300] == 0).all()
