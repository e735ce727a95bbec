"""The matrix-core kernels at head dimensions between their row layouts (zero-padded operand chunks), at the row counts
where the forms of a workgroup change, against the float64 oracle.  Scores are fp32 sums of exact bf16 products, far
inside the tolerance of bf16 inputs; weights of the attention keep fp32 precision at head dimensions other than 128, so
its output may only show its own rounding to bf16."""
import numpy as np
import pytest
import torch

from oracle import epicache_oracle as orc
from paper_2509_17396_amd import synth
from tests import parity_util as pu
from tests.test_gpu_parity import gpu_score
from tests.test_gpu_patch_attention import gpu_patch_attention

pytestmark = pytest.mark.gpu


def case(d, hq, hkv, p, n, values="topic_clusters"):
    w = synth.WORKLOADS["llama32_3b"].scaled(E=2, Hq=hq, Hkv=hkv, d=d, p=p, recipe=values)
    return synth.make_layer(w, layer=d, n_ctx=n)


@pytest.mark.parametrize("reduce", [orc.REDUCE_MAX, orc.REDUCE_SUM], ids=["max", "sum"])
@pytest.mark.parametrize("d", [8, 24, 40, 72, 80, 104, 136, 160, 200, 256])
@pytest.mark.parametrize("hq,hkv,p,n", [(2, 2, 7, 65), (3, 3, 33, 130), (6, 2, 43, 200), (6, 2, 60, 333), (4, 1, 75, 700)],
                         ids=["R7", "R33", "R129", "R180", "R300"])
def test_scores_at_any_head_dim(d, hq, hkv, p, n, reduce):
    print(f"[gpu test] score d={d} Hq={hq} Hkv={hkv} p={p} N={n} reduce={reduce}", flush=True)
    q, k, _ = case(d, hq, hkv, p, n)
    got = gpu_score(q.cuda(), k.cuda(), n, 16, reduce)
    want = orc.score(*pu.oracle_inputs(q, k), n, reduce)
    pu.assert_scores_close(got, want, 1e-4, f"d={d}")


@pytest.mark.parametrize("reduce", [orc.REDUCE_MAX, orc.REDUCE_SUM], ids=["max", "sum"])
@pytest.mark.parametrize("d,hq,hkv,p,n", [(128, 96, 32, 64, 8193), (64, 96, 32, 43, 8250), (40, 144, 16, 61, 4100), (128, 10, 2, 64, 700)],
                         ids=["R192_many_tiles", "R129_many_tiles", "R549_many_tiles", "R320"])
def test_scores_where_the_rows_per_workgroup_change(d, hq, hkv, p, n, reduce):
    """192 rows per workgroup, which only launches with many key tiles use, and 128 where these pad less than 256."""
    print(f"[gpu test] score rows d={d} Hq={hq} Hkv={hkv} p={p} N={n} reduce={reduce}", flush=True)
    q, k, _ = case(d, hq, hkv, p, n)
    got = gpu_score(q.cuda(), k.cuda(), n, 16, reduce)
    for e in range(2):
        want = orc.score(*pu.oracle_inputs(q[e:e + 1], k[e:e + 1]), n, reduce)
        pu.assert_scores_close(got[e:e + 1], want, 1e-4, f"d={d} e={e}")


@pytest.mark.parametrize("causal", [1, 0], ids=["causal_patch", "context_only"])
@pytest.mark.parametrize("d", [8, 32, 40, 64, 96, 120, 128])
@pytest.mark.parametrize("hq,hkv,p,n", [(2, 2, 5, 3), (8, 2, 20, 1000), (6, 2, 64, 95), (8, 1, 37, 129), (64, 64, 130, 70)],
                         ids=["few_keys", "R80", "R192", "R296", "many_heads"])
def test_attention_at_any_head_dim(d, hq, hkv, p, n, causal):
    print(f"[gpu test] attention d={d} Hq={hq} Hkv={hkv} p={p} N={n} causal={causal}", flush=True)
    q, k, v = case(d, hq, hkv, p, n + p, "student_t")
    out, lse, _ = gpu_patch_attention(q, k, v, n, causal)
    v64 = synth.to_f64_numpy(v)
    want, want_lse = orc.patch_attention(*pu.oracle_inputs(q, k), v64, n, bool(causal))
    assert np.abs(lse - want_lse).max() <= 2e-5 * (1 + np.abs(want_lse).max())
    vmax = np.abs(v64[:, :, :n + p]).max()
    tol = 2.0 ** -8 * np.abs(want) + (2.0 ** -9 if d == 128 else 1e-5) * vmax
    assert (np.abs(out - want) <= tol).all(), (np.abs(out - want) / tol).max()
