"""KeyDiff scores where the form of the kernels changes: 8 or 16 lanes per row, short and long chunks of rows, chunk
edges, heads of lengths of their own, and rows too many for the one-pass form, against the float64 oracle."""
import numpy as np
import pytest
import torch

from oracle import epicache_oracle as orc
from paper_2509_17396_amd import synth
from tests.test_gpu_keydiff import ATOL_COS, gpu_keydiff

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 64), ("f32", 32)])
@pytest.mark.parametrize("heads,n", [(2, 127), (2, 257), (3, 1025), (260, 513), (130, 1024), (64, 2047), (1, 8193), (1, 65537)])
def test_keydiff_chunk_edges(dtype, d, heads, n):
    print(f"[gpu test] keydiff {dtype} d={d} heads={heads} N={n}", flush=True)
    g = torch.Generator().manual_seed(n + d)
    k = torch.randn(heads, 1, n, d, generator=g) + 0.3
    k = k.to(torch.bfloat16) if dtype == "bf16" else k
    lengths = [[n - (b % 3) * (n // 3)] for b in range(heads)]
    for n_ctx in (None, lengths):
        got = gpu_keydiff(k, n, n_ctx)
        want = orc.score_keydiff(synth.to_f64_numpy(k), n if n_ctx is None else n_ctx)
        for b in range(heads):
            m = n if n_ctx is None else lengths[b][0]
            assert np.abs(got[b, :, :m] - want[b, :, :m]).max() <= ATOL_COS, (b, m)
            assert (got[b, :, m:] == -7.0).all()
        assert np.array_equal(got, gpu_keydiff(k, n, n_ctx))  # every run adds in the same order
