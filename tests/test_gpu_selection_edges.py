"""Register-resident selection (top-M, ragged per head, ragged pooled) at the sizes where its dispatch changes form,
with the score rows that stress the search: pairs of equal scores, a wide dynamic range, one value everywhere."""
import numpy as np
import pytest

from oracle import epicache_oracle as orc
from paper_2509_17396_amd import binding as ep
from tests import parity_util as pu
from tests.test_gpu_parity import gpu_topk
from tests.test_gpu_ragged import gpu_select, lengths

pytestmark = pytest.mark.gpu


def rows_of(kind, rng, shape):
    if kind == "pairs":      # what an appended block that repeats cached rows produces
        half = rng.random(shape[:-1] + ((shape[-1] + 1) // 2,), dtype=np.float32)
        return np.concatenate([half, half], axis=-1)[..., :shape[-1]].copy()
    if kind == "wide":       # sinks and weights that underflow
        return np.exp(rng.uniform(-80, 5, size=shape)).astype(np.float32)
    return np.full(shape, 0.375, np.float32)


@pytest.mark.parametrize("kind", ["pairs", "wide", "flat"])
@pytest.mark.parametrize("N,M", [(1024, 1), (1025, 1024), (2048, 1000), (2049, 77), (4097, 4096), (8193, 5000),
                                 (16384, 300), (16386, 16385), (24577, 12000), (32768, 32767)])
def test_topk_at_the_edges_of_its_forms(N, M, kind):
    print(f"[gpu test] topk N={N} M={M} {kind}", flush=True)
    s = rows_of(kind, np.random.default_rng(N + M), (1, 3, N))
    got = gpu_topk(s, M)
    pu.assert_keep_valid(got, N, M, kind)
    np.testing.assert_array_equal(got, orc.topk(s, M))


@pytest.mark.parametrize("kind", ["pairs", "wide", "flat"])
@pytest.mark.parametrize("select,n_max,H,m_max", [
    (ep.SELECT_PER_HEAD, 2049, 2, 900), (ep.SELECT_PER_HEAD, 8193, 2, 4000), (ep.SELECT_PER_HEAD, 33000, 1, 9000),
    (ep.SELECT_POOLED, 2048, 8, 700), (ep.SELECT_POOLED, 2049, 8, 1500), (ep.SELECT_POOLED, 9500, 4, 6000),
    (ep.SELECT_POOLED, 11000, 8, 3000), (ep.SELECT_POOLED, 12289, 8, 5000), (ep.SELECT_POOLED, 16385, 2, 8000)])
def test_ragged_selection_at_the_edges_of_its_forms(select, n_max, H, m_max, kind):
    print(f"[gpu test] select_ragged {select} N={n_max} H={H} M={m_max} {kind}", flush=True)
    nb = 3
    rng = np.random.default_rng(n_max + H)
    scores = rows_of(kind, rng, (nb, H, n_max))
    n_ctx = lengths(n_max, nb, H, n_max, (n_max, 0, 63))
    budgets = np.array([m_max, 1, max(1, m_max // 3)])
    keep, n_kept, _ = gpu_select(scores, n_ctx, budgets, m_max, select)
    rows = [[scores[b, h, :n_ctx[b, h]] for h in range(H)] for b in range(nb)]
    want = orc.select_ragged(rows, budgets, select == ep.SELECT_POOLED)
    for b in range(nb):
        for h in range(H):
            assert n_kept[b, h] == len(want[b][h]), f"b={b} h={h}"
            np.testing.assert_array_equal(keep[b, h, :n_kept[b, h]], want[b][h], err_msg=f"b={b} h={h}")
