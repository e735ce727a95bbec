"""Matching at the episode counts where its rule takes two or three centroids at a time, and where the last of a wave's places
hold no episode; the first and the last episode are equal, and so are two neighbours: the lower one is matched."""
import numpy as np
import pytest

from oracle import epicache_oracle as orc
from tests.test_gpu_episodes import COS_TOL, gpu_match

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [66, 100])
@pytest.mark.parametrize("nq", [1, 512, 513])
@pytest.mark.parametrize("E", [1, 2, 8, 9, 11, 12, 13, 16, 17, 24, 25, 36, 37])
def test_matching(E, nq, D):
    print(f"[gpu test] match E={E} queries={nq} D={D}", flush=True)
    rng = np.random.default_rng(E * 1000 + nq + D)
    cent = rng.standard_normal((E, D)).astype(np.float32)
    cent[E - 1] = cent[0]
    cent[E // 2] = cent[max(0, E // 2 - 1)]
    q = (cent[rng.integers(0, E, nq)] + 0.3 * rng.standard_normal((nq, D))).astype(np.float32)
    got, cs = gpu_match(q, cent, float("-inf"))
    want, o_cs = orc.match_queries(q, cent)
    np.testing.assert_allclose(cs, o_cs, atol=COS_TOL)
    for i in range(nq):
        assert not any(np.array_equal(cent[e], cent[got[i]]) for e in range(got[i])), i
        assert got[i] == want[i] or o_cs[i] - orc._cosine(q[i].astype(np.float64), cent[got[i]].astype(np.float64)) <= COS_TOL
