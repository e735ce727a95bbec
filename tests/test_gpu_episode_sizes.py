"""Episode geometry where its kernels change form: more segments than one member list holds, rows that are no multiple
of a vector, one segment, one dimension block more or less."""
import numpy as np
import pytest

from oracle import epicache_oracle as orc
from tests.test_gpu_episodes import COS_TOL, clustered, gpu_match, gpu_medoids

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,D,E", [(1, 64, 1), (4096, 65, 3), (4097, 100, 2), (9000, 66, 5), (700, 1020, 24), (300, 260, 300)])
def test_medoids_and_matching(K, D, E):
    print(f"[gpu test] episodes K={K} D={D} E={E}", flush=True)
    emb, assign = clustered(K + D, K, D, E)
    cent, med = gpu_medoids(emb, assign, E)
    o_cent, o_med = orc.episode_medoids(emb, assign, E)
    np.testing.assert_allclose(cent, o_cent, rtol=1e-5, atol=1e-6)
    for e in range(E):
        if med[e] != o_med[e]:
            assert med[e] >= 0 and assign[med[e]] == e
            gap = orc._cosine(emb[o_med[e]].astype(np.float64), o_cent[e]) - \
                  orc._cosine(emb[med[e]].astype(np.float64), o_cent[e])
            assert 0 <= gap <= COS_TOL
    q = emb[:min(K, 50)] + np.float32(0.1)
    got, cs = gpu_match(q, cent, float("-inf"))
    want, o_cs = orc.match_queries(q, cent)
    np.testing.assert_allclose(cs, o_cs, atol=COS_TOL)
    for i in np.nonzero(got != want)[0]:
        assert o_cs[i] - orc._cosine(q[i].astype(np.float64), cent[got[i]].astype(np.float64)) <= COS_TOL
