"""Medoids on both sides of the rule for their workgroups: 256 clusters and one more, 2048 dims and more, clusters of one member,
of none, and of two equal members, of which the lower one is the medoid."""
import numpy as np
import pytest

from oracle import epicache_oracle as orc
from tests.test_gpu_episodes import COS_TOL, clustered, gpu_medoids

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,E,D", [(520, 256, 60), (520, 257, 60), (3000, 257, 34), (3000, 1000, 64), (90, 3, 2048), (90, 3, 2052),
                                   (200, 2, 4099), (65, 1, 2048), (64, 1, 8192)])
def test_medoids(K, E, D):
    print(f"[gpu test] medoids K={K} E={E} D={D}", flush=True)
    emb, assign = clustered(K + D, K, D, E)
    if E > 2:
        assign[assign == E - 1] = 0                   # nobody in the last cluster
        assign[np.nonzero(assign == 1)[0][1:]] = 0    # at most one in the second
    twin = np.nonzero(assign == 0)[0]
    emb[twin[-1]] = emb[twin[0]]
    cent, med = gpu_medoids(emb, assign, E)
    o_cent, o_med = orc.episode_medoids(emb, assign, E)
    np.testing.assert_allclose(cent, o_cent, rtol=1e-5, atol=1e-6)
    for e in range(E):
        if not (assign == e).any():
            assert med[e] == -1 and not cent[e].any()
        elif med[e] != o_med[e]:
            assert assign[med[e]] == e
            gap = orc._cosine(emb[o_med[e]].astype(np.float64), o_cent[e]) - \
                  orc._cosine(emb[med[e]].astype(np.float64), o_cent[e])
            assert 0 <= gap <= COS_TOL
    assert med[0] != twin[-1] or twin.size == 1
