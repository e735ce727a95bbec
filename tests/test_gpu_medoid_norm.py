"""The medoid where two members' cosines agree to the last bits of fp32: the centroid's squared norm is one sum per lane over every
64th dim, by fma, then the tree over the lanes, in every form of the kernel.  All else of these clusters is exact in fp32 (whole
numbers below 2^24 and their quarters), so the norm's last bit decides, and the clusters are those whose medoid another order of
the sum would change."""
import numpy as np
import pytest

from tests.test_gpu_episodes import gpu_medoids

pytestmark = pytest.mark.gpu


def wave_tree(x):
    while x.shape[-1] > 1:
        x = x[..., 0::2] + x[..., 1::2]
    return x[..., 0]


def squared_norm(c, by_four):
    """Lane l sums dims l, l + 64, .. in order; by_four: four consecutive dims a lane, the last of them first.  Squares and sums are
    exact in float64 here, so that rounding them once is the fma."""
    c = np.pad(c.astype(np.float64), ((0, 0), (0, -c.shape[1] % 256)))
    terms = c.reshape(len(c), -1, 64, 4)[..., ::-1].transpose(0, 1, 3, 2).reshape(len(c), -1, 64) if by_four \
        else c.reshape(len(c), -1, 64)
    lanes = np.zeros((len(c), 64), np.float32)
    for i in range(terms.shape[1]):
        lanes = (lanes + terms[:, i] ** 2).astype(np.float32)
    return wave_tree(lanes)


def close_clusters(seed, dim, tries=8000):
    """Clusters of four members [n, 4, dim] of which the first two are equally close to the centroid up to rounding, and which of
    them is the closest: with the norm as it is summed, and by fours."""
    rng = np.random.default_rng(seed)
    a = rng.integers(-15, 16, (tries, 32))
    b = a + rng.integers(-1, 2, (tries, 32)) * (rng.random((tries, 32)) < 0.06)
    pairs = (dim - 32) // 2
    # the other two lie far off to both sides; their sum makes the centroid long without being like either of them
    h = np.repeat(rng.integers(-2048, 2048, (tries, pairs)), 2, axis=1)
    off = np.repeat(rng.integers(2**22, 2**23 - 2**12, (tries, pairs)), 2, axis=1)
    off[:, 1::2] *= -1
    rows = np.zeros((tries, 4, dim), np.float32)
    rows[:, 0, :32], rows[:, 1, :32] = a, b
    rows[:, 2, 32:32 + 2 * pairs], rows[:, 3, 32:32 + 2 * pairs] = h + off, h - off
    cent = (rows.astype(np.float64).sum(1) / 4).astype(np.float32)
    near = rows[:, :2, :32].astype(np.float64)
    dot = np.einsum("nkd,nd->nk", near, cent[:, :32].astype(np.float64)).astype(np.float32)
    sq = (near ** 2).sum(-1).astype(np.float32)

    def closest(norm):
        cos = dot / (np.sqrt(sq) * np.sqrt(norm)[:, None])
        return np.argmax(cos, axis=1)   # the first of equal ones
    ours, other = closest(squared_norm(cent, False)), closest(squared_norm(cent, True))
    far = np.abs(np.einsum("nd,nd->n", rows[:, 2].astype(np.float64), cent)) / np.linalg.norm(rows[:, 2].astype(np.float64), axis=1)
    take = (ours != other) & (2 * far < (dot / np.sqrt(sq)).min(axis=1))
    return rows[take], cent[take], ours[take]


@pytest.mark.parametrize("dim,clusters,strays", [(384, 0, 0), (512, 6, 3000), (301, 0, 0), (300, 9, 5000), (1024, 0, 0),
                                                 (384, 260, 0), (2052, 0, 0), (2051, 4, 900)])
def test_the_norm_decides(dim, clusters, strays):
    """clusters: how many of them, the rest without a member (0: as many as were found); strays: segments of no cluster, which
    bring more workgroups to each."""
    rows, cent, closest = close_clusters(dim, dim)
    found = len(rows)
    assert found >= 10
    if 0 < clusters < found:
        rows, cent, closest, found = rows[:clusters], cent[:clusters], closest[:clusters], clusters
    episodes = max(found, clusters)
    print(f"[gpu test] medoid norm dim={dim} clusters={episodes} strays={strays}", flush=True)
    rng = np.random.default_rng(dim + 1)
    emb = rng.standard_normal((4 * found + strays, dim)).astype(np.float32)
    assign = np.full(len(emb), -1, np.int32)
    at = np.sort(rng.permutation(len(emb))[:4 * found].reshape(found, 4), axis=1)
    for e in range(found):
        emb[at[e]], assign[at[e]] = rows[e], e
    got_cent, got = gpu_medoids(emb, assign, episodes)
    np.testing.assert_array_equal(got_cent[:found], cent)
    np.testing.assert_array_equal(got[:found], at[np.arange(found), closest])
    assert (got[found:] == -1).all()
