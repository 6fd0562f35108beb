"""Morton order bit-exact at the sizes where the sort and the scans change form
(counted up to 8,192 pairs, tile counts added in the scatter up to 65,536,
scanned above), with tied keys, and for several geometries of uneven size."""
import numpy as np
import pytest

from gpu_util import leaf_table_from_gpu, say

pytestmark = pytest.mark.gpu


def _mesh(n, seed):
    """n triangles of an icosphere, a sixteenth of them copies moved by 1e-9
    of one of the others (tied keys: below the resolution of 21 bits)."""
    from synthetic import icosphere, with_near_duplicates
    level = 0
    while 20 * 4 ** level < n:
        level += 1
    V, T = icosphere(level)
    d = n // 16
    T = T[np.sort(np.random.default_rng(seed).choice(T.shape[0], n - d, replace=False))]
    return with_near_duplicates(V, T, d, 1e-9, seed) if d else (V, T)


@pytest.mark.parametrize("n", [2, 63, 64, 65, 4096, 4097, 8191, 8192, 8193, 65536, 65537])
def test_order_at_sort_edges(n):
    import paper_1806_11558_amd as hm
    from oracle import bem, cluster
    V, T = _mesh(n, 3)
    say("order", n)
    H = hm.HMatrix(V, T, leaf_size=64, eps=1e-4, precision="f32")
    C = bem.centroids(V, T.astype(np.int64))
    keys = cluster.morton_keys(C)
    assert np.array_equal(H.morton_keys(), keys)
    assert n < 32 or np.unique(keys).size < n                 # there are ties
    assert np.array_equal(H.perm(), cluster.morton_order(keys).astype(np.int32))
    if n <= 4097:
        P = cluster.Partition(C, 64, 1.0)
        assert np.array_equal(H.boxes(), P.boxes)
        assert np.array_equal(leaf_table_from_gpu(H), P.leaf_table())
    H.free()


@pytest.mark.parametrize("sizes", [(1, 4097, 7, 300, 1), (70000, 33, 2000)])
def test_order_of_uneven_geometries(sizes):
    import paper_1806_11558_amd as hm
    from oracle import bem, cluster
    meshes = [_mesh(n, 5 + g) for g, n in enumerate(sizes)]
    say("uneven geometries", sizes)
    H = hm.HMatrix.batch(meshes, leaf_size=64, eps=1e-4, precision="f32")
    keys, perm = H.morton_keys(), H.perm()
    for g, (V, T) in enumerate(meshes):
        a, b = H.offsets[g], H.offsets[g + 1]
        k = cluster.morton_keys(bem.centroids(V, T.astype(np.int64)))
        assert np.array_equal(keys[a:b], k)
        assert np.array_equal(perm[a:b], (cluster.morton_order(k) + a).astype(np.int32))
    H.free()
