"""The static pattern of meshes with a vertex in many tets: the rows of the
pattern are sorted and freed of copies by a wavefront in LDS up to 256 keys, by
one lane above.  The oracle is the set of vertex pairs that share a tet."""
import numpy as np
import pytest

from paper_2512_12151_amd import bfal
from scenes.configs import _finish

pytestmark = pytest.mark.gpu


def _fan(k):
    """k tets around the edge (0, 1), from vertex 0 below to vertex 1 above a
    ring of k vertices: row 0 has 3 k keys, k + 1 of them different."""
    a = 2.0 * np.pi * np.arange(k) / k
    rest = np.vstack([[0, 0, -0.5], [0, 0, 0.5], np.stack([np.cos(a), np.sin(a), 0 * a], 1)])
    ring = 2 + np.arange(k)
    tets = np.stack([np.zeros(k, int), ring, np.roll(ring, -1), np.ones(k, int)], 1)
    e = rest[tets[:, 1:]] - rest[tets[:, :1]]
    flip = np.linalg.det(e) < 0
    tets[flip, 1], tets[flip, 2] = tets[flip, 2].copy(), tets[flip, 1].copy()
    fixed = np.zeros(len(rest), np.uint8)
    fixed[0] = 1
    return _finish("fan", 0, rest, tets.astype(np.int32), np.full(k, 1e5), np.full(k, 0.3), np.full(k, 1000.0), fixed,
                   rest.copy(), rest.copy(), rest.copy(), 0.01, np.zeros((0, 4)), np.zeros((0, 4)), np.zeros(0), 1e4,
                   1e-3, 1e-5)


@pytest.mark.parametrize("k", [3, 21, 22, 43, 85, 86, 200])   # 9, 63, 66, 129, 255, 258 and 600 keys
def test_static_pattern_of_a_fan(k):
    sc = _fan(k)
    pb = bfal.Problem.from_scene(bfal.Context(0), sc)
    pb.newton_step(tol=1e-5)
    row_ptr, col = (np.asarray(v) for v in pb.pattern()[:2])
    pairs = {(int(min(i, j)), int(max(i, j))) for t in sc["tets"] for i in t for j in t}
    for r in range(len(row_ptr) - 1):
        want = sorted(j for i, j in pairs if i == r)
        assert col[row_ptr[r]:row_ptr[r + 1]].tolist() == want, f"row {r}"
