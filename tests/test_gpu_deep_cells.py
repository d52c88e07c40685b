"""The re-sort of level-10 cells that split further, at the sizes where its
form changes (one wave up to 64 points, LDS up to 1024, memory above), against
the oracle by the usual parity bar (the exact order inside them included)."""
import numpy as np
import pytest

from tests.parity import compare, run_gpu

pytestmark = pytest.mark.gpu


def clustered(sizes, seed):
    """Clusters of the given sizes, each inside one level-10 cell of the unit
    cube, with a few points in the cells beside them and copies of single
    points among them."""
    rng = np.random.default_rng(seed)
    pts = [np.array([[0, 0, 0], [1, 1, 1]], np.float64), rng.uniform(0, 1, (500, 3))]
    for m in sizes:
        cell = rng.integers(40, 980, 3)
        c = (cell + rng.uniform(0.05, 0.95, (m, 3))) / 1024.0
        c[: m // 8] = c[-1]
        side = (cell + rng.integers(-1, 2, (12, 3)) + rng.uniform(0.1, 0.9, (12, 3))) / 1024.0
        pts += [c, side]
    xyz = np.concatenate(pts).astype(np.float32)
    return xyz[rng.permutation(len(xyz))]


@pytest.mark.parametrize("sizes,cap", [
    ((3, 17, 40, 63, 64, 65, 66, 200), 2), ((300, 1023, 1024, 1025, 255, 256, 257), 60), ((4000, 1024, 1025, 2048), 700),
    ((64,) * 40 + (65,) * 40, 30)])
def test_deep_cells(oracle, sizes, cap):
    from paper_2512_10386_amd.binding import Denoiser
    xyz = clustered(sizes, len(sizes))
    ref = oracle.denoise(xyz, k=8, leaf_cap=cap)
    assert int(ref["leaf_level"].max()) > 10
    den = Denoiser(0, k=8, leaf_cap=cap)
    try:
        compare(run_gpu(den, xyz), ref)
    finally:
        den.close()
