"""Single frames small enough for the one-workgroup octree kernel, at the
edges of its variants (1024, 2048 and 4096 points) and of a wave, against the
oracle by the usual parity bar (bit-exact discrete results, scores to 1e-5):
surfaces, copies of one point, and tight clusters beside a far outlier, whose
level-10 cells and their neighbours are re-sorted on the whole key."""
import numpy as np
import pytest

from paper_2512_10386_amd import synth
from tests.parity import compare, run_gpu

pytestmark = pytest.mark.gpu


def surface(n, rng):
    xyz = rng.normal(size=(n, 3))
    return xyz / np.maximum(np.linalg.norm(xyz, axis=1, keepdims=True), 1e-9) + rng.normal(0, 0.01, (n, 3))


def copies(n, rng):
    xyz = np.tile(rng.normal(size=(1, 3)), (n, 1))
    xyz[n // 2:] = rng.normal(size=(n - n // 2, 3))
    return xyz


def deep(n, rng):
    """A tight cluster on the border of a level-10 cell, loose points around
    it that fall into the cells next to it, and a few outliers 1000 cells
    away (they fix the root cube)."""
    far = rng.uniform(0, 1, (min(n, 6), 3))
    m = max(0, n - len(far))
    near = 0.5 + rng.normal(0, 1e-4, (m // 2, 3))
    loose = 0.5 + rng.normal(0, 2e-3, (m - m // 2, 3))
    return np.concatenate([far, near, loose])


@pytest.mark.parametrize("make", [surface, copies, deep])
@pytest.mark.parametrize("n", [1, 2, 63, 65, 512, 1023, 1024, 1025, 2047, 2048, 2049, 4095, 4096, 4097])
@pytest.mark.parametrize("prm", [dict(), dict(k=8, leaf_cap=16), dict(k=4, leaf_cap=1, min_vox_count=1),
                                 dict(leaf_cap=64, min_leaf_side=0.0004)])
def test_small_frames(oracle, make, n, prm):
    from paper_2512_10386_amd.binding import Denoiser
    rng = np.random.default_rng(n)
    xyz = make(n, rng)[rng.permutation(n)].astype(np.float32)
    ref = oracle.denoise(xyz, **prm)
    den = Denoiser(0, **prm)
    try:
        compare(run_gpu(den, xyz), ref)
    finally:
        den.close()
