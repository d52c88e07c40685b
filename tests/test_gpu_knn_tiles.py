"""kNN work items of 1, 2, 4 and 8 queries (chosen by the number of P1 points)
against the oracle by the usual parity bar: bit-exact neighbour sets and
distances, scores to 1e-5. With the voxel filter off every point is in P1, so
the sizes sit exactly on the rule's edges."""
import pytest

from paper_2512_10386_amd import synth
from tests.parity import compare, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,k,cap,chunk", [
    (4096, 12, 256, 0), (4097, 12, 256, 0), (20_480, 16, 512, 0), (20_481, 16, 512, 0), (40_960, 32, 256, 0),
    (40_961, 32, 256, 0),
    # chunked leaves: partial lists of one- and two-query tiles, merged
    (4096, 33, 4096, 1024), (5000, 64, 5000, 700), (13, 12, 4, 3)])
def test_tile_sizes(oracle, n, k, cap, chunk):
    from paper_2512_10386_amd.binding import Denoiser
    xyz, _ = synth.uniform_cube(n, n)
    prm = dict(k=k, leaf_cap=cap, stages=6)
    ref = oracle.denoise(xyz, **prm)
    assert int(ref["p1"].sum()) == n
    den = Denoiser(0, knn_chunk=chunk, **prm)
    try:
        compare(run_gpu(den, xyz), ref)
    finally:
        den.close()


@pytest.mark.parametrize("n", [50_000, 262_144, 262_145])
def test_isolated_leaves(oracle, n):
    """Leaves of a few points beside dense ones (128 candidates and more per
    query): their queries are items of their own up to 2^18 points."""
    import numpy as np
    from paper_2512_10386_amd.binding import Denoiser
    rng = np.random.default_rng(n)
    m = n // 2000
    lone = rng.uniform(-1, 2, (m, 1, 3)) + rng.normal(0, 0.02, (m, 7, 3))
    dense = rng.uniform(0, 1, (n - 7 * m, 3)) * (1, 1, 0.02)
    xyz = np.concatenate([dense, lone.reshape(-1, 3)])[rng.permutation(n)].astype(np.float32)
    prm = dict(k=12, leaf_cap=1024, stages=6)
    ref = oracle.denoise(xyz, **prm)
    den = Denoiser(0, **prm)
    try:
        compare(run_gpu(den, xyz), ref)
    finally:
        den.close()


@pytest.mark.parametrize("n,k", [(16_384, 64), (16_385, 64), (65_536, 16), (65_537, 16), (196_608, 32), (196_609, 64)])
def test_waves_per_simd(oracle, n, k):
    """The edges of the four-query tiles and of the kernel for six waves."""
    from paper_2512_10386_amd.binding import Denoiser
    xyz, _ = synth.uniform_cube(n, n)
    prm = dict(k=k, leaf_cap=512, stages=6)
    ref = oracle.denoise(xyz, **prm)
    den = Denoiser(0, **prm)
    try:
        compare(run_gpu(den, xyz), ref)
    finally:
        den.close()


@pytest.mark.parametrize("scale", [1e-18, 1e-13, 1.0, 1e17])
def test_bound_scales(oracle, scale):
    """The kNN bound counts halvings by exponents: copies (distance 0), powers
    of two, and scales at which squared distances leave the normal range."""
    import numpy as np
    from paper_2512_10386_amd.binding import Denoiser
    g = np.stack(np.meshgrid(*[np.arange(12.0)] * 3, indexing="ij"), -1).reshape(-1, 3)
    rng = np.random.default_rng(3)
    xyz = np.concatenate([g, g[:300], 2.0 ** rng.integers(-6, 4, (3000, 3)), rng.uniform(0, 12, (2000, 3))])
    xyz = (xyz * scale).astype(np.float32)[rng.permutation(len(xyz))]
    prm = dict(k=16, leaf_cap=512, stages=6)
    ref = oracle.denoise(xyz, **prm)
    den = Denoiser(0, **prm)
    try:
        g = run_gpu(den, xyz)
        assert np.array_equal(g["nbr_idx"], ref["nbr_idx"]) and np.array_equal(g["nbr_d2"], ref["nbr_d2"])
    finally:
        den.close()
