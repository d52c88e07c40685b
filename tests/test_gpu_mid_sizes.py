"""Single frames between the small- and large-input paths against the oracle
by the usual parity bar (bit-exact discrete results, scores to 1e-5): one-wave
selects and top-lambda with the outputs written there (above 3 * 2^16 points at
leaf caps up to 256, above 2^19 up to 512, with and without leaves of more than
256 P1 points), and the kNN, plan and voxel kernels of large inputs (above 2^19 points)."""
import numpy as np
import pytest

from paper_2512_10386_amd import synth
from tests.parity import compare, run_gpu

pytestmark = pytest.mark.gpu


def crowded(n, seed):
    """Surfaces with an over-full leaf (copies of one point) and far outliers."""
    xyz, _ = synth.sphere_plane(seed, n - n // 4 - 4000, n // 4 - 2000, 4000)
    xyz = np.concatenate([xyz, np.repeat(xyz[:1], 2000, 0)])
    return xyz[np.random.default_rng(seed).permutation(len(xyz))]


def tight_clusters(n, seed):
    """Clusters of 20 points far smaller than their spacing: a query's k = 32
    distances fall into two narrow bands."""
    rng = np.random.default_rng(seed)
    c = rng.uniform(0, 1, (n // 20, 1, 3))
    return (c + rng.normal(0, 1e-5, (n // 20, 20, 3))).reshape(-1, 3).astype(np.float32)


def test_banded_distances(oracle):
    from paper_2512_10386_amd.binding import Denoiser
    xyz = tight_clusters(530_000, 8)
    prm = dict(k=32, leaf_cap=256, stages=6)
    ref = oracle.denoise(xyz, **prm)
    den = Denoiser(0, **prm)
    try:
        compare(run_gpu(den, xyz), ref)
    finally:
        den.close()


@pytest.mark.parametrize("make,k,cap,chunk", [
    (lambda: synth.lidar_frame(seed=3, n_az=3073)[0], 12, 256, 0),      # 196,672 points: just above 3 * 2^16
    (lambda: crowded(270_001, 4), 16, 256, 0),
    (lambda: crowded(540_001, 4), 8, 512, 1500),                     # chunked leaves in the parallel plan
    (lambda: crowded(196_608, 5), 16, 256, 0),                       # 3 * 2^16: workgroup selects
    (lambda: synth.lidar_frame(seed=6, n_az=8193)[0], 12, 512, 0)])     # 524,352 points: just above 2^19
def test_mid_sizes(oracle, make, k, cap, chunk):
    from paper_2512_10386_amd.binding import Denoiser
    xyz = np.ascontiguousarray(make())
    ref = oracle.denoise(xyz, k=k, leaf_cap=cap)
    den = Denoiser(0, k=k, leaf_cap=cap, knn_chunk=chunk)
    try:
        compare(run_gpu(den, xyz), ref)
    finally:
        den.close()


@pytest.mark.parametrize("n,prm", [
    (6000, dict(leaf_cap=2)), (6000, dict(leaf_cap=31)), (6000, dict(leaf_cap=33)),
    (60_000, dict(leaf_cap=256)), (60_000, dict(leaf_cap=257)), (60_000, dict(leaf_cap=512)),
    (60_000, dict(leaf_cap=513)), (60_000, dict(leaf_cap=1024)), (60_000, dict(leaf_cap=1025)),
    (60_000, dict(leaf_cap=300, min_leaf_side=0.3))])
def test_voxel_tables(oracle, n, prm):
    """The voxel filter's table sizes at the edges of their leaf caps, with
    over-full leaves (copies of one point; a minimum leaf side)."""
    from paper_2512_10386_amd.binding import Denoiser
    xyz = np.ascontiguousarray(crowded(n, n + prm["leaf_cap"]) if n > 8000 else
                               synth.sphere_plane(prm["leaf_cap"], n - 2000, 1500, 500)[0])
    ref = oracle.denoise(xyz, **prm)
    den = Denoiser(0, **prm)
    try:
        compare(run_gpu(den, xyz), ref)
    finally:
        den.close()


@pytest.mark.parametrize("n,prm", [
    (22_528, dict(leaf_cap=10)), (22_528, dict(leaf_cap=11)),        # the plan kernel, the halo kernel's plan
    (22_528, dict(leaf_cap=256, knn_chunk=16)),                      # too many partial lists: planned again
    (22_528, dict(leaf_cap=256, knn_chunk=11_264)),                  # at most two chunks: no plan kernel
    (22_528, dict(leaf_cap=256, knn_chunk=11_263)),
    (22_528, dict(leaf_cap=256, knn_chunk=1500)),                    # chunked leaves that fit
    (4_000, dict(leaf_cap=1, min_vox_count=1)), (4_000, dict(min_vox_count=50))])
def test_plan_in_halo(oracle, n, prm):
    """The kNN plan by the halo kernel and where the plan kernel takes over."""
    from paper_2512_10386_amd.binding import Denoiser
    xyz = np.ascontiguousarray(synth.sphere_plane(5, n - 3000, 2000, 1000)[0])
    ref = oracle.denoise(xyz, **{a: v for a, v in prm.items() if a != "knn_chunk"})
    den = Denoiser(0, **prm)
    try:
        compare(run_gpu(den, xyz), ref)
    finally:
        den.close()


@pytest.mark.parametrize("nf,chunk", [(10, 0), (11, 0), (11, 20_000)])
def test_queue_order_sizes(nf, chunk):
    """Batches on both sides of the size (2^21 points) above which the kNN
    queue is in leaf order, with and without chunked leaves, against the plain
    call of each frame."""
    import torch
    from paper_2512_10386_amd.binding import BatchDenoiser, Denoiser
    two = [synth.lidar_frame(seed=s, n_az=3100)[0] for s in (1, 2)]  # 198,400 points each
    frames = [two[f % 2] for f in range(nf)]
    off = torch.tensor(np.concatenate([[0], np.cumsum([len(f) for f in frames])]), dtype=torch.int64, device="cuda")
    x = torch.from_numpy(np.concatenate(frames)).cuda()
    assert (len(x) > 2 ** 21) == (nf == 11)
    prm = dict(k=16, leaf_cap=512, knn_chunk=chunk)
    bd, den = BatchDenoiser(0, **prm), Denoiser(0, **prm)
    try:
        out = bd.alloc(len(x), nf)
        bd(x, off, out)
        ref = [den(torch.from_numpy(f).cuda()) for f in two]
        for f in range(nf):
            a, b, r = int(off[f]), int(off[f + 1]), ref[f % 2]
            m = int(r.n_kept)
            assert torch.equal(out.keep[a:b], r.keep) and torch.equal(out.stage[a:b], r.stage)
            assert torch.equal(out.score[a:b].view(torch.int32), r.score.view(torch.int32))
            assert int(out.n_kept[f]) == m and torch.equal(out.kept_idx[a:a + m], r.kept_idx[:m])
    finally:
        bd.close()
        den.close()


@pytest.mark.parametrize("n", [16_383, 16_384, 16_385, 114_687, 114_689, 1_048_575, 1_048_577])
def test_sort_tiles(n):
    """The order of the radix passes at the edges of their tile sizes: by key
    bits 32..62, then by original index."""
    import torch
    from paper_2512_10386_amd.binding import Denoiser
    rng = np.random.default_rng(n)
    xyz = torch.from_numpy(rng.uniform(0, 1, (n, 3)).astype(np.float32)).cuda()
    xyz[n // 2:n // 2 + 400] = xyz[0]
    den = Denoiser(0, k=4, leaf_cap=1024)
    try:
        den(xyz)
        order = den.dump("ORDER", n).cpu().numpy().view(np.uint32)
        key = den.dump("KEYS", n).cpu().numpy().view(np.uint64)
        assert int(den.dump("STATUS", n).cpu().numpy()[0]) == 0
    finally:
        den.close()
    assert np.array_equal(order, np.lexsort((np.arange(n), key >> np.uint64(32))))


@pytest.mark.parametrize("nf,n", [(2, 30_000), (3, 200_000), (300, 1_050_000)])
def test_sort_tiles_of_batches(nf, n):
    """The same with the frame passes of a batch."""
    import torch
    from paper_2512_10386_amd.binding import BatchDenoiser
    rng = np.random.default_rng(nf)
    xyz = torch.from_numpy(rng.uniform(0, 1, (n, 3)).astype(np.float32)).cuda()
    cut = np.sort(rng.integers(0, n + 1, nf - 1))
    off = np.concatenate([[0], cut, [n]])
    den = BatchDenoiser(0, k=4, leaf_cap=1024)
    try:
        den(xyz, torch.tensor(off, dtype=torch.int64, device="cuda"))
        order = den.dump("ORDER", n).cpu().numpy().view(np.uint32)
        key = den.dump("KEYS", n).cpu().numpy().view(np.uint64)
    finally:
        den.close()
    frame = np.repeat(np.arange(nf), np.diff(off))
    assert np.array_equal(order, np.lexsort((np.arange(n), key >> np.uint64(32), frame)))


@pytest.mark.parametrize("one_point", [False, True])
@pytest.mark.parametrize("cap,chunk", [(5000, 5000), (5000, 4999), (4999, 5000), (4999, 4999)])
def test_skipped_launches(oracle, one_point, cap, chunk):
    """Chunk lengths and leaf caps around the number of points: where no leaf
    can have two chunks, and no cell more points than a leaf."""
    from paper_2512_10386_amd.binding import Denoiser
    rng = np.random.default_rng(7)
    xyz = np.ones((5000, 3), np.float32) if one_point else rng.normal(size=(5000, 3)).astype(np.float32)
    ref = oracle.denoise(xyz, leaf_cap=cap, min_vox_count=1)
    den = Denoiser(0, leaf_cap=cap, min_vox_count=1, knn_chunk=chunk)
    try:
        compare(run_gpu(den, xyz), ref)
    finally:
        den.close()


@pytest.mark.parametrize("nf", [1, 2, 64, 65, 300])
def test_frame_counts(nf):
    """Batches at the edges of the key kernel's frame counts, with empty frames,
    against the plain call of each frame."""
    import torch
    from paper_2512_10386_amd.binding import BatchDenoiser, Denoiser
    rng = np.random.default_rng(nf)
    sizes = rng.integers(0, 300, nf)
    sizes[-1] = 5000
    frames = [(rng.normal(size=(m, 3)) * rng.uniform(0.1, 9)).astype(np.float32) for m in sizes]
    off = np.concatenate([[0], np.cumsum(sizes)])
    x = torch.from_numpy(np.concatenate(frames)).cuda()
    prm = dict(k=8, leaf_cap=64, min_vox_count=2)
    bd, den = BatchDenoiser(0, **prm), Denoiser(0, **prm)
    try:
        out = bd.alloc(len(x), nf)
        bd(x, torch.tensor(off, dtype=torch.int64, device="cuda"), out)
        assert int(bd.dump("STATUS", len(x)).cpu().numpy()[0]) == 0
        for f in range(nf):
            if not sizes[f]:
                assert int(out.n_kept[f]) == 0
                continue
            r = den(x[off[f]:off[f + 1]].contiguous())
            assert torch.equal(out.keep[off[f]:off[f + 1]], r.keep)
            assert torch.equal(out.score[off[f]:off[f + 1]].view(torch.int32), r.score.view(torch.int32))
            assert int(out.n_kept[f]) == int(r.n_kept)
    finally:
        bd.close()
        den.close()


def test_over_full_leaves_beside_waves(oracle):
    """Leaves above 256 points (copies of one point) where the voxel filter and
    the selects of the others run a wave each."""
    from paper_2512_10386_amd.binding import Denoiser
    xyz = np.ascontiguousarray(crowded(540_001, 9))
    xyz[:700] = xyz[5000]
    ref = oracle.denoise(xyz, k=8, leaf_cap=256)
    den = Denoiser(0, k=8, leaf_cap=256)
    try:
        g = run_gpu(den, xyz)
        assert (g["leaf_end"] - g["leaf_begin"]).max() > 512
        compare(g, ref)
    finally:
        den.close()
