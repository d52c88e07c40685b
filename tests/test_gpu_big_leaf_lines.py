"""Both sides of the lines between the per-leaf kernels and those for big leaves
that go by the size of the frames: small frames on average (1024 points), frames
split into leaves that are not big (caps of 2400 and 4096). Frames against the
oracle by the usual parity bar, batches against plain calls bit for bit."""
import numpy as np
import pytest

from paper_2512_10386_amd import synth
from tests.parity import compare, run_gpu

pytestmark = pytest.mark.gpu


def scene(n):
    return synth.sphere_plane(n, n - n // 2, n // 2 - n // 10, n // 10)[0]


def sweep(n):
    return synth.lidar_frame(seed=n, n_az=-(-n // 64))[0][:n]


def clustered(n):
    """Nine points in ten in one corner: a leaf near the cap, far above an eighth of the frame."""
    g = np.random.default_rng(n)
    x = g.random((n, 3))
    x[n // 10:] *= 0.04
    return x.astype(np.float32)


@pytest.mark.parametrize("make,n,cap", [
    (sweep, 19_207, 4096), (sweep, 19_208, 4096), (scene, 19_208, 4097), (scene, 12_000, 2400), (scene, 40_000, 2401),
    (clustered, 9_000, 4096), (clustered, 30_000, 4096), (scene, 4_097, 4096), (scene, 4_096, 4096)])
def test_frames_around_the_lines(oracle, make, n, cap):
    from paper_2512_10386_amd.binding import Denoiser
    xyz, prm = np.ascontiguousarray(make(n)), dict(k=16, leaf_cap=cap)
    den = Denoiser(0, **prm)
    try:
        compare(run_gpu(den, xyz), oracle.denoise(xyz, **prm))
    finally:
        den.close()


@pytest.mark.parametrize("sizes,cap", [
    ([1024] * 12, 5000), ([1025] * 12, 5000), ([9000] + [100] * 20, 9000), ([2500, 1, 700] * 4, 4096), ([5000] * 5, 4096)])
def test_batches_around_the_lines(sizes, cap):
    import torch
    from paper_2512_10386_amd.binding import BatchDenoiser, Denoiser
    frames = [scene(max(n, 20))[:n] if i % 2 else sweep(n) for i, n in enumerate(sizes)]
    off = torch.tensor(np.concatenate([[0], np.cumsum(sizes)]), dtype=torch.int64, device="cuda")
    x = torch.from_numpy(np.ascontiguousarray(np.concatenate(frames))).cuda()
    prm = dict(k=12, leaf_cap=cap)
    bd, den = BatchDenoiser(0, **prm), Denoiser(0, **prm)
    try:
        out = bd(x, off)
        for f in range(len(sizes)):
            a, b = int(off[f]), int(off[f + 1])
            r = den(x[a:b].contiguous())
            assert torch.equal(out.keep[a:b], r.keep) and torch.equal(out.stage[a:b], r.stage)
            assert torch.equal(out.score[a:b].view(torch.int32), r.score.view(torch.int32))
    finally:
        bd.close()
        den.close()
