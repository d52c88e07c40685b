"""kNN above 2^19 points (pending buffers of positions, final lists written from
registers) with lists that a buffer of 64 cannot hold beside the query itself:
batches of frames against the same frames in plain calls, which keep keys.
Neighbours, distances, densities and outputs bit for bit."""
import numpy as np
import pytest

from paper_2512_10386_amd import synth

pytestmark = pytest.mark.gpu


def sweeps(n, seed):
    return synth.lidar_frame(seed=seed, n_az=-(-n // 64))[0][:n].astype(np.float32)


def lattice(n, seed):
    """Copies and equal distances: ties at every list's end."""
    return np.random.default_rng(seed).integers(0, 40, (n, 3)).astype(np.float32)


@pytest.mark.parametrize("make,k,cap,chunk", [
    (sweeps, 33, 512, 0), (sweeps, 48, 1024, 0), (sweeps, 63, 256, 0), (sweeps, 64, 512, 0), (lattice, 64, 512, 0),
    (lattice, 40, 256, 0), (sweeps, 64, 1024, 700), (sweeps, 31, 512, 0)])
def test_long_lists_above_2_19(make, k, cap, chunk):
    import torch
    from paper_2512_10386_amd.binding import BatchDenoiser, Denoiser
    sizes = [130_000, 99_991, 1, 120_001, 100_003, 90_007]
    assert (1 << 19) < sum(sizes) < (1 << 20)
    frames = [make(n, f) for f, n in enumerate(sizes)]
    off = torch.tensor(np.concatenate([[0], np.cumsum(sizes)]), dtype=torch.int64, device="cuda")
    x = torch.from_numpy(np.concatenate(frames)).cuda()
    prm = dict(k=k, leaf_cap=cap)
    bd, den = BatchDenoiser(0, knn_chunk=chunk, **prm), Denoiser(0, **prm)
    try:
        print(f"[positions] k={k} cap={cap}", flush=True)
        out = bd(x, off)
        n = sum(sizes)
        idx, d2 = bd.dump("NBR_IDX", n).view(n, k), bd.dump("NBR_D2", n).view(n, k)
        rho, f64 = bd.dump("RHO", n), bd.dump("SCORE64", n)
        for f, m in enumerate(sizes):
            a, b = int(off[f]), int(off[f + 1])
            r = den(x[a:b].contiguous())
            ri, rd = den.dump("NBR_IDX", m).view(m, k), den.dump("NBR_D2", m).view(m, k)
            got = idx[a:b].clone()
            got[got != -1] -= a
            assert torch.equal(got, ri) and torch.equal(d2[a:b].view(torch.int32), rd.view(torch.int32)), f
            assert torch.equal(rho[a:b].view(torch.int64), den.dump("RHO", m).view(torch.int64)), f
            assert torch.equal(out.keep[a:b], r.keep) and torch.equal(out.stage[a:b], r.stage), f
            assert torch.equal(out.score[a:b].view(torch.int32), r.score.view(torch.int32)), f
            assert torch.equal(f64[a:b].view(torch.int64), den.dump("SCORE64", m).view(torch.int64)), f
    finally:
        bd.close()
        den.close()
